"""Host check of the training kernel's weight-fragment reads (csrc/mlp_frag.h),
compiled with g++: over every pair of hidden widths it accepts, no wave reads
outside the matrix it asks for, or outside the buffer that the network holds
(W1, W2 and W2 transposed as halves)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_06250_amd", "csrc")

PROG = r"""
#include <algorithm>
#include <cstdio>
#include "mlp_frag.h"
int main() {
    int bad = 0, whole = 0;
    for (int nin_pad = 64; nin_pad <= 704; nin_pad += 64)
        for (int h1 = 64; h1 <= 256; h1 += 64)
            for (int h2 = 64; h2 <= 256; h2 += 64) {
                const FragLayout f = frag_layout(nin_pad, h1, h2);
                if (f.size * 8 != (int64_t)h1 * nin_pad + 2 * (int64_t)h2 * h1) ++bad;  // halves held
                const int64_t first[4] = {0, f.w2, f.w2t, f.size};
                const int rows[3] = {h1, h2, h1}, cols[3] = {nin_pad, h1, h2};
                const int waves[3] = {h1 / 32, std::max(h1, h2) / 32, h1 / 32};  // that read each
                for (int q = 0; q < 3; ++q) {
                    const int steps = cols[q] / 16;
                    if ((first[q + 1] - first[q]) * 8 != (int64_t)rows[q] * cols[q]) ++bad;
                    int64_t seen = 0;
                    for (int wave = 0; wave < waves[q]; ++wave)
                        for (int s = 0; s < steps + 12; ++s) {  // groups of four, up to two past the end
                            const int64_t at = first[q] + frag_column(wave, rows[q], steps) + frag_step(s, steps) * 64;
                            if (at < first[q] || at + 64 > first[q + 1]) ++bad;
                            if (wave >= rows[q] / 32 || s >= steps) continue;
                            ++seen;  // what is used: its own block and step
                            if (at != first[q] + ((int64_t)wave * steps + s) * 64) ++bad;
                        }
                    if (seen * 64 == first[q + 1] - first[q]) ++whole;
                }
            }
    std::printf("%d bad, %d whole\n", bad, whole);
    return bad != 0 || whole != 11 * 4 * 4 * 3;
}
"""


def test_no_wave_reads_outside_its_matrix(tmp_path):
    src = tmp_path / "frag.cpp"
    src.write_text(PROG)
    exe = tmp_path / "frag"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
