"""Host check of the NUFFT plan's short grids (csrc/nufft_grid.h, compiled with
g++): the rule against a direct count, and which of the whole, 1/8 and 1/64
grids every case of test_gpu_nufft_grids.py and test_gpu_nufft_lists.py runs
on, so that those keep reaching the kernels they are written for."""
import os
import subprocess

import numpy as np
import pytest

from synthetic import make_small_cube

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_06250_amd", "csrc")

PROG = r"""
#include <iostream>
#include <string>
#include "nufft_grid.h"
int main() {
    std::string line;
    while (std::getline(std::cin, line)) {
        std::vector<bool> occ;
        for (char c : line) occ.push_back(c == '1');
        const NufftStretch s = nufft_stretch(occ);
        std::cout << s.b1 << " " << s.p0 << "\n";
    }
}
"""


@pytest.fixture(scope="module")
def stretch(tmp_path_factory):
    d = tmp_path_factory.mktemp("stretch")
    (d / "s.cpp").write_text(PROG)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(d / "s"), str(d / "s.cpp")], check=True)

    def call(grids):
        text = "\n".join("".join("1" if o else "0" for o in g) for g in grids) + "\n"
        out = subprocess.run([str(d / "s")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return call


def _occupied(lam, w, nphi, dphi):
    """Grid points within 4 cells of a channel: n >= 2 nphi points of [0, 2 pi),
    channel j at 2 (lambda^2_j - lambda_0^2) dphi."""
    n = 16
    while n < 2 * nphi:
        n *= 2
    x = np.mod(2 * (lam - np.sum(w * lam) / np.sum(w)) * dphi, 2 * np.pi)[w > 0] * n / (2 * np.pi)
    d = np.abs(np.arange(n)[:, None] - x[None, :])
    return (np.minimum(d, n - d) < 4).any(1)


def _count(occ):
    """(b1, p0) by trying every start."""
    n = len(occ)
    for b1 in (6, 3):
        m = n >> b1
        if m < 16:
            continue
        fits = [p for p in range(n) if not np.roll(occ, -p)[m:].any() and occ[p]]
        if fits:
            return b1, fits
    return 0, [0]


def test_rule_by_direct_count(stretch):
    rng = np.random.default_rng(2)
    grids = []
    for n in (16, 64, 128, 256, 1024, 2048):
        for m in {1, 2, n // 64, n // 64 + 1, n // 8, n // 8 + 1, n // 2, n} - {0}:
            for start in (0, 3, n - 1, n // 2):
                occ = np.zeros(n, bool)
                occ[(start + np.arange(m)) % n] = rng.uniform(size=m) < 0.9
                occ[start] = occ[(start + m - 1) % n] = True
                grids.append(occ)
    for occ, (b1, p0) in zip(grids, stretch(grids)):
        want, starts = _count(occ)
        assert b1 == want and p0 in starts, (len(occ), np.flatnonzero(occ)[:5], b1, p0, want)


def _check_case(stretch, c, nphi, dphi, want):
    occ = _occupied(c["lambda2"], c["weights"], nphi, dphi)
    b1, p0 = stretch([occ])[0]
    assert b1 == want(len(occ)), (nphi, dphi, len(occ), b1)
    if b1:
        assert not np.roll(occ, -p0)[len(occ) >> b1:].any()


@pytest.mark.parametrize("nlos,nchan", [(1, 40), (37, 300)])
@pytest.mark.parametrize("nphi", [63, 100, 256, 401, 1000, 2001, 4001])
def test_short_grid_cases(stretch, nphi, nlos, nchan):
    """test_gpu_nufft_grids.py: 1/8 of the grid at step 0.05; at 0.002 1/64 from
    1024 points on, where that is 16."""
    c = make_small_cube(nlos, nchan, 3, seed=nphi + nlos, nflag=nchan // 20, nsrc=nlos // 3 + 1)
    _check_case(stretch, c, nphi, 0.05, lambda n: 3)
    _check_case(stretch, c, nphi, 0.002, lambda n: 6 if n >= 1024 else 3)


@pytest.mark.parametrize("nlos,nchan,nphi", [(37, 256, 16), (19, 256, 32), (21, 192, 64), (3, 4096, 40),
                                             (21, 384, 128), (9, 400, 200), (5, 64, 600), (5, 700, 1024),
                                             (5, 40, 1500), (5, 100, 4001)])
def test_list_cases(stretch, nlos, nchan, nphi):
    """test_gpu_nufft_lists.py: the whole grid at step 1, 1/8 at 0.05 from 128
    points on, where that is 16."""
    c = make_small_cube(nlos, nchan, 3, seed=nphi + nchan, nflag=nchan // 20, nsrc=nlos // 3 + 1)
    _check_case(stretch, c, nphi, 1.0, lambda n: 0)
    _check_case(stretch, c, nphi, 0.05, lambda n: 3 if n >= 128 else 0)
