// The half weights of the gate network in MFMA-fragment order, as the training
// kernels read them (plain C++, no HIP types, so that it can be checked on the
// host).
//
// A matrix of N rows and K contracted columns is N/32 column blocks of K/16
// steps, 64 uint4 each; the network's buffer holds W1 (h1 x nin_pad), W2
// (h2 x h1) and W2 transposed (h1 x h2).  Wave v computes units 32 v .. + 31 of
// each layer from column block v: waves below h1/32 read W1 and W2 transposed,
// and those of either layer load ahead from W2.  A load that a matrix has no
// block or step for names its last one, and is not used.  (A branch around such
// loads costs the kernel of 20 us one more, in spilled registers.)
#pragma once

#include <stdint.h>

constexpr int frag_block(int block, int rows) { return block < rows / 32 ? block : rows / 32 - 1; }
constexpr int frag_step(int step, int steps) { return step < steps ? step : steps - 1; }
// First uint4 of a column block, from the matrix' first on.
constexpr int64_t frag_column(int block, int rows, int steps) { return (int64_t)frag_block(block, rows) * steps * 64; }

// First uint4 of W2 and of W2 transposed in the buffer, and its length.
struct FragLayout {
    int64_t w2, w2t, size;
};
constexpr FragLayout frag_layout(int nin_pad, int h1, int h2)
{
    const int64_t n1 = (int64_t)h1 * nin_pad / 8, n2 = (int64_t)h2 * h1 / 8;
    return FragLayout{n1, n1 + n2, n1 + 2 * n2};
}
