// Forward and backward of the gate network in two launches (hidden widths up
// to 256; mlp.hip holds the separate kernels for wider networks).
//
// train_rows_kernel: a workgroup of eight waves takes 32 rows of the batch
// through input normalisation, both layers, the head with its loss and output
// gradient, dz2 and dz1, with the activations in LDS; wave v owns hidden units
// 32 v .. 32 v + 31 of each layer, so that its ReLU masks stay in registers.
// Weights are read in MFMA-fragment order (1 KB contiguous per load), four to
// eight K-steps ahead.  x, h1, dz2 and dz1 (half) go to memory in the fragment order
// of the weight-gradient products, whose contracted axis is the batch; column
// sums (bias gradients, W3 gradient, loss) are kept in registers over the
// workgroup's blocks of rows and written once.
// train_wgrad_kernel: dW1 = dz1^T x and dW2 = dz2^T h1 in 64 x 64 tiles, the
// batch shared by the eight waves of a workgroup (and, for large batches, by
// workgroups), partial sums added in order through LDS; the last workgroups
// add the column sums.
//
// What bounds it: latency.  At batch 1024, 576 -> 256 -> 256 the products are
// 1.3 GFLOP (about 1 us of the chip) and 32 workgroups each stream 550 KB of
// weights from L2.  rmsynth_mlp_grad of that batch: 93 us in fifteen kernels and
// two copies before, 29 us now (20 us for the rows: input 5.5, layer 1 3.5, the
// others 1.3 us each; 8.5 us for the weight gradients); batch 4096 129 -> 40 us.
// More than four weight fragments ahead (8: 25 us, 12: 30 us) spills registers.
#include "mlp.h"
#include "mlp_device.h"
#include "mlp_frag.h"

#include <algorithm>

namespace {

constexpr int RB = 32;        // rows per block
constexpr int TW = 8;         // waves per workgroup
constexpr int kMaxWg = 512;   // workgroups of train_rows_kernel (rows of column sums)
constexpr int TG = 4;         // weight fragments loaded ahead
// Channels / 64 of a row held at a time; a row with more is read twice, and every
// row takes the loads of whole groups.  Batch 1024, 4 / 5 / 6: 128 channels 25.5 /
// 26.4 / 27.0 us, 288 30.2 / 29.0 / 29.7, 330 31.3 / 32.7 / 30.8, 400 32.4 / 33.7 / 34.8.
constexpr int CI = 5;
constexpr int WT = 64;        // tile of the weight-gradient kernel

__device__ __forceinline__ f32x16_t mfma(uint4 a, uint4 b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a),
                                                  __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

struct Group {
    uint4 v[TG];
};
__device__ __forceinline__ void load_group(Group& g, const uint4* __restrict__ w, int s0, int ks)
{
#pragma unroll
    for (int i = 0; i < TG; ++i) g.v[i] = w[frag_step(s0 + i, ks) * 64];
}
// acc += A (LDS rows a, 16 columns per step) x the fragments at w; g holds the
// first TG of them.
__device__ __forceinline__ f32x16_t layer(const _Float16* a, const uint4* __restrict__ w, int ks, Group& g)
{
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    auto use = [&](const Group& q, int s0) {
#pragma unroll
        for (int i = 0; i < TG; ++i)
            if (s0 + i < ks) acc = mfma(*reinterpret_cast<const uint4*>(a + 16 * (s0 + i)), q.v[i], acc);
    };
    Group n;
    for (int s0 = 0; s0 < ks; s0 += 2 * TG) {
        load_group(n, w, s0 + TG, ks);
        use(g, s0);
        load_group(g, w, s0 + 2 * TG, ks);
        use(n, s0 + TG);
    }
    return acc;
}

// Four consecutive rows' halves of this lane's column, q-th group of the 32 x 32
// block (rows 8 q + 4 (lane >> 5) .. + 3), into the fragments of the column
// block: fragment (block, step) as in frag order, contracted axis = rows.
__device__ __forceinline__ void store_frag(uint4* __restrict__ F, int64_t frag0, int lane, int q, uint2 h)
{
    uint2* const p = reinterpret_cast<uint2*>(F + (frag0 + (q >> 1)) * 64 + (lane & 31) + 32 * (q & 1));
    p[lane >> 5] = h;
}

struct RowsArgs {
    const float *Q, *U;
    int64_t nvalid, nblk;  // rows, blocks of RB rows
    int nchan, nin_pad, h1, h2;
    const float* w;
    const uint4 *W1f, *W2f, *W2t;
    const float *b1, *b2, *b3;
    const _Float16* W3;
    float phi_scale;
    const float *phi_label, *det_label;
    uint4 *Xf, *H1f, *D1f, *D2f;
    float* part;  // [workgroup][gb1 | gb2 | gW3 (2 h2) | gb3 (2) | loss]
};

__global__ __launch_bounds__(64 * TW, 1) void train_rows_kernel(RowsArgs p)
{
    extern __shared__ float4 smem4[];
    const int LX = p.nin_pad + 8, L1 = p.h1 + 8, L2 = p.h2 + 8;  // row strides (halves)
    _Float16* const sx = reinterpret_cast<_Float16*>(smem4);
    _Float16* const s1 = sx + RB * LX;
    _Float16* const s2 = s1 + RB * L1;  // h2, then dz2
    float* const sg = reinterpret_cast<float*>(s2 + RB * L2);  // [RB][2] output gradient
    float* const sl = sg + 2 * RB;                             // [RB][3] head sums
    const int t = threadIdx.x, lane = t & 63, col = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool on1 = wave < p.h1 / 32, on2 = wave < p.h2 / 32;
    const int n1 = 32 * wave + col, n2 = n1;  // this lane's hidden unit of each layer
    const int ks0 = p.nin_pad / 16, ks1 = p.h1 / 16, ks2 = p.h2 / 16;
    const uint4* const w1 = p.W1f + (int64_t)wave * ks0 * 64 + lane;
    const uint4* const w2 = p.W2f + frag_column(wave, p.h2, ks1) + lane;
    const uint4* const wt = p.W2t + (int64_t)wave * ks2 * 64 + lane;
    const int64_t steps = 2 * p.nblk;  // 16-row steps of the batch
    const float bias1 = on1 ? p.b1[n1] : 0.0f, bias2 = on2 ? p.b2[n2] : 0.0f;
    const float w30 = on2 ? (float)p.W3[n2] : 0.0f, w31 = on2 ? (float)p.W3[p.h2 + n2] : 0.0f;
    float gb1 = 0.0f, gb2 = 0.0f, gw0 = 0.0f, gw1 = 0.0f, gb30 = 0.0f, gb31 = 0.0f, loss = 0.0f;

    for (int64_t blk = blockIdx.x; blk < p.nblk; blk += gridDim.x) {
        const int64_t b0 = blk * RB;
        Group g;
        if (on1) load_group(g, w1, 0, ks0);
        // x = [w Q | w U] / rms of rows 4 wave .. + 3; rows past the batch are
        // zero.  The channels of the four rows are loaded CI x 64 at a time
        // (channels past the end: the last one, weighted 0) and, when that is
        // all of them, kept for the second pass.
        const float *q[4], *u[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t b = b0 + 4 * wave + r, at = (b < p.nvalid ? b : p.nvalid - 1) * p.nchan;
            q[r] = p.Q + at;
            u[r] = p.U + at;
        }
        struct Chan {
            float q[CI][4], u[CI][4];
        } c;
        auto load_chan = [&](int j0) __attribute__((always_inline)) {
            float wj[CI];
#pragma unroll
            for (int i = 0; i < CI; ++i) {
                const int j = j0 + 64 * i + lane < p.nchan ? j0 + 64 * i + lane : p.nchan - 1;
                wj[i] = j0 + 64 * i + lane < p.nchan ? p.w[j] : 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    c.q[i][r] = q[r][j];
                    c.u[i][r] = u[r][j];
                }
            }
#pragma unroll
            for (int i = 0; i < CI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    c.q[i][r] = wj[i] == 0.0f ? 0.0f : wj[i] * c.q[i][r];
                    c.u[i][r] = wj[i] == 0.0f ? 0.0f : wj[i] * c.u[i][r];
                }
        };
        float ss[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int j0 = 0; j0 < p.nchan; j0 += 64 * CI) {
            load_chan(j0);
#pragma unroll
            for (int i = 0; i < CI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    ss[r] = __builtin_fmaf(c.q[i][r], c.q[i][r], __builtin_fmaf(c.u[i][r], c.u[i][r], ss[r]));
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int r = 0; r < 4; ++r) ss[r] += __shfl_xor(ss[r], off, 64);
        bool past[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            ss[r] = ss[r] > 0.0f ? 1.0f / sqrtf(ss[r] / (float)(2 * p.nchan))
                                 : (ss[r] == 0.0f ? 0.0f : ss[r]);  // 1 / rms; NaN stays NaN
            past[r] = b0 + 4 * wave + r >= p.nvalid;
        }
        // Column k of x, rows 4 wave .. + 3, to LDS and as 8 bytes of its fragment.
        // Columns k = first + 64 i + lane: fragment blocks advance by 2 i, the
        // rest is a 32-bit lane offset (at most 2^20 steps).
        char* const xf = reinterpret_cast<char*>(p.Xf + (2 * blk + (wave >> 2)) * 64);
        auto lane_off = [&](int a) {
            return (uint32_t)(((a >> 5) * steps * 64 + (a & 31) + 32 * ((wave >> 1) & 1)) * 16 + 8 * (wave & 1));
        };
        auto put = [&](int first, int j, uint32_t off, const float* v) __attribute__((always_inline)) {
            f16x2_t h[2];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const _Float16 a = half_of(past[r] ? 0.0f : v[r]);
                h[r >> 1][r & 1] = a;
                sx[(4 * wave + r) * LX + first + j + lane] = a;
            }
            *reinterpret_cast<uint2*>(xf + ((first >> 5) + (j >> 5)) * steps * 1024 + off) =
                make_uint2(__builtin_bit_cast(uint32_t, h[0]), __builtin_bit_cast(uint32_t, h[1]));
        };
        const uint32_t offq = lane_off(lane), offu = lane_off((p.nchan & 31) + lane);
        for (int j0 = 0; j0 < p.nchan; j0 += 64 * CI) {
            if (p.nchan > 64 * CI) load_chan(j0);
#pragma unroll
            for (int i = 0; i < CI; ++i) {
                float a[4], e[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    a[r] = c.q[i][r] * ss[r];
                    e[r] = c.u[i][r] * ss[r];
                }
                if (j0 + 64 * i + lane < p.nchan) {
                    put(0, j0 + 64 * i, offq, a);
                    put(p.nchan, j0 + 64 * i, offu, e);
                }
            }
        }
        const float zero[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (2 * p.nchan + lane < p.nin_pad)  // fewer than 64 columns
            put(2 * p.nchan, 0, lane_off((2 * p.nchan & 31) + lane), zero);
        __syncthreads();

        // Layer 1.
        f32x16_t z1;
        uint32_t m1 = 0;
        if (on1) {
            z1 = layer(sx + col * LX + 8 * half, w1, ks0, g);
            load_group(g, w2, 0, ks1);  // (also without on2)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f16x2_t h[2];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float z = z1[4 * q + i] + bias1;
                    if (z > 0.0f) m1 |= 1u << (4 * q + i);
                    const _Float16 a = half_of(z < 0.0f ? 0.0f : z);
                    h[i >> 1][i & 1] = a;
                    s1[(8 * q + 4 * half + i) * L1 + n1] = a;
                }
                store_frag(p.H1f, wave * steps + 2 * blk, lane, q,
                           make_uint2(__builtin_bit_cast(uint32_t, h[0]), __builtin_bit_cast(uint32_t, h[1])));
            }
        }
        __syncthreads();

        // Layer 2.
        f32x16_t z2;
        if (on2) {
            if (!on1) load_group(g, w2, 0, ks1);
            z2 = layer(s1 + col * L1 + 8 * half, w2, ks1, g);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                z2[v] += bias2;
                s2[(8 * (v >> 2) + 4 * half + (v & 3)) * L2 + n2] = half_of(z2[v] < 0.0f ? 0.0f : z2[v]);
            }
        }
        if (on1) load_group(g, wt, 0, ks2);
        __syncthreads();

        // Head: 16 lanes per row; o = W3 h2 + b3, loss, gradient of the batch sum.
        {
            const int row = t >> 4;
            const int64_t b = b0 + row;
            float o0 = 0.0f, o1 = 0.0f;
            for (int c = 8 * (t & 15); c < p.h2; c += 128) {
                const f16x8_t h = *reinterpret_cast<const f16x8_t*>(s2 + row * L2 + c);
                const f16x8_t v0 = *reinterpret_cast<const f16x8_t*>(p.W3 + c);
                const f16x8_t v1 = *reinterpret_cast<const f16x8_t*>(p.W3 + p.h2 + c);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    o0 = __builtin_fmaf((float)h[e], (float)v0[e], o0);
                    o1 = __builtin_fmaf((float)h[e], (float)v1[e], o1);
                }
            }
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) {
                o0 += __shfl_xor(o0, off, 64);
                o1 += __shfl_xor(o1, off, 64);
            }
            o0 += p.b3[0];
            o1 += p.b3[1];
            float g0 = 0.0f, g1 = 0.0f;
            if (b < p.nvalid) {
                const float d = p.det_label[b];
                const float err = o0 - p.phi_label[b] / p.phi_scale;
                const float e = expf(-fabsf(o1));
                const float sig = o1 >= 0.0f ? 1.0f / (1.0f + e) : e / (1.0f + e);
                g0 = 2.0f * d * err;
                g1 = sig - d;
                loss += fmaxf(o1, 0.0f) + log1pf(e) - d * o1 + d * err * err;
                gb30 += g0;
                gb31 += g1;
            }
            if ((t & 15) == 0) {
                sg[2 * row] = g0;
                sg[2 * row + 1] = g1;
            }
        }
        __syncthreads();

        // dz2 = (g W3) where z2 > 0, and the sums over rows that need z2; rows
        // past the batch have no gradient.
        if (on2) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f16x2_t h[2];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 8 * q + 4 * half + i;
                    const float g0 = sg[2 * row], g1 = sg[2 * row + 1];
                    const float z = z2[4 * q + i];
                    const float hv = b0 + row < p.nvalid ? (float)half_of(z < 0.0f ? 0.0f : z) : 0.0f;
                    gw0 = __builtin_fmaf(g0, hv, gw0);
                    gw1 = __builtin_fmaf(g1, hv, gw1);
                    float d = __builtin_fmaf(g0, w30, g1 * w31);
                    if (!(z > 0.0f)) d = 0.0f;
                    gb2 += d;
                    const _Float16 a = half_of(d);
                    h[i >> 1][i & 1] = a;
                    s2[row * L2 + n2] = a;
                }
                store_frag(p.D2f, wave * steps + 2 * blk, lane, q,
                           make_uint2(__builtin_bit_cast(uint32_t, h[0]), __builtin_bit_cast(uint32_t, h[1])));
            }
        }
        __syncthreads();

        // dz1 = (dz2 W2) where z1 > 0.
        if (on1) {
            const f32x16_t d1 = layer(s2 + col * L2 + 8 * half, wt, ks2, g);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f16x2_t h[2];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float d = (m1 >> (4 * q + i)) & 1 ? d1[4 * q + i] : 0.0f;
                    gb1 += d;
                    h[i >> 1][i & 1] = half_of(d);
                }
                store_frag(p.D1f, wave * steps + 2 * blk, lane, q,
                           make_uint2(__builtin_bit_cast(uint32_t, h[0]), __builtin_bit_cast(uint32_t, h[1])));
            }
        }
        __syncthreads();
    }

    // Column sums of this workgroup: the two halves of a wave hold the same
    // column's other rows.
    float* const out = p.part + (int64_t)blockIdx.x * (p.h1 + 3 * p.h2 + 3);
    gb1 += __shfl_xor(gb1, 32, 64);
    gb2 += __shfl_xor(gb2, 32, 64);
    gw0 += __shfl_xor(gw0, 32, 64);
    gw1 += __shfl_xor(gw1, 32, 64);
    if (half == 0) {
        if (on1) out[n1] = gb1;
        if (on2) {
            out[p.h1 + n2] = gb2;
            out[p.h1 + p.h2 + n2] = gw0;
            out[p.h1 + 2 * p.h2 + n2] = gw1;
        }
    }
    if ((t & 15) == 0) {
        sl[3 * (t >> 4)] = gb30;
        sl[3 * (t >> 4) + 1] = gb31;
        sl[3 * (t >> 4) + 2] = loss;
    }
    __syncthreads();
    if (t < 3) {
        float s = sl[t];
        for (int i = 1; i < RB; ++i) s += sl[3 * i + t];
        out[p.h1 + 3 * p.h2 + t] = s;
    }
}

struct WgradArgs {
    const uint4 *D1f, *Xf, *D2f, *H1f;
    int64_t steps;  // 16-row steps of the batch
    int nin_pad, h1, h2;
    float scale, batch;      // 1 / batch, batch
    float *gW1, *gW2;        // [h1][ld1] (ld1 columns stored), [h2][h1]
    int64_t ld1;
    float *gb1, *gb2, *gW3, *gb3, *loss;  // loss may be NULL
    const float* part;       // column sums of nwg workgroups
    int nwg;
    float* plane;            // split batches: raw sums, [split][h1 nin_pad + h2 h1]
};

__global__ __launch_bounds__(64 * TW, 1) void train_wgrad_kernel(WgradArgs p)
{
    extern __shared__ float4 smem4[];
    float* const red = reinterpret_cast<float*>(smem4);  // [TW][WT * WT]
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int tn1 = p.nin_pad / WT, tiles1 = p.h1 / WT * tn1;
    const int tn2 = p.h1 / WT, tiles = tiles1 + p.h2 / WT * tn2;
    int tile = blockIdx.x;
    if (tile >= tiles) {
        // Column sums: 64 columns, the workgroups' rows shared by the waves.
        if (blockIdx.y) return;
        const int nc = p.h1 + 3 * p.h2 + 3, c = 64 * (tile - tiles) + lane;
        float s = 0.0f;
        if (c < nc)
            for (int y = wave; y < p.nwg; y += TW) s += p.part[(int64_t)y * nc + c];
        red[wave * 64 + lane] = s;
        __syncthreads();
        if (wave == 0 && c < nc) {
            for (int i = 1; i < TW; ++i) s += red[i * 64 + lane];
            if (c < p.h1) p.gb1[c] = s * p.scale;
            else if (c < p.h1 + p.h2) p.gb2[c - p.h1] = s * p.scale;
            else if (c < p.h1 + 3 * p.h2) p.gW3[c - p.h1 - p.h2] = s * p.scale;
            else if (c < nc - 1) p.gb3[c - p.h1 - 3 * p.h2] = s * p.scale;
            else if (p.loss) *p.loss = s / p.batch;
        }
        return;
    }
    const bool first = tile < tiles1;
    if (!first) tile -= tiles1;
    const int tn = first ? tn1 : tn2;
    const int tm = tile / tn;
    tile -= tm * tn;
    const uint4* const A = (first ? p.D1f : p.D2f) + (int64_t)(2 * tm) * p.steps * 64 + lane;
    const uint4* const B = (first ? p.Xf : p.H1f) + (int64_t)(2 * tile) * p.steps * 64 + lane;
    const int64_t sb = blockIdx.y * p.steps / gridDim.y, se = (blockIdx.y + 1) * p.steps / gridDim.y;

    f32x16_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    auto add = [&](int64_t s) __attribute__((always_inline)) {
        uint4 a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = A[(i * p.steps + s) * 64];
            b[i] = B[(i * p.steps + s) * 64];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma(a[i], b[j], acc[i][j]);
    };
    int64_t s = sb + wave;
    for (; s + 3 * TW < se; s += 4 * TW) {
        add(s);
        add(s + TW);
        add(s + 2 * TW);
        add(s + 3 * TW);
    }
    for (; s < se; s += TW) add(s);

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                red[wave * WT * WT + (32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * WT + 32 * j + (lane & 31)] =
                    acc[i][j][v];
    __syncthreads();
    for (int e = t; e < WT * WT; e += 64 * TW) {
        float sum = red[e];
#pragma unroll
        for (int i = 1; i < TW; ++i) sum += red[i * WT * WT + e];
        const int64_t m = WT * tm + e / WT, n = WT * tile + e % WT;
        if (p.plane) {
            const int64_t nW1 = (int64_t)p.h1 * p.nin_pad;
            float* const o = p.plane + blockIdx.y * (nW1 + (int64_t)p.h2 * p.h1);
            if (first) o[m * p.nin_pad + n] = sum;
            else o[nW1 + m * p.h1 + n] = sum;
        } else if (first) {
            if (n < p.ld1) p.gW1[m * p.ld1 + n] = sum * p.scale;
        } else {
            p.gW2[m * p.h1 + n] = sum * p.scale;
        }
    }
}

// Split batches: the planes added in order.
__global__ __launch_bounds__(256) void wgrad_planes_kernel(WgradArgs p, int nsplit)
{
    const int64_t nW1 = (int64_t)p.h1 * p.nin_pad, n = nW1 + (int64_t)p.h2 * p.h1;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float s = p.plane[i];
    for (int y = 1; y < nsplit; ++y) s += p.plane[y * n + i];
    s *= p.scale;
    if (i < nW1) {
        const int64_t m = i / p.nin_pad, k = i - m * p.nin_pad;
        if (k < p.ld1) p.gW1[m * p.ld1 + k] = s;
    } else {
        p.gW2[i - nW1] = s;
    }
}

// Half copies of one parameter: row-major w16 (W1 | W2 | W3) and, with frag, the
// fragments of W1, W2 and W2 transposed (rows n, contracted k: fragment
// (n / 32, k / 16), lane (n & 31) + 32 (k / 8 & 1), element k & 7).
__device__ __forceinline__ void put_half(const ParamLayout& L, int64_t i, float v, _Float16* w16, _Float16* frag)
{
    auto at = [](int64_t n, int64_t k, int64_t K) {
        return ((((n >> 5) * (K >> 4) + (k >> 4)) * 64) + (n & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
    };
    const _Float16 h = (_Float16)v;
    const int64_t o2 = L.nW1 + L.h1, o3 = o2 + L.nW2 + L.h2;
    if (i < L.nW1) {
        w16[i] = h;
        if (frag) frag[at(i / L.nin_pad, i % L.nin_pad, L.nin_pad)] = h;
    } else if (i >= o2 && i < o2 + L.nW2) {
        const int64_t e = i - o2, o = e / L.h1, k = e % L.h1;
        w16[L.nW1 + e] = h;
        if (frag) {
            frag[L.nW1 + at(o, k, L.h1)] = h;
            frag[L.nW1 + L.nW2 + at(k, o, L.h2)] = h;
        }
    } else if (i >= o3 && i < o3 + L.nW3) {
        w16[L.nW1 + L.nW2 + (i - o3)] = h;
    }
}

__global__ __launch_bounds__(256) void halves_kernel(ParamLayout L, const float* __restrict__ p,
                                                     _Float16* __restrict__ w16, _Float16* __restrict__ frag)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < L.np()) put_half(L, i, p[i], w16, frag);
}

// Adam (Kingma & Ba, bias-corrected) on the FP32 master parameters, and the
// half copies of the result.
__global__ __launch_bounds__(256) void adam_kernel(ParamLayout L, float* __restrict__ p,
                                                   const float* __restrict__ g, float* __restrict__ m,
                                                   float* __restrict__ v, float lr, float beta1, float beta2,
                                                   float eps, float bc1, float bc2,
                                                   _Float16* __restrict__ w16, _Float16* __restrict__ frag)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= L.np()) return;
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    p[i] = pi;
    put_half(L, i, pi, w16, frag);
}

size_t rows_lds(int nin_pad, int h1, int h2)
{
    return sizeof(_Float16) * RB * (size_t)(nin_pad + 8 + h1 + 8 + h2 + 8) + sizeof(float) * (2 * RB + 3 * RB);
}

unsigned blocks_of(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

bool mlp_rows_supported(int h1, int h2, int nin_pad)
{
    return h1 <= 32 * TW && h2 <= 32 * TW && rows_lds(nin_pad, h1, h2) <= 160 * 1024;
}

int64_t mlp_rows_part_floats(int h1, int h2) { return (int64_t)kMaxWg * (h1 + 3 * h2 + 3); }

hipError_t mlp_launch_rows(const MlpTrainArgs& a, hipStream_t s)
{
    const ParamLayout& L = a.L;
    RowsArgs r{};
    r.Q = a.Q;
    r.U = a.U;
    r.nvalid = a.batch;
    r.nblk = (a.batch + RB - 1) / RB;
    r.nchan = a.nchan;
    r.nin_pad = L.nin_pad;
    r.h1 = L.h1;
    r.h2 = L.h2;
    r.w = a.chan_w;
    r.W1f = a.frag;
    const FragLayout f = frag_layout(L.nin_pad, L.h1, L.h2);
    r.W2f = a.frag + f.w2;
    r.W2t = a.frag + f.w2t;
    r.b1 = a.p + L.nW1;
    r.b2 = r.b1 + L.h1 + L.nW2;
    r.b3 = r.b2 + L.h2 + L.nW3;
    r.W3 = a.W3;
    r.phi_scale = a.phi_scale;
    r.phi_label = a.phi_label;
    r.det_label = a.det_label;
    r.Xf = reinterpret_cast<uint4*>(a.X);
    r.H1f = reinterpret_cast<uint4*>(a.H1);
    r.D1f = reinterpret_cast<uint4*>(a.D1);
    r.D2f = reinterpret_cast<uint4*>(a.D2);
    r.part = a.part;
    const int nwg = (int)std::min<int64_t>(r.nblk, kMaxWg);
    hipLaunchKernelGGL(train_rows_kernel, dim3(nwg), dim3(64 * TW), rows_lds(L.nin_pad, L.h1, L.h2), s, r);
    if (hipError_t e = hipGetLastError()) return e;

    WgradArgs w{};
    w.D1f = r.D1f;
    w.Xf = r.Xf;
    w.D2f = r.D2f;
    w.H1f = r.H1f;
    w.steps = 2 * r.nblk;
    w.nin_pad = L.nin_pad;
    w.h1 = L.h1;
    w.h2 = L.h2;
    w.batch = (float)a.batch;
    w.scale = 1.0f / w.batch;
    w.gW1 = a.grad;
    w.ld1 = a.ld1;
    w.gb1 = a.grad + (int64_t)L.h1 * a.ld1;
    w.gW2 = w.gb1 + L.h1;
    w.gb2 = w.gW2 + L.nW2;
    w.gW3 = w.gb2 + L.h2;
    w.gb3 = w.gW3 + L.nW3;
    w.loss = a.loss;
    w.part = a.part;
    w.nwg = nwg;
    const int tiles = L.h1 / WT * (L.nin_pad / WT) + L.h2 / WT * (L.h1 / WT);
    const int sums = (L.h1 + 3 * L.h2 + 3 + 63) / 64;
    // Shares of 2048 rows (16 steps per wave) while the tiles alone leave CUs idle.
    const int64_t want = std::min<int64_t>({a.batch / 2048, (512 + tiles - 1) / tiles, a.plane_floats / (L.nW1 + L.nW2)});
    const unsigned nsplit = want > 1 ? (unsigned)want : 1u;
    w.plane = nsplit > 1 ? a.plane : nullptr;
    hipLaunchKernelGGL(train_wgrad_kernel, dim3((unsigned)(tiles + sums), nsplit), dim3(64 * TW),
                       sizeof(float) * TW * WT * WT, s, w);
    if (hipError_t e = hipGetLastError()) return e;
    if (nsplit > 1)
        hipLaunchKernelGGL(wgrad_planes_kernel, dim3(blocks_of(L.nW1 + L.nW2)), dim3(256), 0, s, w, (int)nsplit);
    return hipGetLastError();
}

hipError_t mlp_launch_halves(const ParamLayout& L, const float* p, _Float16* w16, uint4* frag, hipStream_t s)
{
    hipLaunchKernelGGL(halves_kernel, dim3(blocks_of(L.np())), dim3(256), 0, s, L, p, w16,
                       reinterpret_cast<_Float16*>(frag));
    return hipGetLastError();
}

hipError_t mlp_launch_adam(const ParamLayout& L, float* p, const float* g, float* m, float* v, float lr,
                           float beta1, float beta2, float eps, float bc1, float bc2, _Float16* w16,
                           uint4* frag, hipStream_t s)
{
    hipLaunchKernelGGL(adam_kernel, dim3(blocks_of(L.np())), dim3(256), 0, s, L, p, g, m, v, lr, beta1, beta2,
                       eps, bc1, bc2, w16, reinterpret_cast<_Float16*>(frag));
    return hipGetLastError();
}
