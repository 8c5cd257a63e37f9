// Faraday-depth transform on a uniform phi grid, by mirrored pairs of depths.
//
// For a tile of 2 NH depths centred on phi_c (half way between its two middle
// depths), phi = phi_c +- h with h = (i + 1/2) dphi, i = 0 .. NH - 1.  With the
// data rotated to the centre, x_j + i y_j = K w_j X_lj exp(-2i a_j phi_c)
// (eqs. (11), (13)), and c = cos(2 a_j h), s = sin(2 a_j h),
//   F(phi_c + h) = (S_xc + S_ys) + i (S_yc - S_xs),
//   F(phi_c - h) = (S_xc - S_ys) + i (S_yc + S_xs),
// where S_xc = sum_j x_j c etc.: four real sums give two complex outputs, half
// the multiply-adds of the direct real form (which needs four for each).
// The rotation is applied while a Q/U tile is packed into LDS; c and s do not
// depend on the tile and are a plan-time table (FP64 argument reduction) that
// stays in every XCD's L2.  The nchan x nphi phase matrix is never formed.
//
// The folded form (FOLD) is the same idea on the other axis: plans whose
// contracted axis is uniform, b_c = b_0 + c db, and whose output grid g is not
// (the adjoint transform on a uniform phi grid, the phi_k being contracted).
// In K-tiles of L contracted channels centred on b_J (half way between two),
// the channels at b_J +- h, h = (i + 1/2) db, enter as S = X+ + X- and
// D = X+ - X-:
//   F_g = K sum_J exp(-2 pi i b_J g) sum_i (S_i cos - i D_i sin)(2 pi h_i g),
// half the multiply-adds again.  The cos/sin table does not depend on J; the
// K-tiles run from the top down and the accumulators are multiplied by
// exp(-2 pi i L db g) before each (Horner's rule), K exp(-2 pi i b_0' g) of the
// lowest tile's centre b_0' in the epilogue.
//
// The table form (TAB) serves grids where neither axis is uniform: the plan
// holds cos and sin of the whole phase matrix (capped in size), the data are
// only weighted, and F = sum_j (x + iy)(c - is) takes the full four products.
//
// The sums run on the matrix cores with FP32 accumulation, in one of
//   FP32   v_mfma_f32_32x32x2_f32 on FP32 operands,
//   split  v_mfma_f32_32x32x16_{bf16,f16} on x = hi + lo in 16 bits each,
//          hi*hi + hi*lo + lo*hi (lo*lo dropped).
//
// Workgroup: 256 threads, 64 LOS x 256 phi, 16 channels per K-step.  Wave w
// owns all 64 LOS and the pairs i = 32 w .. 32 w + 31 (64 phi): 2 LOS groups x
// 4 sums (128 accumulators per lane), so two workgroups share a CU (tiles of 128
// columns: two such tiles of two waves).  A wave's
// table columns are its own, so they go from L2 straight to registers, one
// K-step ahead, in MFMA operand order (1 KB contiguous per load); LDS carries
// only the packed data (8 KB per K-step, triple buffered).  Per K-step and
// wave the split forms issue 24 MFMAs, 8 LDS reads of 16 bytes and the packing
// of 4 channels of 64 LOS.
//
// What bounds it: the matrix cores, at the clock the power limit leaves them.
// 65536 LOS x 2001 phi, bf16x3, no F stored: 0.54 ms with 400 channels, 1.06
// with 800, 2.03 with 1600, so the K-loop alone issues 1290 TFLOP/s, 12 flop for
// each of 2048 padded depths (a library bf16 GEMM of 16384^3 reaches 1375 on the
// same card), and a tile's start and end cost 8 % at 400 channels.  Storing F
// adds 1.5 of 10.9 ms at 1024^2 LOS.
// Packing two K-steps between barriers (six LDS buffers) was 1-2 % slower;
// centring a ragged last tile on what is left of the grid, so that waves with
// no pairs skip the matrix work, gained nothing (the workgroup still waits for
// its full waves).
// Folded, 262144 LOS x 2001 phi -> 400 channels (padded to 512), bf16x3: 3.07 ms
// (6.02 with 96-phi K-tiles and no folding; 3.22 with rows read 32 bytes at a
// time, a K-step's share, which fetched each line of a row four times into L1); table form, 131072 x 400 x 2001:
// 2.16 ms (2.32 with 128 x 128 tiles fed through LDS), 65536 in FP32 3.13 ms
// (3.81 with the phases generated per element).
#include <float.h>

#include <type_traits>

#include "common.h"

namespace {

constexpr int KC = kMirrorChan;      // channels per K-step
constexpr int64_t kSmallWaves = 512;  // see launch_mg

enum { LOAD_ROW4 = 0, LOAD_TAIL = 1, LOAD_ONE = 2, FOLD = 3, TAB_ROW = 4, TAB_PLANE = 5 };

// Tiles of NW waves per workgroup.  Of workgroups of two waves the first two on a
// CU share two of its SIMDs, so that calls which do not fill the chip take twice
// the time (table form, 32768 LOS x 256 ch x 100 phi, FP32: 124 us, in
// pairs 73).
// The folded form is 3-5 % faster with tiles on their own where it takes them.
constexpr int tiles_per_wg(int load, int nw) { return load == FOLD ? 1 : 4 / nw; }

typedef const __attribute__((address_space(4))) f32x4_t* const_f4_ptr;
typedef float f32x2u_t __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));

template <int PREC>
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& lo)
{
    if (PREC == RMSYNTH_SPLIT_FP16) split2_f16(a, b, hi, lo);
    else split2_bf16(a, b, hi, lo);
}

template <int PREC>
__device__ __forceinline__ f32x16_t mfma16(uint4 a, uint4 b, f32x16_t c)
{
    if (PREC == RMSYNTH_SPLIT_FP16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a),
                                                      __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                       __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// LOAD: how Q/U are read.  ROW4: LOS-major rows, 4 n channels, as quads of any
// alignment; TAIL: the same for the other channel counts above 4; ONE: single
// values, frequency-major (ls = 1) and LOS-major below 4 channels (ls = ld, and
// ld 1).  nh: pairs of depths per tile, at most 32 NW; waves past it only pack.
// FOLD: the folded form (LOS-major, any alignment; no flags, no peaks): T is its
// table, nk the K-steps of all K-tiles, ksteps those of one, pad the zero
// channels below channel 0, kbase and krot the K exp(-2 pi i b_0' g) and
// exp(-2 pi i L db g) per output as (cos, sin).
// TAB_ROW, TAB_PLANE: the table form, LOS-major (any alignment) and
// frequency-major: K-steps of 8 channels, base holds (K w_j, 0).
// FLAGS: some channel has weight 0; its (zero) rotation then also clears
// whatever the data hold there, NaN included.
// MG: LOS groups (of 32) per tile; NW: waves of 64 columns per tile (4 or 2).
// The results depend on neither.  tiles_per_wg: 128-column tiles of the table
// form go in pairs, one below the other.
// PEAKS 1: the epilogue also reduces |F|^2 of every LOS over each 64 phi and
// writes one PeakPart per (LOS, 64 phi) for peak_merge_kernel, at
// part[(64-phi block) * part_ld + LOS].  PEAKS 2: F is not stored; one PeakRec
// each instead, for peak_merge_rec_kernel.
template <int LOAD, int PREC, bool FLAGS, int PEAKS, int MG, int NW>
__global__ __launch_bounds__(64 * NW * tiles_per_wg(LOAD, NW), 2) void synth_mirrored_kernel(
    const float* __restrict__ Q, const float* __restrict__ U, int64_t nlos, int64_t ld, int nchan,
    const float2* __restrict__ base, const uint4* __restrict__ T, int nchan_pad, int nk, int nphi,
    int tiles_n, float* __restrict__ Fq, float* __restrict__ Fu, float* __restrict__ Fabs,
    const float* __restrict__ los_scale, PeakPart* __restrict__ part, int64_t part_ld,
    PeakRec* __restrict__ rec, int ldT, int ksteps, int pad, const float2* __restrict__ kbase,
    const float2* __restrict__ krot, int ls, int nh)
{
    static_assert(LOAD != FOLD || (PEAKS == 0 && !FLAGS), "the folded form has no peaks and no flags");
    constexpr bool F32 = PREC == RMSYNTH_FP32;
    constexpr bool TAB = LOAD == TAB_ROW || LOAD == TAB_PLANE;
    // Columns of T are outputs (else mirrored pairs of them); K-steps then
    // contract 8 pairs or channels, as (cos, sin) neighbours.
    constexpr bool COLS = LOAD == FOLD || TAB;
    constexpr bool OCT = LOAD == FOLD || LOAD == TAB_ROW;  // eight lanes share a row
    constexpr bool ONE = LOAD == LOAD_ONE;
    static_assert(NW == 4 || NW == 2, "tiles of four or two waves");
    constexpr int TILE = 64 * NW;    // phi (output columns) per tile
    constexpr int SR = TILE + 4;     // row stride (floats) of the epilogue's tile: conflict-free b128 rows
    constexpr int MT = 32 * MG;      // LOS per tile
    constexpr int RT = 8 * NW, IT = OCT ? MT / RT : 2;  // OCT: rows per pass, passes
    constexpr int PQ = 4 / NW;       // else: quads (TAB_PLANE: pairs) of channels per wave
    constexpr int STEP = 4 * MT * 2;  // uint4 of a packed K-step: [2 channel octets or quad pairs][4][MT]
    union Lds {
        uint4 a[3][STEP];
        float f[MT * SR];
    };
    constexpr int SUB = tiles_per_wg(LOAD, NW);
    __shared__ Lds lds_sub[SUB];
    // Workgroups are dispatched round-robin over the 8 XCDs, each with its own
    // L2: groups of 8 LOS tiles, one per XCD, whose phi tiles then follow one
    // another on it (they read the same Q/U rows).  The whole chip so works on
    // one stretch of the cube (1 % faster than an eighth of the cube per XCD).
    const uint32_t grp = blockIdx.x / (8u * tiles_n), in_grp = blockIdx.x - grp * (8u * tiles_n);
    const uint32_t mleft = gridDim.x / tiles_n - 8u * grp, wide = mleft < 8u ? mleft : 8u;
    const int tn = (int)(in_grp / wide);
    const int n0 = tn * TILE;
    const int t = threadIdx.x & (64 * NW - 1), lane = t & 63;
    const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = SUB == 1 ? wg_wave : wg_wave % NW, sub = SUB == 1 ? 0 : wg_wave / NW;  // wave of its tile, tile
    Lds& lds = lds_sub[sub];
    const int64_t l_tile = ((int64_t)(8u * grp + in_grp % wide) * SUB + sub) * MT;
    // A tile that starts past the cube reads its last LOS and stores nothing.
    const int64_t l0 = SUB == 1 || l_tile < nlos ? l_tile : nlos - 1;
    const int nl = SUB == 1 || l_tile < nlos ? (int)(nlos - l0 < MT ? nlos - l0 : MT) : 0;  // LOS of the tile
    const int half = lane >> 5, col = lane & 31;

    // Pack role: LOS `row` of the tile, channel quads PQ wave .. of the K-step
    // (so that the channel rotations are scalar loads; with 32 LOS both halves of
    // the wave pack the same values).  Rows past the cube read
    // its last LOS; their outputs are never stored.  Channels past the end
    // read the last ones; their rotation is zero, and a non-finite value they
    // pick up there belongs to the same LOS, which it spoils anyway (or, in a
    // flagged channel, is cleared by FLAGS).
    const int row = lane & (MT - 1);
    const int64_t left = nlos - 1 - l0;
    const int lr = row < left ? row : (int)left;
    const float lsc = PREC == RMSYNTH_SPLIT_FP16 ? los_scale[l0 + lr] : 1.0f;
    const int64_t lstride = LOAD == TAB_PLANE ? 1 : ONE ? ls : ld;
    const uint32_t voff = 4u * (uint32_t)(lr * (int)lstride);  // < 2^28: 63 rows of at most 2^20 values
    const float* const Qt = Q + l0 * lstride;
    const float* const Ut = U + l0 * lstride;
    const_f4_ptr bt = (const_f4_ptr)(TAB ? base : base + (int64_t)tn * nchan_pad);
    // OCT: eight lanes share a LOS row, lane cc the pair or channel cc of the
    // K-step, rows rq + RT i: a wave's load covers 8 rows x 32 contiguous bytes.
    const int cc = t & 7, rq = t >> 3;
    uint32_t frow[IT];
    float fsc[IT];
    if constexpr (OCT) {
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int r = rq + RT * i < left ? rq + RT * i : (int)left;
            frow[i] = 4u * (uint32_t)(r * (int)ld);  // < 2^28, as voff
            fsc[i] = PREC == RMSYNTH_SPLIT_FP16 ? los_scale[l0 + r] : 1.0f;
        }
    }
    // Table columns of this wave: [K-step][64-output block][4][64 lanes].
    const uint4* const Tw = T + (COLS ? NW * tn + wave : wave) * 256 + lane;
    const int tstep = COLS ? ldT : 1024;

    struct Data {
        float q[4 * IT], u[4 * IT];  // FOLD: two K-steps; else the first 2 IT
        float w;  // TAB_ROW
    };
    struct Frag {
        uint4 v[4];
    };
    f32x4_t rot[2 * PQ];  // (cos, sin) K w_j of the quads to be packed next

    // FOLD: K-tile and K-step within it of the current step, and of the K-step d
    // further on (at most one K-tile away, or clamped to the last; d is passed
    // where the other forms pass a K-step's number).
    int cj = 0, ck = 0;
    auto ahead = [&](int d, int& j, int& kk) __attribute__((always_inline)) {
        j = cj;
        kk = ck + d;
        if (kk >= ksteps) {
            kk -= ksteps;
            --j;
        }
        if (j < 0) {
            j = 0;
            kk = ksteps - 1;
        }
    };
    // Pair cc of K-step kk: the K-steps 2 n and 2 n + 1 share 16 pairs, two
    // neighbouring ones per lane, so that a row is read 64 bytes at a time.
    auto pair_channels = [&](int d, int& jp, int& jm) __attribute__((always_inline)) {
        int J, kk;
        ahead(d, J, kk);
        const int mid = J * ksteps * KC - pad + ksteps * (KC / 2);
        const int i = KC * (kk >> 1) + 2 * cc + (kk & 1);
        jp = mid + i;
        jm = mid - 1 - i;
    };
    auto load_data = [&](Data& R, int k) __attribute__((always_inline)) {
        if constexpr (LOAD == FOLD) {
            // q, u [4 i ..]: rows i; the upper channels of this K-step (an even
            // one) and the next, then the lower ones of the next and this.
            // Channels past either end are cleared when packed.
            int jp, jm;
            pair_channels(k, jp, jm);
            auto offset = [&](int j) { return 4u * (uint32_t)(j < 0 ? 0 : j < nchan - 1 ? j : nchan - 2); };
            const uint32_t op = offset(jp), om = offset(jm - 1);
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                auto at = [&](const float* b, uint32_t o, float* to) {
                    const f32x2u_t v = *reinterpret_cast<const f32x2u_t*>(reinterpret_cast<const char*>(b) + (frow[i] + o));
                    to[0] = v.x;
                    to[1] = v.y;
                };
                at(Qt, op, R.q + 4 * i);
                at(Ut, op, R.u + 4 * i);
                at(Qt, om, R.q + 4 * i + 2);
                at(Ut, om, R.u + 4 * i + 2);
            }
            return;
        }
        if constexpr (LOAD == TAB_ROW) {
            // q, u [i]: rows i; w: the channel's weight (0 past the end).
            const int jw = 8 * k + cc, j = jw < nchan ? jw : nchan - 1;
            R.w = base[jw].x;
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                R.q[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Qt) + (frow[i] + 4u * (uint32_t)j));
                R.u[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Ut) + (frow[i] + 4u * (uint32_t)j));
            }
            return;
        }
        if constexpr (LOAD == TAB_PLANE) {
#pragma unroll
            for (int i = 0; i < 2 * PQ; ++i) {
                const int jw = 8 * k + 2 * PQ * wave + i, j = jw < nchan ? jw : nchan - 1;
                R.q[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Qt + (int64_t)j * ld) + voff);
                R.u[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Ut + (int64_t)j * ld) + voff);
            }
            return;
        }
#pragma unroll
        for (int p = 0; p < PQ; ++p) {
            const int j0 = k * KC + 4 * (PQ * wave + p);
            float* const q = R.q + 4 * p;
            float* const u = R.u + 4 * p;
            if (LOAD == LOAD_ROW4 || LOAD == LOAD_TAIL) {
                const int j = j0 < nchan - 4 ? j0 : nchan - 4;
                const f32x4u_t a = *reinterpret_cast<const f32x4u_t*>(reinterpret_cast<const char*>(Qt + j) + voff);
                const f32x4u_t b = *reinterpret_cast<const f32x4u_t*>(reinterpret_cast<const char*>(Ut + j) + voff);
                q[0] = a.x; q[1] = a.y; q[2] = a.z; q[3] = a.w;
                u[0] = b.x; u[1] = b.y; u[2] = b.z; u[3] = b.w;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = j0 + i < nchan ? j0 + i : nchan - 1;
                    const int64_t at = (int64_t)j * ld;
                    q[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Qt + at) + voff);
                    u[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Ut + at) + voff);
                }
            }
        }
    };
    // TAIL: the last quad of a row was read from its last 4 channels; its own
    // go to the front (what follows them meets a zero rotation).
    auto align_tail = [&](Data& R, int k) __attribute__((always_inline)) {
        if constexpr (LOAD == LOAD_TAIL) {
#pragma unroll
            for (int p = 0; p < PQ; ++p) {
                const int past = k * KC + 4 * (PQ * wave + p) + 4 - nchan;
                if (past <= 0) continue;
                auto shift = [&](float* v) __attribute__((always_inline)) {
                    const float v1 = v[1], v2 = v[2], v3 = v[3];
                    v[0] = past == 1 ? v1 : past == 2 ? v2 : v3;
                    v[1] = past == 1 ? v2 : v3;
                    v[2] = v3;
                };
                shift(R.q + 4 * p);
                shift(R.u + 4 * p);
            }
        }
    };
    auto load_rot = [&](int k) __attribute__((always_inline)) {
        if (OCT) return;
        if (LOAD == TAB_PLANE) {
#pragma unroll
            for (int p = 0; p < PQ; ++p) rot[p] = bt[4 * k + PQ * wave + p];
            return;
        }
        const int at = (k * KC + 4 * PQ * wave) >> 1;
#pragma unroll
        for (int i = 0; i < 2 * PQ; ++i) rot[i] = bt[at + i];
    };
    auto load_b = [&](Frag& B, int k) __attribute__((always_inline)) {
        if constexpr (LOAD == FOLD) {
            int j;
            ahead(k, j, k);
        }
        const uint4* p = Tw + (int64_t)k * tstep;
#pragma unroll
        for (int i = 0; i < 4; ++i) B.v[i] = p[64 * i];
    };
    // Rotate and pack the quad: FP32 as float4 x, y of quad `wave`; split as
    // the 8-byte half of the channel octet's x hi, x lo, y hi, y lo.
    float px[OCT ? 2 * IT : 4 * PQ], py[OCT ? 2 * IT : 4 * PQ];
    auto rotate1 = [&](const Data& R, int i, int k, bool odd) __attribute__((always_inline)) {
        if constexpr (LOAD == FOLD) {
            // i < IT: S, D of row i as px = (Sx, Dy), py = (Sy, -Dx).  A pair of
            // channels read from the row's start instead of from -1 holds its
            // second one in its first place.
            if (i >= IT) return;
            const float sc = fsc[i];
            int jp, jm;
            pair_channels(k, jp, jm);
            const bool okp = (uint32_t)jp < (uint32_t)nchan, okm = (uint32_t)jm < (uint32_t)nchan;
            const bool start = (odd ? jp : jm) == 0;
            const float* const q = R.q + 4 * i;
            const float* const u = R.u + 4 * i;
            const float qp = odd ? start ? q[0] : q[1] : q[0], qm = odd ? q[2] : start ? q[2] : q[3];
            const float up = odd ? start ? u[0] : u[1] : u[0], um = odd ? u[2] : start ? u[2] : u[3];
            const float xp = okp ? qp * sc : 0.0f, xm = okm ? qm * sc : 0.0f;
            const float yp = okp ? up * sc : 0.0f, ym = okm ? um * sc : 0.0f;
            px[2 * i] = xp + xm;
            px[2 * i + 1] = yp - ym;
            py[2 * i] = yp + ym;
            py[2 * i + 1] = xm - xp;
            return;
        }
        if constexpr (TAB) {
            // TAB_ROW: row i < IT; TAB_PLANE: channel i of the wave's pairs.
            // px = (x, y), py = (y, -x).
            if (i >= (OCT ? IT : 2 * PQ)) return;
            const float w = LOAD == TAB_ROW ? R.w : (i & 1) ? rot[i >> 1].z : rot[i >> 1].x;
            float x = R.q[i] * w, y = R.u[i] * w;
            if (FLAGS) {
                x = w == 0.0f ? 0.0f : x;
                y = w == 0.0f ? 0.0f : y;
            }
            if (PREC == RMSYNTH_SPLIT_FP16) {
                x *= LOAD == TAB_ROW ? fsc[i] : lsc;
                y *= LOAD == TAB_ROW ? fsc[i] : lsc;
            }
            px[2 * i] = x;
            px[2 * i + 1] = y;
            py[2 * i] = y;
            py[2 * i + 1] = -x;
            return;
        }
        const f32x4_t rr = rot[i >> 1];
        const float rc = (i & 1) ? rr.z : rr.x;
        const float rs = (i & 1) ? rr.w : rr.y;
        float xr = __builtin_fmaf(R.q[i], rc, R.u[i] * rs);
        float yr = __builtin_fmaf(R.u[i], rc, -(R.q[i] * rs));
        if (FLAGS) {
            const bool flagged = ((__float_as_uint(rc) | __float_as_uint(rs)) << 1) == 0u;
            xr = flagged ? 0.0f : xr;
            yr = flagged ? 0.0f : yr;
        }
        if (PREC == RMSYNTH_SPLIT_FP16) {
            xr *= lsc;
            yr *= lsc;
        }
        px[i] = xr;
        py[i] = yr;
    };
    auto store_data = [&](int buf) __attribute__((always_inline)) {
        if constexpr (LOAD == TAB_PLANE) {
            // As below, two channels: 8 bytes each.
#pragma unroll
            for (int p = 0; p < PQ; ++p) {
                const int at = PQ * wave + p;
                const float* const x = px + 4 * p;
                const float* const y = py + 4 * p;
                uint2* const a = reinterpret_cast<uint2*>(&lds.a[buf][(at >> 1) * (4 * MT) + row]) + (at & 1);
                uint2 w[4];
                if (F32) {
                    w[0] = make_uint2(__float_as_uint(x[0]), __float_as_uint(x[2]));
                    w[1] = make_uint2(__float_as_uint(x[1]), __float_as_uint(x[3]));
                    w[2] = make_uint2(__float_as_uint(y[0]), __float_as_uint(y[2]));
                    w[3] = make_uint2(__float_as_uint(y[1]), __float_as_uint(y[3]));
                } else {
                    split2<PREC>(x[0], x[1], w[0].x, w[1].x);
                    split2<PREC>(x[2], x[3], w[0].y, w[1].y);
                    split2<PREC>(y[0], y[1], w[2].x, w[3].x);
                    split2<PREC>(y[2], y[3], w[2].y, w[3].y);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) a[2 * MT * e] = w[e];
            }
            return;
        }
        if constexpr (OCT) {
            // rows Re: (Sx, Dy), Im: (Sy, -Dx) (TAB: S = D = X) against columns (cos, sin).  Split:
            // [pair quad][Re hi, Re lo, Im hi, Im lo][row], one dword per pair;
            // FP32: [pair quad][Re, Im][cos part, sin part][row], one float each.
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                uint32_t* const a = reinterpret_cast<uint32_t*>(&lds.a[buf][(cc >> 2) * (4 * MT) + rq + RT * i]) + (cc & 3);
                uint32_t w[4];
                if (F32) {
                    w[0] = __float_as_uint(px[2 * i]);
                    w[1] = __float_as_uint(px[2 * i + 1]);
                    w[2] = __float_as_uint(py[2 * i]);
                    w[3] = __float_as_uint(py[2 * i + 1]);
                } else {
                    split2<PREC>(px[2 * i], px[2 * i + 1], w[0], w[1]);
                    split2<PREC>(py[2 * i], py[2 * i + 1], w[2], w[3]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) a[4 * MT * e] = w[e];
            }
            return;
        }
#pragma unroll
        for (int p = 0; p < PQ; ++p) {
            const int at = PQ * wave + p;
            const float* const x = px + 4 * p;
            const float* const y = py + 4 * p;
            if (F32) {
                // [quad pair][x, y][quad of the pair][row]
                uint4* const a = &lds.a[buf][(at >> 1) * (4 * MT) + (at & 1) * MT + row];
                a[0] = __builtin_bit_cast(uint4, f32x4_t{x[0], x[1], x[2], x[3]});
                a[2 * MT] = __builtin_bit_cast(uint4, f32x4_t{y[0], y[1], y[2], y[3]});
            } else {
                uint2 xh, xl, yh, yl;
                split2<PREC>(x[0], x[1], xh.x, xl.x);
                split2<PREC>(x[2], x[3], xh.y, xl.y);
                split2<PREC>(y[0], y[1], yh.x, yl.x);
                split2<PREC>(y[2], y[3], yh.y, yl.y);
                // [octet][x hi, x lo, y hi, y lo][row], 8-byte halves
                uint2* const a = reinterpret_cast<uint2*>(&lds.a[buf][(at >> 1) * (4 * MT) + row]) + (at & 1);
                a[0] = xh;
                a[2 * MT] = xl;
                a[4 * MT] = yh;
                a[6 * MT] = yl;
            }
        }
    };
    auto load_a = [&](Frag& A, int buf, int g) __attribute__((always_inline)) {
        if (F32) {
            // v[2 p + xy]: quad pair p, this lane's quad of it
#pragma unroll
            for (int i = 0; i < 4; ++i)
                A.v[i] = lds.a[buf][(i >> 1) * (4 * MT) + (i & 1) * (2 * MT) + half * MT + 32 * g + col];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) A.v[i] = lds.a[buf][half * (4 * MT) + i * MT + 32 * g + col];
        }
    };

    // acc[g][s]: LOS group g (32 LOS), sums s = xc, ys, yc, xs (COLS: with Re, Im
    // for x, y and the wave's two blocks of 32 columns for c, s).
    f32x16_t acc[MG][4];
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[g][s][v] = 0.0f;

    // (re, im) <- (re + i im)(r.x - i r.y), few elements at a time: done all at
    // once the accumulators would need a second set of registers.
    auto turn = [](f32x16_t& re, f32x16_t& im, float2 r) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float a = re[v], b = im[v];
            re[v] = __builtin_fmaf(a, r.x, b * r.y);
            im[v] = __builtin_fmaf(b, r.x, -(a * r.y));
            if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    };

    auto mma = [&](const Frag& A, const Frag& B, int g, auto&& midway) __attribute__((always_inline)) {
        if constexpr (F32) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if (p == 1) midway();
                const f32x4_t x = __builtin_bit_cast(f32x4_t, A.v[2 * p]);
                const f32x4_t y = __builtin_bit_cast(f32x4_t, A.v[2 * p + 1]);
                const f32x4_t c = __builtin_bit_cast(f32x4_t, B.v[2 * p]);
                const f32x4_t s = __builtin_bit_cast(f32x4_t, B.v[2 * p + 1]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[g][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], c[i], acc[g][0], 0, 0, 0);
                    acc[g][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(y[i], s[i], acc[g][1], 0, 0, 0);
                    acc[g][2] = __builtin_amdgcn_mfma_f32_32x32x2f32(y[i], c[i], acc[g][2], 0, 0, 0);
                    acc[g][3] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], s[i], acc[g][3], 0, 0, 0);
                }
            }
        } else {
            // v: x hi, x lo, y hi, y lo and c hi, c lo, s hi, s lo
            const uint4 xh = A.v[0], xl = A.v[1], yh = A.v[2], yl = A.v[3];
            const uint4 ch = B.v[0], cl = B.v[1], sh = B.v[2], sl = B.v[3];
            acc[g][0] = mfma16<PREC>(xl, ch, acc[g][0]);
            acc[g][1] = mfma16<PREC>(yl, sh, acc[g][1]);
            acc[g][2] = mfma16<PREC>(yl, ch, acc[g][2]);
            acc[g][3] = mfma16<PREC>(xl, sh, acc[g][3]);
            acc[g][0] = mfma16<PREC>(xh, cl, acc[g][0]);
            acc[g][1] = mfma16<PREC>(yh, sl, acc[g][1]);
            midway();
            acc[g][2] = mfma16<PREC>(yh, cl, acc[g][2]);
            acc[g][3] = mfma16<PREC>(xh, sl, acc[g][3]);
            acc[g][0] = mfma16<PREC>(xh, ch, acc[g][0]);
            acc[g][1] = mfma16<PREC>(yh, sh, acc[g][1]);
            acc[g][2] = mfma16<PREC>(yh, ch, acc[g][2]);
            acc[g][3] = mfma16<PREC>(xh, sh, acc[g][3]);
        }
    };

    // LDS writes and reads of this wave done, then the barrier; unlike
    // __syncthreads() this does not wait for the loads still in flight, which
    // only fill registers.
    auto sync_next = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // Step k contracts buffer k % 3, packs K-step k + 2 into buffer
    // (k + 2) % 3 (last read in step k - 1), loads the table columns of k + 1
    // and the data of k + 4, and reads the first fragments of k + 1 (complete
    // since the previous barrier).  Indices past the end are clamped: such
    // loads and stores stay in bounds and are never used.
    Frag A0, A1;
    int bc = 0;
    auto next = [&](int k, int d) { return LOAD == FOLD ? d : k + d < nk ? k + d : nk - 1; };
    auto step = [&](const Frag& B, Frag& Bn, Data& R, int k, bool odd) __attribute__((always_inline)) {
        const int bf = bc == 2 ? 0 : bc + 1;
        const int bn = bf == 2 ? 0 : bf + 1;
        // The rotations of the next packing are loaded behind the step's last
        // wait for LDS (scalar loads return out of order, so any later wait
        // would cover them too) and ahead of its last matrix instructions.
        auto next_rot = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            load_rot(next(k, 3));
            __builtin_amdgcn_sched_barrier(0);
        };
        align_tail(R, next(k, 2));
        load_b(Bn, next(k, 1));
        if (MG == 2) load_a(A1, bc, 1);
        __builtin_amdgcn_sched_barrier(0);
        mma(A0, B, 0, [] {});
#pragma unroll
        for (int i = 0; i < 4 * PQ; ++i) rotate1(R, i, next(k, 2), odd);
        store_data(bn);
        __builtin_amdgcn_sched_barrier(0);
        if (LOAD != FOLD) load_data(R, next(k, 4));
        else if (odd) load_data(R, 3);
        load_a(A0, bf, 0);
        if (MG == 2) mma(A1, B, MG - 1, next_rot);
        else next_rot();
        __builtin_amdgcn_sched_barrier(0);
        sync_next();
        bc = bf;
        if (LOAD == FOLD && ++ck == ksteps) {
            ck = 0;
            --cj;
        }
    };

    Data R0, R1;
    Frag B0, B1;
    if (LOAD == FOLD) cj = nk / ksteps - 1;
    load_data(R0, 0);
    if (LOAD != FOLD) load_data(R1, next(0, 1));
    load_rot(0);
    load_b(B0, 0);
    align_tail(R0, 0);
    align_tail(R1, next(0, 1));
#pragma unroll
    for (int i = 0; i < 4 * PQ; ++i) rotate1(R0, i, 0, false);
    store_data(0);
    load_rot(next(0, 1));
#pragma unroll
    for (int i = 0; i < 4 * PQ; ++i) rotate1(LOAD == FOLD ? R0 : R1, i, next(0, 1), true);
    store_data(1);
    load_data(R0, next(0, 2));
    if (LOAD != FOLD) load_data(R1, next(0, 3));
    load_rot(next(0, 2));
    sync_next();
    load_a(A0, 0, 0);
    if constexpr (LOAD == FOLD) {
        // The outputs of this lane: columns 64 wave + col (Re, Im in acc[g][0],
        // acc[g][2]) and 32 further (acc[g][3], acc[g][1]).  Before each K-tile
        // acc <- r acc (the first time on zeros); ksteps is even.
        const float2 r0 = krot[n0 + 64 * wave + col], r1 = krot[n0 + 64 * wave + 32 + col];
        for (int k = 0; k < nk; k += 2) {
            if (ck == 0) {
#pragma unroll
                for (int g = 0; g < MG; ++g) {
                    turn(acc[g][0], acc[g][2], r0);
                    turn(acc[g][3], acc[g][1], r1);
                }
            }
            step(B0, B1, R0, k, false);
            step(B1, B0, R0, k + 1, true);
        }
    } else {
        int k = 0;
        for (; k + 1 < nk; k += 2) {
            step(B0, B1, R0, k, false);
            step(B1, B0, R1, k + 1, true);
        }
        if (k < nk) step(B0, B1, R0, k, false);
    }

    // Epilogue.  Rows of this lane: 32 g + 8 (v >> 2) + 4 half + (v & 3).
    if (PREC == RMSYNTH_SPLIT_FP16) {
        // Undo the per-LOS scale 2^e: multiply by 2^-e, formed from the
        // scale's exponent (exact; no division).
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t l = l0 + 32 * g + 8 * (v >> 2) + 4 * half + (v & 3);
                const float sc = los_scale[l < nlos ? l : nlos - 1];
                const float inv = __builtin_ldexpf(1.0f, 1 - __builtin_amdgcn_frexp_expf(sc));
#pragma unroll
                for (int s = 0; s < 4; ++s) acc[g][s][v] *= inv;
            }
    }
    // The sums become the outputs in place: Fq, Fu of column cp in acc[g][0],
    // acc[g][2], of column cm in acc[g][1], acc[g][3].
    const int cp = COLS ? 64 * wave + col : nh + 32 * wave + col;            // +h
    const int cm = COLS ? 64 * wave + 32 + col : nh - 1 - 32 * wave - col;  // -h
    if constexpr (COLS) {
#pragma unroll
        for (int g = 0; g < MG; ++g) {
            if constexpr (LOAD == FOLD) {
                turn(acc[g][0], acc[g][2], kbase[n0 + cp]);
                turn(acc[g][3], acc[g][1], kbase[n0 + cm]);
            }
            const f32x16_t re = acc[g][3];
            acc[g][3] = acc[g][1];
            acc[g][1] = re;
        }
    } else {
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float xc = acc[g][0][v], ys = acc[g][1][v], yc = acc[g][2][v], xs = acc[g][3][v];
            acc[g][0][v] = xc + ys;
            acc[g][1][v] = xc - ys;
            acc[g][2][v] = yc - xs;
            acc[g][3][v] = yc + xs;
        }
    }
    // Outputs go through LDS (free once every wave has passed the last K-step's
    // barrier), one quantity of the whole tile at a time, so that a store covers
    // a row's 256 phi: rows of nphi floats are in general not 16-byte aligned,
    // and the 128-byte pieces that one wave holds of a row would each touch two
    // cache lines (1024^2 LOS x 400 ch x 2001 phi, bf16x3: 12.3 -> 10.9 ms with the
    // tile order above; the non-temporal hint is 2 % of it).
    float* const sm = lds.f;
    auto put = [&](int g, int v, float p, float m) __attribute__((always_inline)) {
        float* const r = sm + (32 * g + 8 * (v >> 2) + 4 * half + (v & 3)) * SR;
        r[cp] = p;
        r[cm] = m;
    };
    auto put_all = [&](auto&& value) __attribute__((always_inline)) {
        if (!COLS && 32 * wave >= nh) return;
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                put(g, v, value(acc[g][0][v], acc[g][2][v], cp), value(acc[g][1][v], acc[g][3][v], cm));
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    if constexpr (PEAKS != 2) {
        constexpr int LR = TILE / 4, RW = 64 / LR;  // lanes per row, rows per wave and pass
        const int lc = 4 * (lane % LR), r0 = RW * wave + lane / LR;
        const int n4 = nphi - n0 - lc;  // phi left at this lane's first column
        auto store_rows = [&](float* F) __attribute__((always_inline)) {
            float* out = F + (l0 + r0) * nphi + n0 + lc;
            const float* in = sm + r0 * SR + lc;
#pragma unroll 4
            for (int i = r0; i < nl; i += NW * RW, out += NW * RW * (int64_t)nphi, in += NW * RW * SR) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(in);
                if (n4 >= 4) {
                    __builtin_nontemporal_store(v, reinterpret_cast<f32x4u_t*>(out));
                } else {
                    if (n4 > 0) out[0] = v.x;
                    if (n4 > 1) out[1] = v.y;
                    if (n4 > 2) out[2] = v.z;
                }
            }
        };
        put_all([](float q, float, int) { return q; });
        sync_next();
        store_rows(Fq);
        sync_next();
        put_all([](float, float u, int) { return u; });
        sync_next();
        store_rows(Fu);
        if (Fabs) {
            sync_next();
            put_all([](float q, float u, int) { return sqrtf(q * q + u * u); });
            sync_next();
            store_rows(Fabs);
        }
        if constexpr (PEAKS != 0) sync_next();
    }
    if constexpr (PEAKS != 0) {
        // |F|^2 (columns past the grid: -1): thread (LOS `row`, 64-phi block
        // `wave`) scans its row in phi order (strict >: ties to the lower phi)
        // and writes one record.  A |F|^2 that is not finite marks the record.
        put_all([&](float q, float u, int c) { return n0 + c < nphi ? __builtin_fmaf(q, q, u * u) : -1.0f; });
        sync_next();
        float best = -1.0f;
        int bk = 0;
        bool bad = false;
        // PEAKS 2: |F|^2 just before and after the best (prv, nxt) and at the
        // two ends of the 64 (first, last); -1 where there is none.
        float prv = -1.0f, nxt = -1.0f, first = -1.0f, last = -1.0f;
        bool want_next = false;
        const float* const frow = sm + row * SR + 64 * wave;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float4 m4 = reinterpret_cast<const float4*>(frow)[q];
            const float mm[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = mm[e];
                bad |= !(v <= FLT_MAX);
                if constexpr (PEAKS == 2) {
                    if (q == 0 && e == 0) first = v;
                    if (want_next) nxt = v;
                    want_next = false;
                    if (v > best) {
                        prv = last;
                        nxt = -1.0f;
                        want_next = true;
                    }
                    last = v;
                }
                if (v > best) {
                    best = v;
                    bk = 4 * q + e;
                }
            }
        }
        const int64_t l = l0 + lane;
        const int blk = TILE / 64 * tn + wave;
        const bool mine = lane < nl && 64 * blk < nphi;
        const int idx = bad ? -2 : 64 * blk + bk;
        if constexpr (PEAKS == 1) {
            if (mine) part[blk * part_ld + l] = PeakPart{best, idx};
        } else {
            // Fq, then Fu, through the same LDS rows: each thread picks up the
            // value at its column.
            sync_next();
            put_all([](float q, float, int) { return q; });
            sync_next();
            const float pq = frow[bk];
            sync_next();
            put_all([](float, float u, int) { return u; });
            sync_next();
            const float pu = frow[bk];
            if (mine) rec[blk * part_ld + l] = PeakRec{best, idx, pq, pu, prv, nxt, first, last};
        }
    }
}

// Plan-time tables (FP64 argument reduction, FP32 sin/cos):
//   base[tile][j] = K w_j (cos, sin)(2 pi phi_c b_j), phi_c the tile's centre;
//   T[K-step][32-pair block][4][lane], (c, s) = (cos, sin)(2 pi (i + 1/2) dphi b_j)
//   for pair i = 32 block + (lane & 31):
//     split: c hi, c lo, s hi, s lo of the channel octet lane >> 5;
//     FP32:  c, s of quad lane >> 5, then c, s of quad 2 + (lane >> 5).
__global__ void mirror_tables_kernel(const double* __restrict__ bj, const float* __restrict__ wj,
                                     int nchan_pad, int nk, int ftiles, int tile, double phi0, double dphi,
                                     double K, float2* __restrict__ base, uint4* __restrict__ Tbf,
                                     uint4* __restrict__ Thf, uint4* __restrict__ Tf32)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < (int64_t)nk * 256) {
        const int ks = (int)(idx >> 8), blk = (int)(idx >> 6) & 3, lane = (int)idx & 63;
        const double h = ((double)(32 * blk + (lane & 31)) + 0.5) * dphi;
        uint4* const at[3] = {Tbf + (idx - lane) * 4 + lane, Thf + (idx - lane) * 4 + lane,
                              Tf32 + (idx - lane) * 4 + lane};
        float c[8], s[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) phase_cos_sin(h * bj[ks * KC + 8 * (lane >> 5) + i], c[i], s[i]);
        uint32_t b[4][4], f[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            split2_bf16(c[2 * i], c[2 * i + 1], b[0][i], b[1][i]);
            split2_bf16(s[2 * i], s[2 * i + 1], b[2][i], b[3][i]);
            split2_f16(c[2 * i], c[2 * i + 1], f[0][i], f[1][i]);
            split2_f16(s[2 * i], s[2 * i + 1], f[2][i], f[3][i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            at[0][64 * i] = make_uint4(b[i][0], b[i][1], b[i][2], b[i][3]);
            at[1][64 * i] = make_uint4(f[i][0], f[i][1], f[i][2], f[i][3]);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                phase_cos_sin(h * bj[ks * KC + 4 * (2 * p + (lane >> 5)) + i], c[i], s[i]);
            at[2][64 * (2 * p)] = __builtin_bit_cast(uint4, f32x4_t{c[0], c[1], c[2], c[3]});
            at[2][64 * (2 * p + 1)] = __builtin_bit_cast(uint4, f32x4_t{s[0], s[1], s[2], s[3]});
        }
    }
    if (idx < (int64_t)ftiles * nchan_pad) {
        const int tt = (int)(idx / nchan_pad), j = (int)(idx % nchan_pad);
        float c, s;
        phase_cos_sin((phi0 + ((double)tt * tile + (tile / 2 - 0.5)) * dphi) * bj[j], c, s);
        const float kw = (float)(K * (double)wj[j]);
        base[idx] = make_float2(kw * c, kw * s);
    }
}

// Tables of the folded form (FP64 argument reduction, FP32 sin/cos):
//   T[K-step][64-output block][4][lane], (c, s) = (cos, sin)(2 pi (i + 1/2) db g)
//   of the 8 pairs of the K-step: split: hi, lo of (c, s) of the pair quad
//   lane >> 5 for output lane & 31, then for output 32 + (lane & 31); FP32: for
//   each pair quad the same two outputs, c for lanes 0-31, s for lanes 32-63;
//   kbase = K (cos, sin)(2 pi b_0' g), krot = (cos, sin)(2 pi L db g).
__global__ void fold_tables_kernel(const double* __restrict__ grid, int nphi_pad, int ksteps, double b0c,
                                   double db, double K, float2* __restrict__ kbase,
                                   float2* __restrict__ krot, uint4* __restrict__ Tbf,
                                   uint4* __restrict__ Thf, uint4* __restrict__ Tf32)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < (int64_t)ksteps * nphi_pad) {  // 64 lanes per 64-output block
        const int kk = (int)(idx / nphi_pad), at = (int)(idx % nphi_pad), lane = at & 63;
        const int64_t o = 4 * (idx - lane) + lane;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const double g = grid[at - lane + 32 * cb + (lane & 31)];
            float c[4], s[4];
            uint32_t h[4], l[4];
            auto phase = [&](int quad) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    phase_cos_sin(((double)(16 * (kk >> 1) + 2 * (4 * quad + e) + (kk & 1)) + 0.5) * db * g, c[e], s[e]);
            };
            phase(lane >> 5);
#pragma unroll
            for (int e = 0; e < 4; ++e) split2_bf16(c[e], s[e], h[e], l[e]);
            Tbf[o + 64 * (2 * cb)] = make_uint4(h[0], h[1], h[2], h[3]);
            Tbf[o + 64 * (2 * cb + 1)] = make_uint4(l[0], l[1], l[2], l[3]);
#pragma unroll
            for (int e = 0; e < 4; ++e) split2_f16(c[e], s[e], h[e], l[e]);
            Thf[o + 64 * (2 * cb)] = make_uint4(h[0], h[1], h[2], h[3]);
            Thf[o + 64 * (2 * cb + 1)] = make_uint4(l[0], l[1], l[2], l[3]);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                phase(p);
                const f32x4_t v = lane < 32 ? f32x4_t{c[0], c[1], c[2], c[3]} : f32x4_t{s[0], s[1], s[2], s[3]};
                Tf32[o + 64 * (2 * p + cb)] = __builtin_bit_cast(uint4, v);
            }
        }
    }
    if (idx < nphi_pad) {
        float c, s;
        phase_cos_sin(b0c * grid[idx], c, s);
        kbase[idx] = make_float2((float)K * c, (float)K * s);
        phase_cos_sin((double)(ksteps * KC) * db * grid[idx], c, s);
        krot[idx] = make_float2(c, s);
    }
}

// Table of the table form: T[K-step][64-output block][4][lane] as in the folded
// form, (c, s) = (cos, sin)(2 pi b_j phi_k) of the K-step's 8 channels;
// ew_j = (K w_j, 0).
__global__ void phase_table_kernel(const double* __restrict__ bj, const double* __restrict__ phik,
                                   const float* __restrict__ wj, int nchan_pad, int nphi_pad, double K,
                                   float2* __restrict__ ew, uint4* __restrict__ Tbf,
                                   uint4* __restrict__ Thf, uint4* __restrict__ Tf32)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < (int64_t)(nchan_pad / 8) * nphi_pad) {
        const int kk = (int)(idx / nphi_pad), at = (int)(idx % nphi_pad), lane = at & 63;
        const int64_t o = 4 * (idx - lane) + lane;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const double g = phik[at - lane + 32 * cb + (lane & 31)];
            float c[2][4], s[2][4];  // both channel quads
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) phase_cos_sin(g * bj[8 * kk + 4 * p + e], c[p][e], s[p][e]);
            uint32_t h[4], l[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float ce = lane < 32 ? c[0][e] : c[1][e], se = lane < 32 ? s[0][e] : s[1][e];
                split2_bf16(ce, se, h[e], l[e]);
            }
            Tbf[o + 64 * (2 * cb)] = make_uint4(h[0], h[1], h[2], h[3]);
            Tbf[o + 64 * (2 * cb + 1)] = make_uint4(l[0], l[1], l[2], l[3]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float ce = lane < 32 ? c[0][e] : c[1][e], se = lane < 32 ? s[0][e] : s[1][e];
                split2_f16(ce, se, h[e], l[e]);
            }
            Thf[o + 64 * (2 * cb)] = make_uint4(h[0], h[1], h[2], h[3]);
            Thf[o + 64 * (2 * cb + 1)] = make_uint4(l[0], l[1], l[2], l[3]);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const f32x4_t v = lane < 32 ? f32x4_t{c[p][0], c[p][1], c[p][2], c[p][3]}
                                            : f32x4_t{s[p][0], s[p][1], s[p][2], s[p][3]};
                Tf32[o + 64 * (2 * p + cb)] = __builtin_bit_cast(uint4, v);
            }
        }
    }
    if (idx < nchan_pad) ew[idx] = make_float2((float)(K * (double)wj[idx]), 0.0f);
}

template <int LOAD, int PREC, int MG, int NW>
hipError_t launch(const rmsynth_plan_s& p, const ExecArgs& a)
{
    constexpr bool tab = LOAD == TAB_ROW || LOAD == TAB_PLANE;
    constexpr int kc = tab ? 8 : KC;
    // Folded: K-tiles of ksteps K-steps, kpad channels below channel 0.
    const int nk = LOAD == FOLD ? (p.nchan + p.kpad) / KC : (p.nchan + kc - 1) / kc;
    const int tiles_n = LOAD == FOLD || tab ? (p.nphi + 64 * NW - 1) / (64 * NW) : p.ftiles;
    constexpr int sub = tiles_per_wg(LOAD, NW), rows = 32 * MG * sub;  // LOS per workgroup
    const int64_t blocks = (a.nlos + rows - 1) / rows * tiles_n;
    if (blocks <= 0) return hipSuccess;
    const bool rows_one = LOAD == LOAD_ONE && a.layout == RMSYNTH_LOS_MAJOR;  // below 4 channels
    const int64_t ld = rows_one ? 1 : a.ld;
    const int ls = rows_one ? p.nchan : 1;
    const uint4* T = PREC == RMSYNTH_FP32 ? p.d_Tf32 : PREC == RMSYNTH_SPLIT_FP16 ? p.d_Thf : p.d_Tbf;
#define RMS_LAUNCH(G, P)                                                                                    \
    hipLaunchKernelGGL((synth_mirrored_kernel<LOAD, PREC, G, P, MG, NW>), dim3((unsigned)blocks),            \
                       dim3(64 * NW * sub), 0, a.stream, a.Q, a.U, a.nlos, ld, p.nchan, p.d_base, T, p.nchan_pad, \
                       nk, p.nphi, tiles_n, a.Fq, a.Fu, a.Fabs, a.los_scale, a.peak_part, a.peak_part_ld,     \
                       a.peak_rec, 4 * p.nphi_pad, p.ksteps, p.kpad, p.d_kbase, p.d_krot, ls,                 \
                       mirror_tile(p) / 2)
#define RMS_LAUNCH_P(G)                                                               \
    do {                                                                              \
        if constexpr (PREC != RMSYNTH_FP32 && LOAD != FOLD) { /* elsewhere peaks are a kernel of their own */ \
            if (a.peak_rec) RMS_LAUNCH(G, 2);                                         \
            else if (a.peak_part) RMS_LAUNCH(G, 1);                                   \
            else RMS_LAUNCH(G, 0);                                                    \
        } else {                                                                      \
            RMS_LAUNCH(G, 0);                                                         \
        }                                                                             \
    } while (0)
    if constexpr (LOAD != FOLD) {
        if (p.any_flagged) RMS_LAUNCH_P(true);
        else RMS_LAUNCH_P(false);
    } else {
        RMS_LAUNCH_P(false);  // adjoint plans weight every channel 1
    }
#undef RMS_LAUNCH_P
#undef RMS_LAUNCH
    return hipGetLastError();
}

// Half-height tiles where full ones would leave half of the chip's 1024 SIMDs
// without a wave: such a call is bound by the latency of one tile (64^2 LOS x
// 128 ch x 201 phi, 64 full tiles of 4 waves: bf16x3 12.7 -> 9.8 us, FP32 24.1 ->
// 15.8; 64 LOS x 400 x 2001, 8 tiles: 19.4 -> 14.5).  At 256 full tiles both take
// the same time (26 us), at 512 the half-height ones 10 % more.
template <int LOAD, int PREC, int NW>
hipError_t launch_mg(const rmsynth_plan_s& p, const ExecArgs& a)
{
    const int64_t waves = (a.nlos + 63) / 64 * ((p.nphi + 64 * NW - 1) / (64 * NW)) * NW;
    return waves <= kSmallWaves ? launch<LOAD, PREC, 1, NW>(p, a) : launch<LOAD, PREC, 2, NW>(p, a);
}

// Output columns come in tiles of 256, or of 128 where that pads fewer.  A narrow
// tile packs its rows for half the matrix work, so what the matrix cores bound
// gains less than what is not padded.
template <int LOAD, int PREC>
hipError_t launch_cols(const rmsynth_plan_s& p, const ExecArgs& a)
{
    const int64_t n128 = (p.nphi + 127) / 128, n256 = (p.nphi + 255) / 256, tiles = (a.nlos + 63) / 64;
    bool narrow = n128 < 2 * n256;
    if constexpr (LOAD == FOLD) {
        // One narrow tile gains (262144 LOS x 1201 -> 100 channels bf16x3 1.14 ->
        // 1.09 ms).  The split forms read the rows once per tile and are bound by
        // that: three instead of two wide ones lose (288 channels 1.96 -> 2.24).
        // FP32 gains (1201 -> 288 channels 5.01 -> 3.93 ms) once there are
        // workgroups for every SIMD (500 -> 300 channels: 4096 LOS 42 us wide, 70
        // narrow, 16384 137 and 138, 65536 532 and 422).
        narrow = narrow && (p.nphi <= 128 || (PREC == RMSYNTH_FP32 && tiles * n128 >= 1024));
    } else {
        // The time of a workgroup times the most that a CU is given of them, in
        // units of a half-height one (launch_mg); narrow ones take 17/16 (FP32) or
        // 19/16 (split) of a wide one's.  256 channels x 300 phi, wide and narrow:
        // 8192 LOS bf16x3 24 and 26 us, FP32 68 and 71; 65536 LOS 163 and 148,
        // 511 and 396; 880 phi bf16x3 342 and 346.  With few channels the stores of F
        // take longest, which wide tiles make in longer pieces (200000 LOS, wide and
        // narrow: 24 ch x 600 phi bf16x3 248 and 287, 7 x 300 FP32 157 and 174, but
        // 17 x 300 219 and 182); the search stores none (12 x 300 98 and 85).
        auto rounds = [](int64_t full) { return full <= 128 ? 1 : 2 * ((full + 255) / 256); };
        const int few = a.peak_rec ? 0 : PREC == RMSYNTH_FP32 ? 16 : 64;
        narrow = narrow && (n128 == 1 || p.nchan >= few) &&
                 (PREC == RMSYNTH_FP32 ? 17 : 19) * rounds((tiles + 1) / 2 * n128) < 16 * rounds(tiles * n256);
    }
    return narrow ? launch_mg<LOAD, PREC, 2>(p, a) : launch_mg<LOAD, PREC, 4>(p, a);
}

// Mirrored pairs.  Grids of at most 128 phi are one tile of 64 pairs: on two waves,
// in pairs of tiles, or, where that would leave the chip short of waves, on the
// first two of the four (the others pack; the values are the same).  With tiles
// of 128 pairs on four waves, 262144 LOS x 24 ch x 20 phi took, bf16x3 61 us, FP32
// 110 (now 39 and 62), 131072 x 128 x 100 bf16x3 72 (57), 4096 x 400 x 100 bf16x3
// 15 (19 on two waves).
template <int LOAD, int PREC>
hipError_t launch_pairs(const rmsynth_plan_s& p, const ExecArgs& a)
{
    const int64_t waves = (a.nlos + 63) / 64 * 4;
    return mirror_tile(p) == 128 && waves > kSmallWaves ? launch_mg<LOAD, PREC, 2>(p, a)
                                                                         : launch_mg<LOAD, PREC, 4>(p, a);
}

template <int PREC>
hipError_t launch_load(const rmsynth_plan_s& p, const ExecArgs& a)
{
    const bool planes = a.layout != RMSYNTH_LOS_MAJOR;
    if (p.cuniform) return launch_cols<FOLD, PREC>(p, a);
    if (p.etab) return planes ? launch_cols<TAB_PLANE, PREC>(p, a) : launch_cols<TAB_ROW, PREC>(p, a);
    if (planes || p.nchan < 4) return launch_pairs<LOAD_ONE, PREC>(p, a);
    // Quads of any alignment: with single values, 10007 LOS x 333 ch x 777 phi took
    // 80 us in bf16x3 (now 60) and 165 in FP32 (145), 65536 LOS 405 (297) and 819
    // (711).  The move of the row's last quad costs 1 %, so 4 n channels go without.
    return p.nchan % 4 ? launch_pairs<LOAD_TAIL, PREC>(p, a) : launch_pairs<LOAD_ROW4, PREC>(p, a);
}

}  // namespace

hipError_t launch_synth_mirrored(const rmsynth_plan_s& p, const ExecArgs& a, int precision)
{
    if (precision == RMSYNTH_FP32) return launch_load<RMSYNTH_FP32>(p, a);
    if (precision == RMSYNTH_SPLIT_FP16) return launch_load<RMSYNTH_SPLIT_FP16>(p, a);
    return launch_load<RMSYNTH_SPLIT_BF16>(p, a);
}

hipError_t launch_mirror_tables(const rmsynth_plan_s& p, hipStream_t stream)
{
    const int nk = (p.nchan + KC - 1) / KC;
    const int64_t n = std::max<int64_t>((int64_t)nk * 256, (int64_t)p.ftiles * p.nchan_pad);
    hipLaunchKernelGGL(mirror_tables_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       p.d_b, p.d_w, p.nchan_pad, nk, p.ftiles, mirror_tile(p), p.phi0, p.dphi, p.K, p.d_base, p.d_Tbf,
                       p.d_Thf, p.d_Tf32);
    return hipGetLastError();
}

hipError_t launch_fold_tables(const rmsynth_plan_s& p, hipStream_t stream)
{
    // centre of the lowest K-tile: channel -kpad + L/2 - 1/2
    const double b0c = p.kb0 + (0.5 * p.ksteps * KC - 0.5 - p.kpad) * p.kdb;
    const int64_t n = (int64_t)p.ksteps * p.nphi_pad;
    hipLaunchKernelGGL(fold_tables_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       p.d_phi, p.nphi_pad, p.ksteps, b0c, p.kdb, p.K, p.d_kbase, p.d_krot, p.d_Tbf,
                       p.d_Thf, p.d_Tf32);
    return hipGetLastError();
}

hipError_t launch_phase_table(const rmsynth_plan_s& p, hipStream_t stream)
{
    const int64_t n = std::max<int64_t>((int64_t)(p.nchan_pad / 8) * p.nphi_pad, p.nchan_pad);
    hipLaunchKernelGGL(phase_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p.d_b,
                       p.d_phi, p.d_w, p.nchan_pad, p.nphi_pad, p.K, p.d_base, p.d_Tbf, p.d_Thf, p.d_Tf32);
    return hipGetLastError();
}
