// RM-CLEAN: deconvolution of the Faraday spectrum by the RMSF (the use of
// R(phi), eq. (12), that Section 2.2 names and leaves unsupported; Section 4).
// Hogbom's iteration on a uniform phi grid, for every LOS independently:
//
//   r <- F;  C <- 0
//   repeat at most max_iter times:
//     p = lowest index maximising |r_k|^2;  stop when |r_p| < cutoff
//     c = gain r_p;  C_p += c;  r_k -= c R((k - p) dphi)  for every k
//   restored_k = r_k + sum_m C_m G((k - m) dphi),  G(x) = exp(-4 ln2 x^2 / fwhm^2)
//
// One wave per LOS, the residual in registers (element k = 64 e + lane, at
// most 64 per lane: nphi <= 4096).  An iteration is bound by vector
// instructions, 64 E lanes of them per wave, so it is written for few:
//   pick      |r|^2 and running maxima of E/8 elements each (2.5 instructions
//             an element), the wave's maximum by DPP; the element that holds
//             it is then looked for with scalar branches, lowest index first,
//             group by group, and its r read from the owner lane
//   stop      |r|^2 against the smallest square whose root reaches the cutoff
//   subtract  R from LDS at one address per wave plus constants (the table is
//             staged padded to 64 E + N - 1 entries, so no index is clamped)
//   C         the row's own load and store, waited for after the subtraction
// Widths step by 2 to 8 elements per lane; those below the previous width
// need no test for the end of the grid.  65536 LOS x 2001 phi, 8 picks a LOS:
// 1.37 -> 0.90 ms, the time of a copy of its 32 bytes an element (0.88 ms);
// 32768 LOS x 601: 225 -> 137 us; 512 x 700, a chain of 24 picks: 41 -> 22 us.
// R on the doubled grid (m - (N-1)) dphi, m = 0 .. 2N-2, and G on the same
// offsets are built per call into the workspace (FP64 argument reduction,
// FP32 sin/cos and accumulation in channel order, as the RMSF).  A per-lane
// bit mask remembers which of its elements hold a component; the restore
// visits only those, and around each only the elements where G is not 0.  A
// LOS whose F is not finite is flagged (niter = -1, every output NaN).
#include <float.h>
#include <math.h>

#include "common.h"

namespace {

constexpr int kWaves = 4;  // LOS (waves) per workgroup

// R((m - (N-1)) dphi) = K sum_j w_j exp(-2i x a_j) and G at the same offsets:
// 4 offsets per workgroup, whose 256 threads take the sines and cosines of 256
// channels at a time into LDS; 8 threads then add them in channel order.  (One
// thread per offset was a chain of 400 FP64 reductions on a sixteenth of the CUs:
// 90 us for 2001 phi x 400 channels, now 12.)
constexpr int kTabM = 4, kTabJ = 256;

__global__ __launch_bounds__(256) void rmclean_tables_kernel(
    const double* __restrict__ bj, const float* __restrict__ wj, int nchan, int N, double dphi,
    float K, double fwhm, float2* __restrict__ R2, float* __restrict__ G)
{
    __shared__ float cs[2][kTabM][kTabJ + 4];
    __shared__ float wl[kTabJ];
    const int tid = threadIdx.x, m0 = blockIdx.x * kTabM;
    const int am = tid & (kTabM - 1), ai = (tid / kTabM) & 1;  // the sum of threads 0 .. 7
    float sum = 0.0f;
    for (int j0 = 0; j0 < nchan; j0 += kTabJ) {
        const int n = min(kTabJ, nchan - j0);
        const bool in = tid < n;
        const double b = in ? bj[j0 + tid] : 0.0;
        wl[tid] = in ? wj[j0 + tid] : 0.0f;
#pragma unroll 2
        for (int m = 0; m < kTabM; ++m) {
            float c, s;
            phase_cos_sin((double)(m0 + m - (N - 1)) * dphi * b, c, s);
            cs[0][m][tid] = c;
            cs[1][m][tid] = -s;
        }
        __syncthreads();
        if (tid < 2 * kTabM) {
#pragma unroll 16
            for (int j = 0; j < n; ++j) {
                const float w = wl[j];
                const float t = __builtin_fmaf(w, cs[ai][am][j], sum);
                sum = w == 0.0f ? sum : t;
            }
        }
        __syncthreads();
    }
    const int m = m0 + am;
    if (tid >= 2 * kTabM || m >= 2 * N - 1) return;
    reinterpret_cast<float*>(R2)[2 * m + ai] = K * sum;
    if (ai) return;
    const double z = (double)(m - (N - 1)) * dphi / fwhm;
    G[m] = (float)exp(-4.0 * 0.69314718055994530942 * z * z);
}

template <int CTRL>
__device__ __forceinline__ float dpp_max(float v)
{
    const int x = __builtin_bit_cast(int, v);
    return __builtin_fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, CTRL, 0xf, 0xf, false)));
}

// Largest value of the wave, in every lane: row_shr 1, 2, 4, 8 leave a row's
// maximum in its lane 15, row_bcast15 and row_bcast31 carry it to lane 63.
__device__ __forceinline__ float wave_max(float v)
{
    v = dpp_max<0x111>(v);
    v = dpp_max<0x112>(v);
    v = dpp_max<0x114>(v);
    v = dpp_max<0x118>(v);
    v = dpp_max<0x142>(v);
    v = dpp_max<0x143>(v);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// Registers: 2 E for the residual, the rest for reads of R in flight.
constexpr int waves_per_simd(int E) { return E <= 32 ? 4 : E <= 40 ? 3 : 2; }

// E elements per lane; those from E0 on may lie past the grid.
template <int E, int E0>
__global__ __launch_bounds__(64 * kWaves, waves_per_simd(E)) void rmclean_kernel(
    const float* Fq, const float* Fu, int64_t nlos, int N, const float2* __restrict__ R2g,
    const float* __restrict__ G, float gain, float stop2, int max_iter, int reach, float* rq,
    float* ru, float* cq, float* cu, float* __restrict__ Rq, float* __restrict__ Ru,
    int32_t* __restrict__ niter)
{
    extern __shared__ float4 smem4[];
    float2* R2 = reinterpret_cast<float2*>(smem4);
    const bool restore = Rq != nullptr;
    for (int i = threadIdx.x; i < N - 1 + 64 * E; i += 64 * kWaves)
        R2[i] = i < 2 * N - 1 ? R2g[i] : make_float2(0.0f, 0.0f);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t l = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (l >= nlos) return;  // uniform per wave; no block barrier follows
    const int64_t row = l * N;

    // Elements past the grid (k >= N) hold whatever the padding makes of
    // them; their |r|^2 is taken as -1, and they are never stored.
    float xr[E], xi[E];
    bool bad = false;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = 64 * e + lane;
        const int kc = k < N ? k : N - 1;
        xr[e] = Fq[row + kc];
        xi[e] = Fu[row + kc];
        bad |= !(__builtin_fabsf(xr[e]) <= FLT_MAX && __builtin_fabsf(xi[e]) <= FLT_MAX);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = 64 * e + lane;
        if (k < N) {
            cq[row + k] = 0.0f;
            cu[row + k] = 0.0f;
        }
    }
    if (__any(bad)) {
        const float nan = __builtin_nanf("");
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = 64 * e + lane;
            if (k < N) {
                rq[row + k] = nan;
                ru[row + k] = nan;
                cq[row + k] = nan;
                cu[row + k] = nan;
                if (restore) {
                    Rq[row + k] = nan;
                    Ru[row + k] = nan;
                }
            }
        }
        if (niter && lane == 0) niter[l] = -1;
        return;
    }

    constexpr int GS = (E + 7) / 8, NG = (E + GS - 1) / GS;  // elements per group, groups
    auto power = [&](int e, float a, float b) {
        const float a2 = __builtin_fmaf(a, a, b * b);
        return e < E0 || 64 * e + lane < N ? a2 : -1.0f;
    };
    uint64_t has = 0;  // bit e: element 64 e + lane holds a component
    int it = 0;
    for (; it < max_iter; ++it) {
        float gm[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            gm[g] = power(g * GS, xr[g * GS], xi[g * GS]);
#pragma unroll
            for (int i = 1; i < GS; ++i)
                if (g * GS + i < E)
                    gm[g] = __builtin_fmaxf(gm[g], power(g * GS + i, xr[g * GS + i], xi[g * GS + i]));
        }
        float best = gm[0];
#pragma unroll
        for (int g = 1; g < NG; ++g) best = __builtin_fmaxf(best, gm[g]);
        best = wave_max(best);
        if (!(best >= stop2)) break;  // also when no element is a number any more
        int bk = 0;
        float br = 0.0f, bi = 0.0f;
        auto pick = [&]() {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (!__ballot(gm[g] == best)) continue;
#pragma unroll
                for (int i = 0; i < GS; ++i) {
                    const int e = g * GS + i;
                    if (e >= E) break;
                    // taken again (E more registers would hold the first)
                    float a = xr[e], b = xi[e];
                    asm volatile("" : "+v"(a), "+v"(b));
                    const uint64_t at = __ballot(power(e, a, b) == best);
                    if (!at) continue;
                    const int j = __builtin_ctzll(at);
                    bk = 64 * e + j;
                    br = lane_value(a, j);
                    bi = lane_value(b, j);
                    has |= lane == j ? uint64_t(1) << e : 0;
                    return;
                }
            }
        };
        pick();
        const float cr = gain * br, ci = gain * bi;
        // Loaded at one address in every lane (only its owner's value counts).
        float* const pq = cq + row + bk;
        float* const pu = cu + row + bk;
        float c0 = *pq, c1 = *pu;
        const float2* const Rk = R2 + (N - 1 - bk) + lane;
        // the reads of the next few elements fly while these are updated
        constexpr int B = E <= 24 ? 8 : 4;
        float2 R[2][B];
#pragma unroll
        for (int i = 0; i < B && i < E; ++i) R[0][i] = Rk[64 * i];
#pragma unroll
        for (int e0 = 0; e0 < E; e0 += B) {
            const int cur = e0 / B & 1;
#pragma unroll
            for (int i = 0; i < B; ++i)
                if (e0 + B + i < E) R[cur ^ 1][i] = Rk[64 * (e0 + B + i)];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int e = e0 + i;
                if (e >= E) break;
                const float2 r = R[cur][i];
                xr[e] = __builtin_fmaf(-cr, r.x, __builtin_fmaf(ci, r.y, xr[e]));
                xi[e] = __builtin_fmaf(-cr, r.y, __builtin_fmaf(-ci, r.x, xi[e]));
                asm volatile("" : "+v"(xr[e]), "+v"(xi[e]));  // here, not behind the branch below
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" : "+v"(c0), "+v"(c1));  // the loads stay ahead of the subtraction
        if (lane == (bk & 63)) {
            *pq = c0 + cr;
            *pu = c1 + ci;
        }
    }
    if (niter && lane == 0) niter[l] = it;
    // a copy the compiler takes for another value: no address of the loads
    // above stays in registers through the iterations
    int lane2 = lane;
    asm volatile("" : "+v"(lane2));
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = 64 * e + lane2;
        if (k < N) {
            rq[row + k] = xr[e];
            ru[row + k] = xi[e];
        }
    }
    if (!restore) return;
    // restored = residual + components convolved with G, component by
    // component in (e, lane) order (the outer loop is kept rolled: only the
    // inner one indexes the register arrays).
    const int last = 2 * N - 2;
#pragma unroll 1
    for (int e = 0; e < E; ++e) {
        uint64_t m = __ballot((has >> e) & 1);
        float vr = 0.0f, vi = 0.0f;
        if ((has >> e) & 1) {
            vr = cq[row + 64 * e + lane2];
            vi = cu[row + 64 * e + lane2];
        }
        while (m) {
            const int j = __builtin_ctzll(m);
            m &= m - 1;
            const int kc = 64 * e + j;
            const float c_r = lane_value(vr, j), c_i = lane_value(vi, j);
            const int base = N - 1 - kc;
            constexpr int B = 4;
#pragma unroll
            for (int e0 = 0; e0 < E; e0 += B) {
                if (64 * (e0 + B) <= kc - reach || 64 * e0 > kc + reach) continue;
#pragma unroll
                for (int e2 = e0; e2 < e0 + B && e2 < E; ++e2) {
                    const int t = base + 64 * e2 + lane2;
                    const float g = G[t < last ? t : last];
                    xr[e2] = __builtin_fmaf(c_r, g, xr[e2]);
                    xi[e2] = __builtin_fmaf(c_i, g, xi[e2]);
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = 64 * e + lane2;
        if (k < N) {
            Rq[row + k] = xr[e];
            Ru[row + k] = xi[e];
        }
    }
}

struct CleanArgs {
    const float *Fq, *Fu;
    int64_t nlos;
    int N;
    const float2* R2;
    const float* G;
    float gain, stop2;
    int max_iter, reach;
    float *rq, *ru, *cq, *cu, *Rq, *Ru;
    int32_t* niter;
    hipStream_t s;
};

template <int E, int E0>
hipError_t launch_e(const CleanArgs& a)
{
    const size_t lds = (size_t)(a.N - 1 + 64 * E) * sizeof(float2);
    for (int64_t l0 = 0; l0 < a.nlos;) {
        const int64_t n = std::min<int64_t>(a.nlos - l0, max_items(kWaves, 64 * kWaves));
        const int64_t off = l0 * a.N;
        hipLaunchKernelGGL((rmclean_kernel<E, E0>), dim3((unsigned)((n + kWaves - 1) / kWaves)),
                           dim3(64 * kWaves), lds, a.s, a.Fq + off, a.Fu + off, n, a.N, a.R2, a.G,
                           a.gain, a.stop2, a.max_iter, a.reach, a.rq + off, a.ru + off, a.cq + off,
                           a.cu + off, a.Rq ? a.Rq + off : nullptr, a.Ru ? a.Ru + off : nullptr,
                           a.niter ? a.niter + l0 : nullptr);
        if (hipError_t e = hipGetLastError()) return e;
        l0 += n;
    }
    return hipSuccess;
}

// The narrowest width that holds the grid.
template <int E0, int E, int... WIDER>
hipError_t launch_width(const CleanArgs& a)
{
    if constexpr (sizeof...(WIDER) > 0)
        if (a.N > 64 * E) return launch_width<E, WIDER...>(a);
    return launch_e<E, E0>(a);
}

// Smallest x >= 0 whose rounded square root is at least cutoff (>= 0, finite).
float square_reaching(float cutoff)
{
    float x = cutoff * cutoff;
    while (x > 0.0f && sqrtf(x) >= cutoff) x = nextafterf(x, 0.0f);
    while (sqrtf(x) < cutoff) x = nextafterf(x, INFINITY);
    return x;
}

}  // namespace

size_t rmclean_table_bytes(const rmsynth_plan_s& p)
{
    return (size_t)round_up((int64_t)(2 * p.nphi - 1) * (int64_t)sizeof(float2), 256) +
           (size_t)round_up((int64_t)(2 * p.nphi - 1) * (int64_t)sizeof(float), 256);
}

hipError_t launch_rmclean(const rmsynth_plan_s& p, const float* Fq, const float* Fu, int64_t nlos,
                          float gain, float cutoff, int max_iter, double fwhm, float* rq, float* ru,
                          float* cq, float* cu, float* Rq, float* Ru, int32_t* niter, void* ws,
                          hipStream_t s)
{
    const int N = p.nphi;
    float2* R2 = static_cast<float2*>(ws);
    float* G = reinterpret_cast<float*>(static_cast<char*>(ws) +
                                        round_up((int64_t)(2 * N - 1) * (int64_t)sizeof(float2), 256));
    hipLaunchKernelGGL(rmclean_tables_kernel, dim3((unsigned)((2 * N - 1 + kTabM - 1) / kTabM)), dim3(256), 0,
                       s, p.d_b, p.d_w, p.nchan, N, p.dphi, (float)p.K, fwhm, R2, G);
    if (hipError_t e = hipGetLastError()) return e;
    if (nlos == 0) return hipSuccess;
    // G = 2^(-4 z^2) at z beam widths rounds to 0 from z = 6.124 on
    const double span = 6.125 * fwhm / std::fabs(p.dphi) + 2.0;
    const int reach = span < N ? (int)span : N;
    const CleanArgs a{Fq, Fu, nlos, N, R2, G, gain, square_reaching(cutoff), max_iter, reach,
                      rq, ru, cq, cu, Rq, Ru, niter, s};
    return launch_width<0, 4, 6, 8, 10, 12, 16, 20, 24, 28, 32, 40, 48, 56, 64>(a);
}
