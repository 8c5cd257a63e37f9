// Faraday-depth transform on a uniform phi grid by a non-uniform FFT (the
// FFT evaluation the paper proposes in place of the direct sums of
// eqs. (15)-(16), Section 4).  With phi_k = phi_c + m dphi, m = k - kc,
// eq. (11) is a type-1 non-uniform DFT in m:
//
//   F_k = sum_j c_j exp(-i m x_j),  c_j = K w_j P_j exp(-2i a_j phi_c),
//                                   x_j = 2 a_j dphi (mod 2 pi),
//
// evaluated by gridding each c_j onto n >= 2N uniform points of [0, 2 pi)
// with the "exponential of semicircle" kernel psi of width W grid cells
// (Barnett, Magland & af Klinteberg 2019), an n-point FFT, and division of
// mode m by the kernel's Fourier transform psi_hat(m).  The gridding weights
// (per grid point, the channels within the kernel's reach), c_j's rotation,
// the twiddles and 1/psi_hat are plan-time tables built on the host in FP64.
//
// A band of lambda^2 occupies one stretch of the grid, often a small one.  The
// plan rotates the grid so that the stretch starts at point 0 (a phase per
// mode, kept with 1/psi_hat) and, when it fits the first n / 2^B1 points, only
// those are gridded: a first FFT pass of radix 2^B1 would see one non-zero
// input per butterfly and copy it to its 2^B1 outputs, so the next pass reads
// its inputs straight from the short grid.
//
// T = n / 8 threads (16 to 512) per LOS, or one per point on small grids with many
// channels; several LOS per workgroup of up to 256 threads where T is less.  The channels' c_j go to LDS; each thread sums
// grid points from their lists of entries (a fixed order, no atomics; the
// entries of 64 neighbouring points are interleaved, so that a wave reads
// them contiguously, the first of each block of points a block ahead: 32768 LOS x
// 64 ch x 1500 phi 335 -> 264 us).  The FFT runs as Stockham passes of radix 8 or 16 in
// registers, three for n / 2^B1 up to 4096, through LDS; the last one scales
// its modes and stores them.
//
// What bounds it: VALU issue (60 % of the time at the first size below,
// SQ_ACTIVE_INST_VALU over SQ_BUSY_CU_CYCLES) and the waits between the passes of
// a LOS.  Per launch, before (radix-16 passes
// over the whole grid, one contiguous list of entries per point) and after:
//   262144 LOS x 400 ch x 2001 phi, 1/8 of 4096 points    4.07 -> 2.66 ms
//   262144 x 288 x 1201, 1/64 of 4096                     4.59 -> 1.88 ms
//   262144 x 128 x 201, all of 512                        0.86 -> 0.40 ms
//   65536 x 1024 x 4001, all of 8192                      3.34 -> 1.98 ms
#include <type_traits>

#include "common.h"

namespace {

constexpr int kThreads = 256;  // threads per workgroup where several LOS share one

__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(__builtin_fmaf(a.x, b.x, -a.y * b.y), __builtin_fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// -i z
__device__ __forceinline__ float2 cmul_mi(float2 z) { return make_float2(z.y, -z.x); }

// DFTs of 2, 4, 8 and 16 points in registers, X_q = sum_r x_r exp(-2 pi i r q / R),
// in place.  The roots of unity are the exact values cos(pi/4) = sqrt(2)/2,
// cos(pi/8), sin(pi/8).
constexpr float kC4 = 0.70710678118654752440f;   // cos(pi/4)
constexpr float kC8 = 0.92387953251128675613f;   // cos(pi/8)
constexpr float kS8 = 0.38268343236508977173f;   // sin(pi/8)

__device__ __forceinline__ void dft2(float2* x)
{
    const float2 a = x[0], b = x[1];
    x[0] = cadd(a, b);
    x[1] = csub(a, b);
}
__device__ __forceinline__ void dft4(float2& x0, float2& x1, float2& x2, float2& x3)
{
    const float2 a0 = cadd(x0, x2), a1 = csub(x0, x2);
    const float2 a2 = cadd(x1, x3), a3 = cmul_mi(csub(x1, x3));
    x0 = cadd(a0, a2);
    x1 = cadd(a1, a3);
    x2 = csub(a0, a2);
    x3 = csub(a1, a3);
}
__device__ __forceinline__ void dft4(float2* x) { dft4(x[0], x[1], x[2], x[3]); }
// 8 points: DFT4 of the even and the odd samples, X_q = E_q + w8^q O_q.
__device__ __forceinline__ void dft8(float2* x)
{
    float2 e0 = x[0], e1 = x[2], e2 = x[4], e3 = x[6];
    float2 o0 = x[1], o1 = x[3], o2 = x[5], o3 = x[7];
    dft4(e0, e1, e2, e3);
    dft4(o0, o1, o2, o3);
    o1 = make_float2(kC4 * (o1.x + o1.y), kC4 * (o1.y - o1.x));     // x w8^1
    o2 = cmul_mi(o2);                                               // x w8^2
    o3 = make_float2(kC4 * (o3.y - o3.x), -kC4 * (o3.x + o3.y));    // x w8^3
    x[0] = cadd(e0, o0); x[4] = csub(e0, o0);
    x[1] = cadd(e1, o1); x[5] = csub(e1, o1);
    x[2] = cadd(e2, o2); x[6] = csub(e2, o2);
    x[3] = cadd(e3, o3); x[7] = csub(e3, o3);
}
// 16 points as 4 x 4: r = 4 r1 + r2, q = q1 + 4 q2;
// X_{q1 + 4 q2} = sum_r2 w4^{r2 q2} w16^{r2 q1} [sum_r1 x_{4 r1 + r2} w4^{r1 q1}].
__device__ __forceinline__ void dft16(float2* x)
{
    float2 y[4][4];
#pragma unroll
    for (int r2 = 0; r2 < 4; ++r2) {
        y[r2][0] = x[r2]; y[r2][1] = x[4 + r2]; y[r2][2] = x[8 + r2]; y[r2][3] = x[12 + r2];
        dft4(y[r2]);
    }
    // w16^m for m = r2 q1: 1, 2, 3 (r2 = 1); 2, 4, 6 (r2 = 2); 3, 6, 9 (r2 = 3)
    const float2 w1 = make_float2(kC8, -kS8), w2 = make_float2(kC4, -kC4), w3 = make_float2(kS8, -kC8);
    const float2 w6 = make_float2(-kC4, -kC4), w9 = make_float2(-kC8, kS8);
    y[1][1] = cmul(y[1][1], w1); y[1][2] = cmul(y[1][2], w2); y[1][3] = cmul(y[1][3], w3);
    y[2][1] = cmul(y[2][1], w2); y[2][2] = cmul_mi(y[2][2]); y[2][3] = cmul(y[2][3], w6);
    y[3][1] = cmul(y[3][1], w3); y[3][2] = cmul(y[3][2], w6); y[3][3] = cmul(y[3][3], w9);
#pragma unroll
    for (int q1 = 0; q1 < 4; ++q1) {
        float2 z0 = y[0][q1], z1 = y[1][q1], z2 = y[2][q1], z3 = y[3][q1];
        dft4(z0, z1, z2, z3);
        x[q1] = z0; x[q1 + 4] = z1; x[q1 + 8] = z2; x[q1 + 12] = z3;
    }
}
template <int R>
__device__ __forceinline__ void dft(float2* x)
{
    if constexpr (R == 2) dft2(x);
    else if constexpr (R == 4) dft4(x);
    else if constexpr (R == 8) dft8(x);
    else dft16(x);
}

// LDS position of grid element i: the low five bits XOR-ed with bits 4 to 8, so
// that the strided accesses of the passes fall on distinct banks; a
// permutation inside each aligned block of 512 elements.
__device__ __forceinline__ int swz(int i) { return i ^ ((i >> 4) & 31); }

// Radices (log2) of the passes over the 2^M points that are left after the
// copying first one: at most 4, as radix 32 takes too many registers for
// enough waves (4096 points as 8 x 16 x 32: 3.9 ms on the case above).  2048 points
// end with radix 8, one butterfly per thread where the modes are stored (32768 LOS
// x 64 ch x 600 phi: 133 us as 8 x 16 x 16, 123 as 16 x 16 x 8).
template <int M>
struct Radices {
    static constexpr int count = M <= 4 ? 1 : M <= 8 ? 2 : M <= 12 ? 3 : 4;
    static constexpr int log2r(int i)
    {
        return count == 1 ? M : count == 2 ? (i == 0 ? M / 2 : M - M / 2)
               : M == 11 ? (i < 2 ? 4 : 3)
               : count == 3 ? (i == 0 ? M / 3 : i == 1 ? (M - M / 3) / 2 : M - M / 3 - (M - M / 3) / 2)
                            : (i < 3 ? 3 : M - 9);
    }
};

// Butterfly j of a Stockham pass of radix R on sub-transforms of length NS:
// inputs src(j, r) = element j + r n/R, twiddled by w^r, w = exp(-2 pi i k / (NS R)),
// k = j mod NS, then an R-point DFT.  The pass's table holds w^1, w^2, w^3, w^4,
// w^8, w^12 (those below R), NS values each, so that a wave reads neighbouring
// ones; the other powers are one product.
template <int R, int NS, class Src>
__device__ __forceinline__ void butterfly(float2* v, int j, const float2* __restrict__ tw, Src&& src)
{
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src(j, r);
    if constexpr (NS > 1) {
        const float2* const w = tw + (j & (NS - 1));
        float2 lo[4];
#pragma unroll
        for (int r = 1; r < (R < 4 ? R : 4); ++r) {
            lo[r] = w[(r - 1) * NS];
            v[r] = cmul(v[r], lo[r]);
        }
#pragma unroll
        for (int q = 4; q < R; q += 4) {
            const float2 hi = w[(2 + q / 4) * NS];
            v[q] = cmul(v[q], hi);
#pragma unroll
            for (int r = 1; r < 4; ++r) v[q + r] = cmul(v[q + r], cmul(hi, lo[r]));
        }
    }
    dft<R>(v);
}
constexpr int table_rows(int R) { return R <= 4 ? R - 1 : 2 + R / 4; }

// The passes from number I on, NS the sub-transform length reached.  The first
// pass reads src (the short grid, or the grid itself); all but the last write
// the grid; the last gives its modes to out(index, value).  The swizzle is
// linear over XOR and the bits of j and r (NS or n/R times) do not overlap: an
// element's place is that of j XOR a constant.
template <int LOGN, int B1, int T, int I, int NS, class Src, class Out>
__device__ __forceinline__ void fft_passes(float2* grid, const float2* __restrict__ tw, int t, Src&& src, Out&& out)
{
    using Rad = Radices<LOGN - B1>;
    constexpr int n = 1 << LOGN, R = 1 << Rad::log2r(I);
    constexpr int NB = (n / R + T - 1) / T;
    constexpr bool all = n / R % T == 0;
    if constexpr (I == Rad::count - 1) {
        static_assert(NS * R == n, "passes cover log2 n");
#pragma unroll 1
        for (int b = 0; b < NB; ++b) {
            const int j = t + T * b;
            if (all || j < n / R) {
                float2 v[R];
                butterfly<R, NS>(v, j, tw, src);
#pragma unroll
                for (int r = 0; r < R; ++r) out(j + r * NS, v[r]);
            }
        }
    } else {
        // The first pass of a short grid writes elsewhere than it reads.  Any
        // other is in place: every thread's reads finish before any write.
        constexpr bool in_place = !(I == 0 && B1 > 0);
        float2 v[NB][R];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int j = t + T * b;
            if (all || j < n / R) butterfly<R, NS>(v[b], j, tw, src);
        }
        if (in_place) __syncthreads();
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int j = t + T * b;
            if (all || j < n / R) {
                const int k = j & (NS - 1);
                const int base = swz((j - k) * R + k);
#pragma unroll
                for (int r = 0; r < R; ++r) grid[base ^ swz(r * NS)] = v[b][r];
            }
        }
        __syncthreads();
        constexpr int next = n >> Rad::log2r(I + 1);
        fft_passes<LOGN, B1, T, I + 1, NS * R>(
            grid, tw + (NS > 1 ? table_rows(R) * NS : 0), t,
            [grid](int j, int r) { return grid[swz(j) ^ swz(r * next)]; }, out);
    }
}

// One radix-8 butterfly per thread and pass up to 4096 points (16 points per
// thread: 2.76 against 2.64 ms on the case above).
constexpr int threads_per_los(int logn)
{
    return logn >= 12 ? 512 : logn <= 7 ? 16 : 1 << (logn - 3);
}

// Threads of a LOS with many channels on a small grid: one per point.  Its c_j
// leave little LDS for other LOS, and the lists take longer than the FFT.
constexpr int most_threads(int logn) { return logn >= 5 && logn <= 8 ? 1 << logn : threads_per_los(logn); }

// Threads that share a grid point's list.
constexpr int grid_parts(int logn, int b1)
{
    return b1 && threads_per_los(logn) > (1 << (logn - b1)) ? threads_per_los(logn) >> (logn - b1) : 1;
}

// float2 of LDS per LOS: the grid, with the c_j behind it, or in it where the
// short grid (behind both) is what gridding writes.
inline int64_t lds_points(int logn, int b1, int nchan)
{
    const int64_t n = int64_t(1) << logn;
    return b1 ? std::max<int64_t>(n, nchan) + (n >> b1) * grid_parts(logn, b1) : n + nchan;
}

template <int LOGN, int B1, int T>
__global__ __launch_bounds__(std::max(kThreads, T)) void nufft_kernel(
    const float* __restrict__ Q, const float* __restrict__ U, int64_t nlos, int nchan,
    const float2* __restrict__ rot, const int2* __restrict__ blk, const int2* __restrict__ ent,
    const float2* __restrict__ tw, const float2* __restrict__ deconv, int N, int kc, int per_los,
    float* __restrict__ Fq, float* __restrict__ Fu, float* __restrict__ Fabs)
{
    constexpr int n = 1 << LOGN, M = n >> B1;
    extern __shared__ float4 smem4[];
    const int t = threadIdx.x & (T - 1);
    // The LOS of the workgroup that this thread works on, the same over a wave
    // (and then known to be, for scalar addresses) when T is at least 64.
    int grp = threadIdx.x / T;
    if (T >= 64) grp = __builtin_amdgcn_readfirstlane(grp);
    const int64_t l = (int64_t)blockIdx.x * (blockDim.x / T) + grp;
    const bool valid = l < nlos;
    const int64_t lr = valid ? l : nlos - 1;  // spare groups redo the last LOS and store nothing
    float2* const grid = reinterpret_cast<float2*>(smem4) + grp * per_los;
    float2* const cb = B1 ? grid : grid + n;
    float2* const g = B1 ? grid + (per_los - M * grid_parts(LOGN, B1)) : grid;

    // Block p / 64 of grid points: its first entry and the entries per point (lists
    // shorter than the block's longest end in entries of weight 0; a multiple
    // of S).  S threads share a point's list where there are fewer points than
    // threads.  A thread's points are in NP blocks, the same ones over a wave.
    constexpr int S = grid_parts(LOGN, B1), NP = S == 1 ? (M + T - 1) / T : 1;
    static_assert(S == 1 || (B1 == 6 && kNufftListPad % S == 0), "whole shares of a list");
    const int wave = T > 64 ? __builtin_amdgcn_readfirstlane(t >> 6) : 0;
    int2 b[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int at = S == 1 ? (T * i >> 6) + wave : wave & ((M - 1) >> 6);
        b[i] = blk[M % T == 0 || at < (M + 63) / 64 ? at : 0];
    }
    // The first entries of a block are loaded a block ahead.
    constexpr int PRE = 4;
    int2 pre[PRE];
    auto load_first = [&](int i) __attribute__((always_inline)) {
        const int2* const e = ent + b[i].x + ((t + T * i) & 63);
#pragma unroll
        for (int q = 0; q < PRE; ++q)
            if (q < b[i].y) pre[q] = e[64 * q];
    };
    if (S == 1) load_first(0);

    // c_j = rot_j (Q_j + i U_j); flagged channels are in no gridding list.
    const float* q = Q + lr * nchan;
    const float* u = U + lr * nchan;
    for (int j = t; j < nchan; j += T) cb[j] = cmul(rot[j], make_float2(q[j], u[j]));
    __syncthreads();
    // Gridding: g_p = sum over the channels within reach of p of psi_jp c_j.
    auto add = [&](float2& acc, int2 en) __attribute__((always_inline)) {
        const float w = __int_as_float(en.y);
        const float2 c = cb[en.x];
        acc.x = __builtin_fmaf(w, c.x, acc.x);
        acc.y = __builtin_fmaf(w, c.y, acc.y);
    };
    auto sum_entries = [&](float2 acc, const int2* e, int count) __attribute__((always_inline)) {
        int i = 0;
        for (; i + 4 <= count; i += 4) {
            const int2 e0 = e[64 * i], e1 = e[64 * i + 64], e2 = e[64 * i + 128], e3 = e[64 * i + 192];
            add(acc, e0);
            add(acc, e1);
            add(acc, e2);
            add(acc, e3);
        }
        for (; i < count; ++i) add(acc, e[64 * i]);
        return acc;
    };
    if constexpr (S == 1) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            int2 cur[PRE];
#pragma unroll
            for (int q = 0; q < PRE; ++q) cur[q] = pre[q];
            if (i + 1 < NP) load_first(i + 1);
            float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
            for (int q = 0; q < PRE; ++q)
                if (q < b[i].y) add(acc, cur[q]);
            const int p = t + T * i;
            if (b[i].y > PRE) acc = sum_entries(acc, ent + b[i].x + 64 * PRE + (p & 63), b[i].y - PRE);
            if (M % T == 0 || p < M) {
                if (B1) g[p] = acc;
                else g[swz(p)] = acc;
            }
        }
    } else {
        const int p = t & (M - 1), part = t / M;
        const int each = b[0].y / S;
        g[t] = sum_entries(make_float2(0.0f, 0.0f), ent + b[0].x + 64 * each * part + (p & 63), each);
        __syncthreads();
        if (t < M) {
            float2 acc = g[t];
#pragma unroll
            for (int i = 1; i < S; ++i) acc = cadd(acc, g[t + i * M]);
            g[t] = acc;
        }
    }
    __syncthreads();

    // G_m = sum_p g_p exp(-2 pi i m p / n), F_k = deconv_k G_{(k - kc) mod n}.
    float* const fq = Fq + lr * N;
    float* const fu = Fu + lr * N;
    float* const fa = Fabs ? Fabs + lr * N : nullptr;
    constexpr int step = n >> Radices<LOGN - B1>::log2r(0);
    auto src = [g](int j, int r) { return B1 ? g[(j >> B1) + r * (step >> B1)] : g[swz(j) ^ swz(r * step)]; };
    auto at = [](auto* base, uint32_t k) -> decltype(auto) {  // base[k], 32-bit offset
        using E = std::remove_pointer_t<decltype(base)>;
        using C = std::conditional_t<std::is_const_v<E>, const char, char>;
        return *reinterpret_cast<E*>(reinterpret_cast<C*>(base) + (uint32_t)sizeof(E) * k);
    };
    auto out = [=](int m, float2 x) __attribute__((always_inline)) {
        const uint32_t k = (m + kc) & (n - 1);
        if (valid && k < (uint32_t)N) {
            const float2 d = at(deconv, k);
            if (B1) x = cmul(x, d);
            else x = make_float2(x.x * d.x, x.y * d.x);
            __builtin_nontemporal_store(x.x, &at(fq, k));
            __builtin_nontemporal_store(x.y, &at(fu, k));
            if (fa) at(fa, k) = sqrtf(x.x * x.x + x.y * x.y);
        }
    };
    fft_passes<LOGN, B1, T, 0, 1 << B1>(grid, tw, t, src, out);
}

template <int M>
void add_passes(int ns, std::vector<std::pair<int, int>>& out)
{
    for (int i = 0; i < Radices<M>::count; ++i) {
        out.push_back({1 << Radices<M>::log2r(i), ns});
        ns <<= Radices<M>::log2r(i);
    }
}

int log2_of(int n)
{
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

}  // namespace

std::vector<std::pair<int, int>> nufft_passes(int n, int b1)
{
    std::vector<std::pair<int, int>> v;
    switch (log2_of(n) - b1) {
        case 4: add_passes<4>(1 << b1, v); break;
        case 5: add_passes<5>(1 << b1, v); break;
        case 6: add_passes<6>(1 << b1, v); break;
        case 7: add_passes<7>(1 << b1, v); break;
        case 8: add_passes<8>(1 << b1, v); break;
        case 9: add_passes<9>(1 << b1, v); break;
        case 10: add_passes<10>(1 << b1, v); break;
        case 11: add_passes<11>(1 << b1, v); break;
        case 12: add_passes<12>(1 << b1, v); break;
        default: add_passes<13>(1 << b1, v); break;
    }
    return v;
}

size_t nufft_lds_bytes(const rmsynth_plan_s& p)
{
    return (size_t)lds_points(log2_of(p.nufft_n), p.nufft_b1, p.nchan) * sizeof(float2);
}

hipError_t launch_nufft(const rmsynth_plan_s& p, const float* Q, const float* U, int64_t nlos,
                        float* Fq, float* Fu, float* Fabs, hipStream_t s)
{
    const int logn = log2_of(p.nufft_n);
    const size_t each = nufft_lds_bytes(p);
    // LOS per workgroup: 256 threads' worth, within 40 KB of LDS (four
    // workgroups on a CU) unless one LOS alone takes more.
    const int64_t fit = std::max<int64_t>(1, (int64_t)(40960 / each));
    // Before and after, 32768 LOS of a band over half the circle: 64 phi (128 points),
    // 200 channels 82 -> 79 us, 800 434 -> 237, 4096 7620 -> 1535; fewer channels
    // lose (128: 51 -> 60).  128 phi, 400 138 -> 127 (300: 96 -> 105), 3000 2185 ->
    // 785; 32 phi, 300 107 -> 88 (200: 61 -> 65).  Larger grids fill the lanes as
    // they are.
    const bool many = p.nchan >= std::max(3 << logn >> 1, logn < 7 ? 256 : 0);
    const int T = many ? most_threads(logn) : threads_per_los(logn);
    const int64_t per = std::min<int64_t>(std::max(1, kThreads / T), fit);
    const int64_t max_los = max_items(per, per * T);
    for (int64_t l0 = 0; l0 < nlos;) {
        const int64_t n = std::min<int64_t>(nlos - l0, max_los);
        const float* q = Q + l0 * p.nchan;
        const float* u = U + l0 * p.nchan;
        float* fq = Fq + l0 * p.nphi;
        float* fu = Fu + l0 * p.nphi;
        float* fa = Fabs ? Fabs + l0 * p.nphi : nullptr;
#define RMS_NUFFT_T(L, B, TT)                                                                         \
    hipLaunchKernelGGL((nufft_kernel<L, B, TT>), dim3((unsigned)((n + per - 1) / per)),                     \
                       dim3((unsigned)(per * T)), (size_t)per * each, s, q, u, n, p.nchan, p.d_nufft_rot,  \
                       p.d_nufft_blk, p.d_nufft_ent, p.d_nufft_tw, p.d_nufft_deconv, p.nphi, p.nufft_kc,   \
                       (int)(each / sizeof(float2)), fq, fu, fa)
#define RMS_NUFFT(L, B)                                                \
    do {                                                               \
        if (T > threads_per_los(L)) RMS_NUFFT_T(L, B, most_threads(L)); \
        else RMS_NUFFT_T(L, B, threads_per_los(L));                    \
    } while (0)
#define RMS_NUFFT_3(L)                      \
    do {                                    \
        if (p.nufft_b1 == 3) RMS_NUFFT(L, 3); \
        else RMS_NUFFT(L, 0);               \
    } while (0)
#define RMS_NUFFT_6(L)                      \
    do {                                    \
        if (p.nufft_b1 == 6) RMS_NUFFT(L, 6); \
        else RMS_NUFFT_3(L);                \
    } while (0)
        switch (logn) {
            case 4: RMS_NUFFT(4, 0); break;
            case 5: RMS_NUFFT(5, 0); break;
            case 6: RMS_NUFFT(6, 0); break;
            case 7: RMS_NUFFT_3(7); break;
            case 8: RMS_NUFFT_3(8); break;
            case 9: RMS_NUFFT_3(9); break;
            case 10: RMS_NUFFT_6(10); break;
            case 11: RMS_NUFFT_6(11); break;
            case 12: RMS_NUFFT_6(12); break;
            case 13: RMS_NUFFT_6(13); break;
            default: return hipErrorInvalidValue;
        }
#undef RMS_NUFFT_6
#undef RMS_NUFFT_3
#undef RMS_NUFFT
#undef RMS_NUFFT_T
        if (hipError_t e = hipGetLastError()) return e;
        l0 += n;
    }
    return hipSuccess;
}
