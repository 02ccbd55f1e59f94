// Tall products with more than 64 inner columns on the matrix cores: out_p = Q1_p W_p (step 3 above
// n = 64), X W of the backward and of the chunked driver.  Same contract as the apply kernel for
// n <= 64 (apply_mfma.hip).
//
// Bound by the FP64 matrix cores (2 m n k operations at 12.5 flop/B and more) and, close behind, by
// HBM, so the design keeps the products fed: W_p's tiles sit in LDS in operand order, one 64-value
// record per 4 x 16 tile; a wave's 16 rows of Q1 come straight from memory in operand order, 16 bytes
// a lane (two inner columns), eight loads ahead of their products, across the ends of row blocks
// too.  As many output tiles as fit share one read of Q1 (eight waves on one W image of up to 150 KB):
// fewer tiles per wave leave the loads too little time (1,000,000 x 100 times 100 x 100: 0.65 ms so,
// 0.70 ms with four of seven tiles on two work-groups per CU, 0.79 ms with every block staged through
// LDS).
// A second operand pair (q1b and the next n rows of W) makes one product of X0 W0 + X1 W1, so that the
// backward writes its result once instead of reading it back.
#include <algorithm>

#include "tsqr_internal.h"

namespace tsqr {
namespace {

constexpr int kWaves = 8;
constexpr int kGroup = 8;                  // loads in flight: 8 pairs of inner columns per lane

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

template <typename T> struct MfmaW;
template <> struct MfmaW<double> {
    typedef d4_t acc_t;
    // pairs at 8-byte alignment: global loads need no more than that
    typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
    static __device__ __forceinline__ acc_t run(double a, double b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int i) { return (lane >> 4) + 4 * i; }
};
template <> struct MfmaW<float> {
    typedef f4_t acc_t;
    typedef float pair_t __attribute__((ext_vector_type(2), aligned(4)));
    static __device__ __forceinline__ acc_t run(float a, float b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int i) { return 4 * (lane >> 4) + i; }
};

// k-steps of the product: pairs of inner columns in groups of eight, step 2 h + e covers the inner
// columns 8 h + 2 q + e, q = 0..3 (any order serves as long as both operands use it)
inline int steps_of(int64_t n) { return 2 * (int)((n + 7) / 8); }
inline size_t wide_lds(size_t elem, int64_t n, int nsrc, int nt)
{
    return elem * (size_t)steps_of(n) * nsrc * nt * 64;
}

// One work-group per (panel, 16 NT-column slice y, row chunk rc); the 1-D grid keeps the slices of one
// panel on one XCD as in the narrow kernel.
template <typename T, typename To, int NT>
__global__ void __launch_bounds__(kWaves * 64)
k_apply_wide(int64_t rows, int n, int b, const T *q1, int64_t ldq, const T *q1b, int64_t ldqb,
             const double *__restrict__ W, int64_t ldw, int64_t wstride, int k,
             To *out0, int64_t ld0, int k0, To *out1, int64_t ld1,
             int64_t panels, int ny, int nrc)
{
    using M = MfmaW<T>;
    typedef typename M::acc_t acc_t;
    typedef typename M::pair_t pair_t;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *wl = reinterpret_cast<T *>(smem_raw);                  // [steps][NT][64]
    const int64_t bid = blockIdx.x;
    const int SL = ny * nrc;
    const int64_t grp = bid / (8 * SL);
    const int rem = (int)(bid - grp * 8 * SL);
    const int sl = rem >> 3;
    const int y = sl % ny, rc = sl / ny;
    const int64_t p = grp * 8 + (rem & 7);
    if (p >= panels) return;
    const int j0 = y * 16 * NT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 15, lr = lane >> 4;
    const double *Wp = W + p * wstride * ldw;
    const int64_t rb = p * (int64_t)b;
    const int nr = (int)min((int64_t)b, rows - rb);
    const int nblk = (nr + 15) >> 4;
    const int steps = 2 * ((n + 7) / 8), ng1 = (steps / 2 + kGroup - 1) / kGroup;
    const int ng = q1b ? 2 * ng1 : ng1;       // groups ng1.. belong to the second operand

    // this wave's row blocks b0, b0 + bstep, ...; (block, group) pairs in sequence, the next one's
    // loads issued before the current one's products
    const int b0 = w + kWaves * rc, bstep = kWaves * nrc;
    // pair h of row (block, lc): columns 8 h + 2 lr and the next; past column n - 1 zero, loaded
    // from columns n - 2, n - 1 instead
    auto fetch = [&](int blk, int g, pair_t (&a)[kGroup]) {
        const int r = min(blk * 16 + lc, nr - 1);
        const T *row = g < ng1 ? q1 + (rb + r) * ldq : q1b + (rb + r) * ldqb;
        if (g >= ng1) g -= ng1;
#pragma unroll
        for (int h = 0; h < kGroup; ++h) {
            const int c = 8 * (kGroup * g + h) + 2 * lr;
            a[h] = *(const pair_t *)(row + min(c, n - 2));
        }
    };
    auto fix = [&](int g, pair_t (&a)[kGroup]) {
        if (g >= ng1) g -= ng1;
        if (8 * kGroup * (g + 1) <= n) return;
#pragma unroll
        for (int h = 0; h < kGroup; ++h) {
            const int c = 8 * (kGroup * g + h) + 2 * lr;
            const T x0 = a[h][0], x1 = a[h][1];
            a[h][0] = (c + 1 < n) ? x0 : ((c + 1 == n) ? x1 : T(0));
            a[h][1] = (c + 1 < n) ? x1 : T(0);
        }
    };
    pair_t cur[kGroup], nxt[kGroup];
    if (b0 < nblk) fetch(b0, 0, nxt);
    {
        // W's loads twelve at a time from clamped in-bounds places, so that they are in flight together
        constexpr int U = 12;
        const int total = (q1b ? 2 : 1) * steps * NT * 64;
        for (int e0 = tid; e0 < total; e0 += U * kWaves * 64) {
            T v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = e0 + u * kWaves * 64;
                const int l = e & 63, t = e >> 6;
                const int nt = t % NT, s2 = t / NT, half = s2 >= steps ? 1 : 0, s = s2 - half * steps;
                const int kk = 8 * (s >> 1) + 2 * (l >> 4) + (s & 1), j = j0 + 16 * nt + (l & 15);
                const double x = Wp[(int64_t)(min(kk, n - 1) + (e < total ? half * n : 0)) * ldw + min(j, k - 1)];
                v[u] = (e < total && kk < n && j < k) ? (T)x : T(0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = e0 + u * kWaves * 64;
                if (e < total) wl[e] = v[u];
            }
        }
    }
    __syncthreads();
    const T *wk = wl + lane;
    const int jl = j0 + lc;
    for (int blk = b0; blk < nblk; blk += bstep) {
        acc_t acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = acc_t{0, 0, 0, 0};
        for (int g = 0; g < ng; ++g) {
#pragma unroll
            for (int h = 0; h < kGroup; ++h) cur[h] = nxt[h];
            if (g + 1 < ng) fetch(blk, g + 1, nxt);
            else if (blk + bstep < nblk) fetch(blk + bstep, 0, nxt);
            fix(g, cur);
            const int gl = g < ng1 ? g : g - ng1;
            const int hs = min(kGroup, steps / 2 - kGroup * gl);
            const T *ws = wk + (size_t)(2 * kGroup * gl + (g < ng1 ? 0 : steps)) * NT * 64;
            // each block of products ends with 20 wait states: an FP64 result may be read by the vector
            // unit 19 after its product, which the compiler does not keep where the two paths meet
            auto settle = [&] {
#pragma unroll
                for (int t = 0; t + 1 < NT; ++t) asm volatile("" : "+v"(acc[t]));
                asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[NT - 1]));
            };
            if (hs == kGroup) {
#pragma unroll
                for (int h = 0; h < kGroup; ++h)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[t] = M::run(cur[h][e], ws[((2 * h + e) * NT + t) * 64], acc[t]);
                settle();
            } else {
#pragma unroll
                for (int h = 0; h < kGroup; ++h)
                    if (h < hs) {
#pragma unroll
                        for (int e = 0; e < 2; ++e)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                acc[t] = M::run(cur[h][e], ws[((2 * h + e) * NT + t) * 64], acc[t]);
                        settle();
                    }
            }
        }
        // columns below k0 go to out0, the rest to out1 (shifted by k0)
        const int cnt = min(16, nr - blk * 16);
        To *const o0 = out0 + (rb + blk * 16) * ld0;
        To *const o1 = out1 ? out1 + (rb + blk * 16) * ld1 : o0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int j = jl + 16 * t;
            if (j >= k) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = M::row(lane, i);
                if (r >= cnt) continue;
                To *o = j < k0 ? o0 + r * ld0 + j : o1 + r * ld1 + (j - k0);
                *o = (To)acc[t][i];
            }
        }
    }
}

template <typename T, typename To, int NT>
hipError_t apply_wide_nt(int64_t rows, int64_t n, int b, const void *q1, int64_t ldq,
                         const void *q1b, int64_t ldqb, const double *W, int64_t ldw,
                         int64_t wstride, int k, void *out0, int64_t ld0, int k0, void *out1,
                         int64_t ld1, hipStream_t st)
{
    const size_t lds = wide_lds(sizeof(T), n, q1b ? 2 : 1, NT);
    auto kern = k_apply_wide<T, To, NT>;
    hipError_t e = ensure_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    const int64_t panels = ceil_div(rows, b);
    const int ny = (int)ceil_div(k, 16 * NT);
    // row chunks where there are few panels: about 512 work-groups (two rounds of the chip), at least
    // one row block a wave
    const int max_chunks = (int)ceil_div(ceil_div(b, 16), kWaves);
    const int64_t want = 512 / (panels * ny);
    const int nrc = (int)std::max<int64_t>(1, std::min<int64_t>(max_chunks, want));
    const int64_t blocks = ceil_div(panels, 8) * 8 * ny * nrc;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kWaves * 64), lds, st, rows, (int)n, b,
                       (const T *)q1, ldq, (const T *)q1b, ldqb, W, ldw, wstride, k, (To *)out0, ld0,
                       k0, (To *)out1, ld1, panels, ny, nrc);
    return hipGetLastError();
}

constexpr size_t kMaxLds = 160 * 1024, kWideLds = 150 * 1024;

template <typename T, typename To>
hipError_t apply_wide_t(int64_t rows, int64_t n, int b, const void *q1, int64_t ldq, const void *q1b,
                        int64_t ldqb, const double *W, int64_t ldw, int64_t wstride, int k, void *out0,
                        int64_t ld0, int k0, void *out1, int64_t ld1, hipStream_t st,
                        int one_slice)
{
    // Column slices per panel: as few as keep W's tiles within one work-group's LDS and eight
    // accumulator tiles (every slice reads Q1 again, from L2), and more where a launch has so few
    // panels that half the chip would be idle
    const int tiles = (int)ceil_div(k, 16), nsrc = q1b ? 2 : 1;
    int ny = 1;
    auto nt_of = [&](int s) { return (int)ceil_div(tiles, s); };
    if (one_slice) {
        if (nt_of(1) > 8 || wide_lds(sizeof(T), n, nsrc, nt_of(1)) > kMaxLds)
            return hipErrorInvalidValue;
    } else {
        while (ny < tiles && (nt_of(ny) > 8 || wide_lds(sizeof(T), n, nsrc, nt_of(ny)) > kWideLds)) ++ny;
        const int64_t groups = ceil_div(rows, b) * ceil_div(ceil_div(std::min<int64_t>(b, rows), 16), kWaves);
        while (ny < tiles && groups * ny < 128) ++ny;
    }
#define TSQR_NT(NT)                                                                               \
    case NT:                                                                                      \
        return apply_wide_nt<T, To, NT>(rows, n, b, q1, ldq, q1b, ldqb, W, ldw, wstride, k, out0, \
                                        ld0, k0, out1, ld1, st)
    switch (nt_of(ny)) {
        TSQR_NT(1);
        TSQR_NT(2);
        TSQR_NT(3);
        TSQR_NT(4);
        TSQR_NT(5);
        TSQR_NT(6);
        TSQR_NT(7);
        TSQR_NT(8);
    default: return hipErrorInvalidValue;
    }
#undef TSQR_NT
}

}  // namespace

hipError_t launch_apply_wide(int q_dtype, int out_dtype, int64_t rows, int64_t n, int b,
                             const void *q1, int64_t ldq, const double *W, int64_t ldw,
                             int64_t wstride, int k, void *out0, int64_t ld0, int k0, void *out1,
                             int64_t ld1, hipStream_t st, int one_slice)
{
    if (n < 2 || n > kNmaxWide) return hipErrorInvalidValue;
#define TSQR_ARGS                                                                                     \
    rows, n, b, q1, ldq, nullptr, 0, W, ldw, wstride, k, out0, ld0, k0, out1, ld1, st, one_slice
    if (q_dtype == F64)
        return out_dtype == F64 ? apply_wide_t<double, double>(TSQR_ARGS)
                                : apply_wide_t<double, float>(TSQR_ARGS);
    return out_dtype == F64 ? apply_wide_t<float, double>(TSQR_ARGS)
                            : apply_wide_t<float, float>(TSQR_ARGS);
#undef TSQR_ARGS
}

hipError_t launch_gemm2(int64_t rows, int64_t n, const double *X0, int64_t ldx0, const double *X1,
                        int64_t ldx1, const double *W, double *out, int64_t ldo, hipStream_t st)
{
    if (n < 1 || n > kNmaxPad) return hipErrorInvalidValue;
    // 512 to 2,048 rows per work-group, 512 to 1,024 work-groups where there are that many rows (W is
    // the same for all of them)
    const int b = (int)std::min<int64_t>(2048, std::max<int64_t>(128, ceil_div(ceil_div(rows, 768), 128) * 128));
    if (n == 1) {      // the pair loads need two columns
        hipError_t e = launch_gemm_mfma(F64, F64, rows, 1, b, X0, ldx0, W, 1, 0, 1, out, ldo, 1, nullptr,
                                        0, 0, st);
        if (e != hipSuccess || !X1) return e;
        return launch_gemm_mfma(F64, F64, rows, 1, b, X1, ldx1, W + 1, 1, 0, 1, out, ldo, 1, nullptr, 0, 1,
                                st);
    }
    return apply_wide_t<double, double>(rows, n, b, X0, ldx0, X1, ldx1, W, n, 0, (int)n, out, ldo, (int)n,
                                        nullptr, 0, st, 0);
}

}  // namespace tsqr
