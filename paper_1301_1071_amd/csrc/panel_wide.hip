// Panels wider than 128 columns (128 < n <= TSQR_NMAX), and the tree levels above n = 64: blocked
// Householder on panels of up to 2048 rows in global memory, one launch sequence for all panels of a
// tree level.
//
// Step 1 of direct TSQR (Sec. III-B) for panels too wide for one work-group's registers.  The
// columns are factored in blocks of 32 (16 for panels of more than 1024 rows), for every panel of
// the level at once:
//   * k_wide_block: one work-group per panel factors the block's columns, held in registers, with
//     the register-panel body (panel_blk_body.h) and leaves V (strictly below the diagonal) and the
//     block's compact-WY T (on and above it) in the block's place in the scratch panel, and R's
//     diagonal block in the stacked R;
//   * k_wide_update: one work-group per panel and 16 columns to the right applies
//     A <- (I - V T^T V^T) A: W = V^T A over the rows (each wave its row tiles, on the matrix cores),
//     summed over the waves in LDS, Y = T^T W, A -= V Y; the block's rows, now final, go to the
//     stacked R.  The strip of A stays in registers between the two products, so it is read and
//     written once per block.
// Q1 = H_1 ... H_n [I; 0] is formed from the last block to the first with the same update (T in
// place of T^T) on the columns from the block's first on, the block's own starting as identity columns.
//
// Why launches instead of one work-group per panel: a level has few panels (25 at 25,088 x 256, one
// at the top), and a panel's update is nearly all of its work, so the columns are what can be spread
// over the chip.  100,000 x 256 QR: 545 ms with the unblocked kernel, which walked a panel from L2
// once per column; 5.0 ms so (1.8 ms block factorizations, 1.2 ms updates, 1.4 ms forming Q1).  What
// bounds it: the column steps of a block (a chain as in the register panels: 33 to 54 us per block of
// 32 up to one panel a CU, 112 to 126 us at 391 panels, the first tree level of 1,000,000 x 100) and,
// in the updates, waves that wait for V and the strip before their products.  60,000 x 512 R: 8.5 ms.
//
// Rows past the panel's last row of input (short last panel) count as zero; V, W and A vanish there.
#include <algorithm>

#include "panel_blk_body.h"

namespace tsqr {
namespace {

using namespace blkpanel;

constexpr int kMaxWideRows = 2048;

// Shapes of the block factorization: rows up to NW RT 16, more than 16 (NCT - 1) and up to 16 NCT
// columns (Narrow: the last block of a width that leaves 16 or fewer)
template <int NCT_, int RT_, int NW_> struct WideShape {
    static constexpr int NCT = NCT_, RT = RT_, NW = NW_, B = NW_ * RT_ * 16;
};
using Shape512 = WideShape<2, 4, 8>;
using Shape1024 = WideShape<2, 8, 8>;
using Narrow512 = WideShape<1, 4, 8>;
using Narrow1024 = WideShape<1, 8, 8>;
using Shape2048 = WideShape<1, 16, 8>;      // panels of more than 1,024 rows (4 n, n > 256)

// One panel's rows and place: rows of input, scratch panel (row-major, ld n), stacked R
struct WidePanel {
    int bp;                 // rows of input
    size_t scratch;         // element offset of the scratch panel
};
__device__ __forceinline__ WidePanel wide_panel(int64_t rows, int b, int64_t pstride, int64_t p)
{
    return {(int)min((int64_t)b, rows - p * b), (size_t)(p * pstride)};
}

template <typename Tin, typename T, typename C>
__global__ void __launch_bounds__(C::NW * 64)
k_wide_block(int64_t rows, int n, int b, int j0, int nb, const Tin *X, int64_t ldx, T *gp,
             int64_t pstride, double *__restrict__ S)
{
    const int64_t p = blockIdx.x;
    const WidePanel wp = wide_panel(rows, b, pstride, p);
    T *P = gp + wp.scratch + (size_t)j0 * n + j0;
    double *Sp = S + (p * n + j0) * n;
    // left of the diagonal block R is zero
    for (int e = threadIdx.x; e < nb * j0; e += C::NW * 64) {
        const int r = e / j0;
        Sp[(int64_t)r * n + (e - r * j0)] = 0.0;
    }
    // the first block comes from the input, the others from the updated scratch panel
    const Tin *src = X ? X + p * b * ldx : (const Tin *)P;
    factor_blk_panel<Tin, T, C::NCT, C::RT, C::NW, PM_VT>(wp.bp - j0, nb, src, X ? ldx : n, P, n,
                                                          Sp + j0, n, 0);
}

// LDS of the update: per-wave products, their sum, T and Y (16 NV rows)
template <typename T, int NV, int NW> struct UpdSmem {
    T red[NW][NV][256];
    T w[NV][256];
    T t[16 * NV][16 * NV + 1];
    T y[16 * NV][17];
};

// FORMQ 0: columns c0 + 16 strip of the panel (from X while the scratch is not yet filled), 1: of
// Q1.  V: columns j0 .. j0 + nb, NV = ceil(nb / 16) tiles.  The 1-D grid keeps a panel's strips on
// one XCD (work-group b runs on XCD b % 8), whose L2 then serves V to all of them.
//
// Loads are issued ahead of the products and without per-element tests: rows past the panel and
// columns past nb stand in with other, finite elements, because A's rows there are zero in W = V^T A
// and not stored after A -= V Y, and T's rows there are zero; only V's top tiles (unit lower
// triangular, T above) are selected element by element.  Strips of 32 columns (V read half as often, but
// one work-group per CU instead of two) measured slower in all but the first of a level's launches.
template <typename Tin, typename T, int NV, int RT, int NW, bool FORMQ>
__global__ void __launch_bounds__(NW * 64)
k_wide_update(int64_t rows, int n, int b, int j0, int nb, int64_t panels, int strips, const Tin *X,
              int64_t ldx, T *gp, int64_t pstride, T *q1, double *__restrict__ S)
{
    using K = BlkT<T>;
    typedef typename K::acc_t acc_t;
    typedef T pair_t __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    __shared__ UpdSmem<T, NV, NW> sm;
    const int64_t bid = blockIdx.x;
    const int64_t grp = bid / (8 * strips);
    const int rem = (int)(bid - grp * 8 * strips);
    const int64_t p = grp * 8 + (rem & 7);
    if (p >= panels) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 15, lr = lane >> 4;
    const WidePanel wp = wide_panel(rows, b, pstride, p);
    const int c0 = (FORMQ ? j0 : j0 + nb) + 16 * (rem >> 3);      // first column of the strip
    const int c = c0 + lc, cc = min(c, n - 1);
    T *const Ps = gp + wp.scratch + (size_t)j0 * n;               // row j0 of the scratch panel
    const T *V = Ps + j0;                                         // the block's V
    const int nr = wp.bp - j0;                                    // rows that count
    const int lrow = K::rit(lr, 0);
    T *const qb = FORMQ ? q1 + (p * b + j0) * (int64_t)n : nullptr;

    // A: this wave's row tiles (tile g = rt NW + w); zero past the panel
    acc_t P[RT];
    auto fetch_a = [&](auto *src, int64_t ld) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int r0 = 16 * (rt * NW + w);
            if (r0 + 16 <= nr) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    P[rt][i] = (T)(src + (int64_t)(r0 + K::rit(0, i)) * ld)[lrow * ld + cc];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = r0 + K::rit(0, i) + lrow;
                    P[rt][i] = r < nr ? (T)src[r * ld + cc] : T(0);
                }
            }
        }
    };
    if constexpr (FORMQ) {
        if (c0 >= j0 + nb) {
            fetch_a(qb, n);
        } else {
            // the block's own columns start as identity columns (the last strip may go past them only
            // where the block is the last one)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 16 * (rt * NW + w) + K::rit(0, i) + lrow;
                    P[rt][i] = (r == c - j0 && r < nr) ? T(1) : T(0);
                }
        }
    } else {
        if (X) fetch_a(X + (p * b + j0) * ldx, ldx);
        else fetch_a(Ps, (int64_t)n);
    }
    for (int e = tid; e < 256 * NV * NV; e += NW * 64) {
        const int r = e / (16 * NV), k = e - r * 16 * NV;
        sm.t[r][k] = (r <= k && k < nb) ? V[(size_t)r * n + k] : T(0);
    }
    // V at (r, k) of the top tiles: unit lower triangular
    auto v_fix = [&](T v, int r, int k) { return r > k ? v : (r == k ? T(1) : T(0)); };
    // row r of V, or row 0 past the panel (a panel without rows here reads the block's top row)
    auto v_row = [&](int r) { return V + (int64_t)(r < nr ? r : 0) * n; };
    auto fetch_c = [&](int rt, T (&v)[NV][4]) {          // accumulator layout: element (row, lc)
        const int r0 = 16 * (rt * NW + w);
#pragma unroll
        for (int a = 0; a < NV; ++a) {
            const int k = 16 * a + lc < nb ? 16 * a + lc : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v[a][i] = r0 + 16 <= nr ? (V + (int64_t)(r0 + K::rit(0, i)) * n)[lrow * n + k]
                                        : v_row(r0 + K::rit(0, i) + lrow)[k];
        }
    };
    // W = V^T A over the rows
    acc_t acc[1][NV];
#pragma unroll
    for (int a = 0; a < NV; ++a) acc[0][a] = acc_t{0, 0, 0, 0};
    T vn[NV][4];
    fetch_c(0, vn);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        T v[NV][4];
#pragma unroll
        for (int a = 0; a < NV; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[a][i] = vn[a][i];
        if (rt + 1 < RT) fetch_c(rt + 1, vn);
        if (rt == 0 && w < NV) {
#pragma unroll
            for (int a = 0; a < NV; ++a)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[a][i] = v_fix(v[a][i], 16 * w + K::rit(0, i) + lrow, 16 * a + lc);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int a = 0; a < NV; ++a) acc[0][a] = K::mfma(v[a][i], P[rt][i], acc[0][a]);
    }
#pragma unroll
    for (int a = 0; a < NV; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) sm.red[w][a][K::rit(lr, i) * 16 + lc] = acc[0][a][i];
    // V's tiles in the row-major operand layout, pairs of columns (8 h + 2 lr and the next); with an odd
    // nb (the last block) the columns one by one
    const bool odd = (nb & 1) != 0;
    auto fetch_r = [&](int rt, T (&v)[4 * NV]) {
        const T *row = v_row(16 * (rt * NW + w) + lc);
#pragma unroll
        for (int h = 0; h < 2 * NV; ++h) {
            const int k = 8 * h + 2 * lr;
            if (!odd) {
                const pair_t x = *(const pair_t *)(row + (k < nb ? k : 0));
                v[2 * h] = x[0];
                v[2 * h + 1] = x[1];
            } else {
                v[2 * h] = row[k < nb ? k : 0];
                v[2 * h + 1] = row[k + 1 < nb ? k + 1 : 0];
            }
        }
    };
    T rn[4 * NV];
    fetch_r(0, rn);
    __syncthreads();
    for (int e = tid; e < NV * 256; e += NW * 64) {
        T s = T(0);
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) s += sm.red[ww][e >> 8][e & 255];
        sm.w[e >> 8][e & 255] = s;
    }
    __syncthreads();
    // -Y_a = -sum_k op(T)_{a k} W_k, one wave per tile a
    if (w < NV) {
        acc_t y = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int kk = 16 * k + 4 * q + lr;
                const T av = FORMQ ? sm.t[16 * w + lc][kk] : sm.t[kk][16 * w + lc];
                y = K::mfma(av, sm.w[k][(4 * q + lr) * 16 + lc], y);
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) sm.y[16 * w + K::rit(lr, i)][lc] = -y[i];
    }
    __syncthreads();
    T yb[4 * NV];                         // -Y at (8 h + 2 lr + e, lc): inner order of the pairs
#pragma unroll
    for (int q = 0; q < 4 * NV; ++q) yb[q] = sm.y[8 * (q >> 1) + 2 * lr + (q & 1)][lc];
    // A -= V Y
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        T a[4 * NV];
#pragma unroll
        for (int q = 0; q < 4 * NV; ++q) a[q] = rn[q];
        if (rt + 1 < RT) fetch_r(rt + 1, rn);
        if (rt == 0 && w < NV) {
#pragma unroll
            for (int q = 0; q < 4 * NV; ++q)
                a[q] = v_fix(a[q], 16 * w + lc, 8 * (q >> 1) + 2 * lr + (q & 1));
        }
#pragma unroll
        for (int q = 0; q < 4 * NV; ++q) P[rt] = K::mfma(a[q], yb[q], P[rt]);
    }
    auto store_a = [&](T *dst) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int r0 = 16 * (rt * NW + w);
            if (r0 + 16 <= nr) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c < n) (dst + (int64_t)(r0 + K::rit(0, i)) * n)[lrow * n + c] = P[rt][i];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = r0 + K::rit(0, i) + lrow;
                    if (r < nr && c < n) dst[(int64_t)r * n + c] = P[rt][i];
                }
            }
        }
    };
    if constexpr (FORMQ) {
        store_a(qb);
        // the rows above the block are zero in the block's own columns
        if (c0 < j0 + nb)
            for (int e = tid; e < 16 * min(j0, wp.bp); e += NW * 64) {
                const int r = e >> 4, k = c0 + (e & 15);
                if (k < j0 + nb) q1[(p * b + r) * (int64_t)n + k] = T(0);
            }
    } else {
        store_a(Ps);
        // the block's rows of R (zero past the panel's rows)
        if (w < NV) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * w + K::rit(0, i) + lrow;
                if (r < nb && c < n) S[(p * n + j0 + r) * n + c] = r < nr ? (double)P[0][i] : 0.0;
            }
        }
    }
}

template <typename Tin, typename T, typename C>
hipError_t wide_block(int64_t rows, int n, int b, int j0, int nb, const void *X, int64_t ldx,
                      void *gp, int64_t pstride, double *S, hipStream_t st)
{
    // every column tile holds columns, every row of the block fits: what the panel body assumes
    if (nb <= 16 * (C::NCT - 1) || nb > 16 * C::NCT || b - j0 > C::B) return hipErrorInvalidValue;
    constexpr size_t lds = sizeof(BlkSmem<T, C::NCT, C::NW>) + sizeof(BlkTail<T, C::NCT>);
    auto kern = k_wide_block<Tin, T, C>;
    hipError_t e = ensure_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(rows, b)), dim3(C::NW * 64), lds, st, rows, n, b,
                       j0, nb, (const Tin *)X, ldx, (T *)gp, pstride, S);
    return hipGetLastError();
}

template <typename Tin, typename T, int NV, int RT, bool FORMQ>
hipError_t wide_update_l(int64_t rows, int n, int b, int j0, int nb, const void *X, int64_t ldx,
                         void *gp, int64_t pstride, void *q1, double *S, hipStream_t st)
{
    constexpr int NW = 8;
    const int64_t panels = ceil_div(rows, b);
    const int strips = (int)ceil_div(n - (FORMQ ? j0 : j0 + nb), 16);
    if (strips == 0) return hipSuccess;
    hipLaunchKernelGGL((k_wide_update<Tin, T, NV, RT, NW, FORMQ>),
                       dim3((unsigned)(ceil_div(panels, 8) * 8 * strips)), dim3(NW * 64), 0, st, rows, n,
                       b, j0, nb, panels, strips, (const Tin *)X, ldx, (T *)gp, pstride, (T *)q1, S);
    return hipGetLastError();
}

// height: rows from the block's first on, of the tallest panel
template <typename Tin, typename T, bool FORMQ>
hipError_t wide_update(int height, int64_t rows, int n, int b, int j0, int nb, const void *X,
                       int64_t ldx, void *gp, int64_t pstride, void *q1, double *S, hipStream_t st)
{
#define TSQR_UPD(NV, RT)                                                                          \
    wide_update_l<Tin, T, NV, RT, FORMQ>(rows, n, b, j0, nb, X, ldx, gp, pstride, q1, S, st)
    if (nb > 16) return height <= 512 ? TSQR_UPD(2, 4) : TSQR_UPD(2, 8);
    return height <= 512 ? TSQR_UPD(1, 4) : height <= 1024 ? TSQR_UPD(1, 8) : TSQR_UPD(1, 16);
#undef TSQR_UPD
}

template <typename Tin, typename T>
hipError_t factor_wide(int64_t rows, int n, int b, const void *X, int64_t ldx, void *q1, double *S,
                       void *gp, int64_t pstride, hipStream_t st)
{
    const int width = b <= 1024 ? 32 : 16;
    for (int j0 = 0; j0 < n; j0 += width) {
        const int nb = std::min(width, n - j0);
        const int height = b - j0;
        const void *src = j0 == 0 ? X : nullptr;
        hipError_t e;
#define TSQR_BLK(SH)                                                                              \
    (j0 == 0 ? wide_block<Tin, T, SH>(rows, n, b, j0, nb, src, ldx, gp, pstride, S, st)                    \
             : wide_block<T, T, SH>(rows, n, b, j0, nb, src, ldx, gp, pstride, S, st))
        // (the first block is never narrow: n > 64)
#define TSQR_BLK_LAST(SH) wide_block<T, T, SH>(rows, n, b, j0, nb, nullptr, ldx, gp, pstride, S, st)
        if (b > 1024) e = TSQR_BLK(Shape2048);
        else if (nb <= 16) e = height > 512 ? TSQR_BLK_LAST(Narrow1024) : TSQR_BLK_LAST(Narrow512);
        else if (height > 512) e = TSQR_BLK(Shape1024);
        else e = TSQR_BLK(Shape512);
#undef TSQR_BLK_LAST
#undef TSQR_BLK
        if (e != hipSuccess) return e;
        e = j0 == 0 ? wide_update<Tin, T, false>(height, rows, n, b, j0, nb, src, ldx, gp, pstride, nullptr, S, st)
                    : wide_update<T, T, false>(height, rows, n, b, j0, nb, src, ldx, gp, pstride, nullptr, S, st);
        if (e != hipSuccess) return e;
    }
    if (!q1) return hipSuccess;
    for (int j0 = (n - 1) / width * width; j0 >= 0; j0 -= width) {
        const int nb = std::min(width, n - j0);
        hipError_t e = wide_update<T, T, true>(b - j0, rows, n, b, j0, nb, nullptr, 0, gp, pstride, q1, nullptr,
                                                st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

bool factor_wide_ok(int64_t n, int b) { return n > kNmaxPad && n <= kNmaxWide && b <= kMaxWideRows; }

hipError_t launch_factor_wide(int in_dtype, int dtype, int64_t rows, int64_t n, int b,
                              const void *X, int64_t ldx, void *q1, double *S, void *gpanel,
                              hipStream_t st)
{
    if (!factor_wide_ok(n, b) || b < n || !gpanel) return hipErrorInvalidValue;
    const int64_t ps = n * ((int64_t)b + 1);
    if (dtype == F64) {
        if (in_dtype != F64) return hipErrorInvalidValue;
        return factor_wide<double, double>(rows, (int)n, b, X, ldx, q1, S, gpanel, ps, st);
    }
    if (in_dtype == F64) return factor_wide<double, float>(rows, (int)n, b, X, ldx, q1, S, gpanel, ps, st);
    return factor_wide<float, float>(rows, (int)n, b, X, ldx, q1, S, gpanel, ps, st);
}

int wide_tree_rows(int64_t n) { return (int)(1024 / n * n); }

hipError_t launch_factor_wide_inplace(int64_t rows, int64_t n, int b, double *X, void *q1, double *S,
                                      hipStream_t st)
{
    // whole n-row blocks, so that no panel is shorter than n and T's rows stay inside it
    if (n <= 64 || n > kNmaxPad || rows % n || b % n || b < n || b > 1024) return hipErrorInvalidValue;
    return factor_wide<double, double>(rows, (int)n, b, X, n, q1, S, X, (int64_t)b * n, st);
}

}  // namespace tsqr
