// Top of the tree (one work-group): sign normalisation of R~, the info flag, and the SVD of R.
//
// Sec. III-B: the single reduce task ends with R~; the factorization with a positive diagonal is
// unique for full-rank A (Sec. I), so R = D R~ with D = diag(sign(R~_jj)), sign(0) = +1, and the
// step-3 blocks become Q2_p D.  For the SVD variant the reduce task also computes R = U_R S V^T
// (the paper treats this n x n SVD as negligible and names no method): one-sided Jacobi
// (Hestenes) on R^T, columns rotated until pairwise orthogonal, in parallel round-robin order.
// U_R is passed down the tree so that U = Q U_R comes out of step 3 in the same pass as Q.
//
// Up to n = 100 the columns of G and J sit in one work-group's LDS.  Wider, they sit in global
// scratch and the rotations run block by block (k_jacobi_block): the columns are cut into blocks, one
// work-group rotates the columns of one pair of blocks in its LDS, and a round-robin over the block
// pairs, one launch per round, makes a sweep.
#include <algorithm>
#include <type_traits>

#include "tsqr_internal.h"

namespace tsqr {
namespace {

constexpr size_t kLdsPerWorkgroup = 160 * 1024;   // LDS one work-group may hold on gfx950

// player at position `pos` of round `r` in the round-robin tournament of np players
// (0 <= pos < np, 0 <= r < np - 1): player 0 stays, the others rotate by one place per round.
// pos - 1 + r < 2 (np - 1), so one conditional subtraction is the reduction modulo np - 1.
__device__ __forceinline__ int rr_player(int pos, int r, int np)
{
    int x = pos - 1 + r;
    if (x >= np - 1) x -= np - 1;
    return pos == 0 ? 0 : 1 + x;
}

// reciprocal square root: hardware estimate plus two Newton steps (a few ulp)
__device__ __forceinline__ double rsqrt_nr(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = y * fma(-0.5 * x * y, y, 1.5);
    return y * fma(-0.5 * x * y, y, 1.5);
}

constexpr int kSvdThreads = 1024;   // 16 waves: 64 groups of 16 lanes, one column pair each

// DPP lane move; the patterns used here (quad_perm, row_ror, row_newbcast) read a valid lane for
// every lane, so the old value is never used and needs no zeroing (bound_ctrl)
template <int CTRL> __device__ __forceinline__ double dpp_d(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Sum over the 16 lanes of a group (one DPP row): butterflies within quads, rotations by 4 and 8
// across the quads, then lane 0's sum broadcast to the row so every lane of the group takes the
// same rotation decision.
__device__ __forceinline__ double group16_sum(double v)
{
    v += dpp_d<0xB1>(v);          // quad_perm [1,0,3,2]
    v += dpp_d<0x4E>(v);          // quad_perm [2,3,0,1]
    v += dpp_d<0x124>(v);         // row_ror:4
    v += dpp_d<0x128>(v);         // row_ror:8
    return dpp_d<0x150>(v);       // row_newbcast:0
}

typedef double d2_t __attribute__((ext_vector_type(2)));

// v summed over the 64 lanes of a wave (every lane gets the same sum)
__device__ __forceinline__ double wave64_sum(double v)
{
    v = group16_sum(v);
    const auto l1 = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h1 = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(h1[0], l1[0]) + __hiloint2double(h1[1], l1[1]);
    const auto l2 = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h2 = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(h2[0], l2[0]) + __hiloint2double(h2[1], l2[1]);
}

// cos^2 + sin^2 brought to 1: the rotations of a column multiply, so a common bias of their lengths
// would add up in J and in the singular values (|J^T J - I| at 4,000 x 50, Gaussian: 1.4e-14
// without, 5e-15 with)
__device__ __forceinline__ void unit_rotation(double c, double s, double &cs, double &sn)
{
    const double e = 0.5 * fma(-s, s, fma(-c, c, 1.0));
    cs = fma(c, e, c);
    sn = fma(s, e, s);
}

// Squared column norms between which the angle can be formed unscaled: products of two of them, which
// are fourth powers of the entries, then keep clear of both ends of the range of FP64, also after the
// rotations of a sweep have brought one down to the rounding error of another.  Zero counts as inside.
__device__ __forceinline__ bool far_norm(double ss) { return ss != 0.0 && !(ss > 1e-80 && ss < 1e140); }

// The rotation (cs, sn; rc = 1 / cos) that makes two columns orthogonal, from their squared norms al,
// be and dot product ga; false where they are orthogonal to the tolerance already.  FAR: the
// norms may lie far out, so the three are scaled by the power of two that brings the largest to 2^500
// (exact: the same bits where both forms stay in range), which holds for norms up to 1e290 apart.
// |ga| is among them because a tracked norm may have become 0.  Scaling every pair cost 2% of the SVD
// of 60,000 x 40 and its gradient and 2.6% of the SVD of 8,000 x 160, a branch in the step as much at
// n = 40; so the rounds exist twice.
template <bool FAR>
__device__ __forceinline__ bool jacobi_angle(double al, double be, double ga, double tol2, double &cs,
                                             double &sn, double &rc)
{
    if constexpr (FAR) {
        const int e = 500 - __builtin_amdgcn_frexp_exp(fmax(fmax(al, be), __builtin_fabs(ga)));
        al = ldexp(al, e);
        be = ldexp(be, e);
        ga = ldexp(ga, e);
    }
    if (!(ga != 0.0 && ga * ga > tol2 * (al * be))) return false;
    // tan 2 theta = 2 ga / (be - al): with h = hypot(d, g2), cos^2 = (1 + |d| / h) / 2 and
    // sin = g2 sign(d) / (2 h cos); cos >= 1/sqrt(2), so neither cancels
    const double d = be - al, g2 = 2.0 * ga;
    const double rh = rsqrt_nr(fma(d, d, g2 * g2));
    const double c2 = fma(0.5 * __builtin_fabs(d), rh, 0.5);
    rc = rsqrt_nr(c2);
    unit_rotation(c2 * rc, 0.5 * g2 * rh * rc, cs, sn);
    if (d < 0.0) sn = -sn;
    return true;
}

// One rotation of the columns p, q of G and V (LDS, even ld, a zero row below an odd n) by LANES
// lanes (16 or 64; lane gl holds the row pairs gl + LANES j).  nrm holds the squared norms of the
// columns: the rotation changes them by -+ t g_p . g_q, so only g_p . g_q is summed here; they are
// formed afresh before every sweep.  Returns whether the pair was rotated (the same in all lanes).
//
// Bound by instruction issue (all pairs of a round share one CU, 2 to 4 waves per SIMD): hence one
// dot instead of three, 16-byte accesses, and the angle by two reciprocal square roots.
template <int LANES, int NC, bool FAR>
__device__ __forceinline__ bool rotate_pair(double *gp, double *gq, double *vp, double *vq, int ld,
                                            int gl, double *np_, double *nq_, double tol2)
{
    d2_t x[NC], y[NC];
    double g0 = 0.0, g1 = 0.0;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int r = 2 * (gl + LANES * j);
        const int rc = (j + 1 < NC) ? r : min(r, ld - 2);       // only the last chunk can overhang
        x[j] = *(const d2_t *)(gp + rc);
        y[j] = *(const d2_t *)(gq + rc);
    }
    const double al = *np_, be = *nq_;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const bool in = (j + 1 < NC) || 2 * (gl + LANES * j) < ld;
        const double x0 = in ? x[j][0] : 0.0, x1 = in ? x[j][1] : 0.0;
        g0 = fma(x0, y[j][0], g0);
        g1 = fma(x1, y[j][1], g1);
    }
    const double ga = LANES == 16 ? group16_sum(g0 + g1) : wave64_sum(g0 + g1);
    double cs, sn, rc;
    if (!jacobi_angle<FAR>(al, be, ga, tol2, cs, sn, rc)) return false;
    d2_t u[NC], v[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int r = 2 * (gl + LANES * j);
        const int rc2 = (j + 1 < NC) ? r : min(r, ld - 2);
        u[j] = *(const d2_t *)(vp + rc2);
        v[j] = *(const d2_t *)(vq + rc2);
    }
    if (gl == 0) {
        const double dt = sn * rc * ga;                          // t ga
        *np_ = fmax(al - dt, 0.0);
        *nq_ = fmax(be + dt, 0.0);
    }
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int r = 2 * (gl + LANES * j);
        if ((j + 1 < NC) || r < ld) {
            *(d2_t *)(gp + r) = cs * x[j] - sn * y[j];
            *(d2_t *)(gq + r) = sn * x[j] + cs * y[j];
            *(d2_t *)(vp + r) = cs * u[j] - sn * v[j];
            *(d2_t *)(vq + r) = sn * u[j] + cs * v[j];
        }
    }
    return true;
}

constexpr int kMaxSweeps = 60;
// Largest cosine of two columns left by the sweeps, per column: a tenth below 1e-15, so that V is
// orthogonal to 1e-15 n also after its own rounding
constexpr double kJacobiTol = 0.9e-15;

// NPAD: column capacity.  LDSM: the Jacobi columns live in LDS (known at compile time, so that
// their accesses are LDS instructions, not flat ones that could reach either memory); else in the
// global scratch G, Vw, where k_jacobi_block has already run `first` sweeps and rot tells whether
// the last of them still rotated (the sweeps left are run here, a column pair at a time).
template <int NPAD, bool LDSM>
__global__ void __launch_bounds__(kSvdThreads)
k_finalize(int n, const double *__restrict__ Rt, double *__restrict__ R, float *__restrict__ Rf,
           int64_t ldr, double *__restrict__ Wtop, int k, int want_q, int want_u,
           double *S, float *Sf, double *__restrict__ V,
           float *__restrict__ Vf, int64_t ldv, double *G, double *Vw,
           int32_t *__restrict__ info, int keep_info, int first, const int32_t *rot)
{
    extern __shared__ __align__(16) double sm[];
    __shared__ double d_s[NPAD];
    __shared__ double s_sv[NPAD];
    __shared__ double s_sg[NPAD];
    __shared__ int perm[NPAD];
    __shared__ int s_zero, s_nonfinite, s_rot, s_far;

    const int tid = threadIdx.x;
    const int nth = blockDim.x;

    if (tid == 0) { s_zero = 0x7fffffff; s_nonfinite = 0; s_far = 0; }
    __syncthreads();
    for (int i = tid; i < n; i += nth) {
        const double rii = Rt[(int64_t)i * n + i];
        d_s[i] = (rii >= 0.0) ? 1.0 : -1.0;
        if (rii == 0.0) atomicMin(&s_zero, i);
    }
    for (int e = tid; e < n * n; e += nth) {
        const int r = e / n, c = e - r * n;
        if (c >= r && !isfinite(Rt[e])) s_nonfinite = 1;
    }
    __syncthreads();
    for (int e = tid; e < n * n; e += nth) {
        const int r = e / n, c = e - r * n;
        const double v = (c >= r) ? d_s[r] * Rt[e] : 0.0;
        if (R) R[(int64_t)r * ldr + c] = v;
        if (Rf) Rf[(int64_t)r * ldr + c] = (float)v;
        if (want_q) Wtop[(int64_t)r * k + c] = (r == c) ? d_s[r] : 0.0;
    }
    const int kq = want_q ? n : 0;

    if (want_u || S != nullptr || Sf != nullptr) {
        const int ld = LDSM ? n + (n & 1) : n;
        double *gG = LDSM ? sm : G;                        // column-major
        double *gV = LDSM ? sm + (size_t)n * ld : Vw;
        const int grp = tid >> 4, gl = tid & 15;           // 16-lane group and lane within it
        const int ngrp = nth >> 4;
        const double tol = kJacobiTol * (double)n;
        const double tol2 = tol * tol;
        const int np = n + (n & 1);                        // players of the round-robin tournament
        const int npairs = np / 2;
        // one-sided Jacobi on R^T (column r of R^T is row r of R): R^T J = G with orthogonal
        // columns, so R = J diag(|g|) (G diag(|g|)^{-1})^T, i.e. U_R = J and V = G / |g|.
        // Rotating the rows of the triangular R converges in far fewer sweeps than rotating its
        // columns when R is ill conditioned.
        if constexpr (LDSM) {
            for (int e = tid; e < n * ld; e += nth) {
                const int r = e / ld, c = e - r * ld;
                gG[e] = (c >= r && c < n) ? d_s[r] * Rt[(int64_t)r * n + c] : 0.0;
                gV[e] = (r == c) ? 1.0 : 0.0;
            }
            for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
                __syncthreads();
                if (tid == 0) s_rot = 0;
                for (int c = grp; c < n; c += ngrp) {
                    double ss = 0.0;
                    for (int i = gl; i < n; i += 16) ss = fma(gG[c * ld + i], gG[c * ld + i], ss);
                    ss = group16_sum(ss);
                    if (gl == 0) {
                        s_sv[c] = ss;
                        if (far_norm(ss)) s_far = 1;       // stays set: the next sweeps scale too
                    }
                }
                __syncthreads();
                const bool far = __builtin_amdgcn_readfirstlane(s_far) != 0;
                bool any = false;
                auto rounds = [&](auto FAR) {
                    // round 0 pairs position grp with np - 1 - grp; from round to round every player
                    // but number 0 moves up by one
                    int ia = grp, ib = np - 1 - grp;
                    for (int round = 0; round < np - 1; ++round) {
                        if (grp < npairs && ia < n && ib < n)
                            any |= rotate_pair<16, NPAD / 32, decltype(FAR)::value>(
                                gG + ia * ld, gG + ib * ld, gV + ia * ld, gV + ib * ld, ld, gl, &s_sv[ia],
                                &s_sv[ib], tol2);
                        if (grp > 0) ia = ia + 1 == np ? 1 : ia + 1;
                        ib = ib + 1 == np ? 1 : ib + 1;
                        __syncthreads();
                    }
                };
                if (far) rounds(std::true_type{});
                else rounds(std::false_type{});
                if (any && gl == 0) s_rot = 1;             // every writer stores the same value
                __syncthreads();
                if (s_rot == 0) break;
            }
        } else if (rot[0] != 0) {
            for (int sweep = first; sweep < kMaxSweeps; ++sweep) {
                __syncthreads();
                if (tid == 0) s_rot = 0;
                __syncthreads();
                for (int round = 0; round < np - 1; ++round) {
                    for (int t = grp; t < npairs; t += ngrp) {      // uniform within each group
                        const int a = rr_player(t, round, np), bq = rr_player(np - 1 - t, round, np);
                        if (a >= n || bq >= n) continue;
                        double *gp = gG + (int64_t)a * n, *gq = gG + (int64_t)bq * n;
                        double *vp = gV + (int64_t)a * n, *vq = gV + (int64_t)bq * n;
                        double al = 0.0, be = 0.0, ga = 0.0;
                        for (int i = gl; i < n; i += 16) {
                            al = fma(gp[i], gp[i], al);
                            be = fma(gq[i], gq[i], be);
                            ga = fma(gp[i], gq[i], ga);
                        }
                        al = group16_sum(al);
                        be = group16_sum(be);
                        ga = group16_sum(ga);
                        double cs, sn, rc;
                        if (!jacobi_angle<true>(al, be, ga, tol2, cs, sn, rc)) continue;
                        for (int i = gl; i < n; i += 16) {
                            const double x = gp[i], y = gq[i], u = vp[i], v = vq[i];
                            gp[i] = cs * x - sn * y;
                            gq[i] = sn * x + cs * y;
                            vp[i] = cs * u - sn * v;
                            vq[i] = sn * u + cs * v;
                        }
                        if (gl == 0) s_rot = 1;
                    }
                    __syncthreads();
                }
                if (s_rot == 0) break;
            }
        }
        __syncthreads();
        // singular values; gauge: the largest-magnitude entry of each v_k = g_k / |g_k| is
        // positive (lowest index on ties).  One 16-lane group per column
        for (int c = grp; c < n; c += ngrp) {
            double ss = 0.0, vmax = -1.0;
            int imax = 0;
            for (int i = gl; i < n; i += 16) {
                const double g = gG[(int64_t)c * ld + i], a = fabs(g);
                ss = fma(g, g, ss);
                if (a > vmax) { vmax = a; imax = i; }
            }
            ss = group16_sum(ss);
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                const double ov = __shfl_xor(vmax, off, 64);
                const int oi = __shfl_xor(imax, off, 64);
                if (ov > vmax || (ov == vmax && oi < imax)) { vmax = ov; imax = oi; }
            }
            if (gl == 0) {
                s_sv[c] = sqrt(ss);
                s_sg[c] = (gG[(int64_t)c * ld + imax] < 0.0) ? -1.0 : 1.0;
            }
        }
        __syncthreads();
        // descending, the lower index first on ties, a NaN (non-finite input) behind every number: a
        // total order, so that perm is a permutation of the columns whatever the values
        for (int c = tid; c < n; c += nth) {
            auto key = [&](int j) { return s_sv[j] == s_sv[j] ? s_sv[j] : -1.0; };
            const double kc = key(c);
            int rank = 0;
            for (int j = 0; j < n; ++j) {
                const double kj = key(j);
                rank += (kj > kc) || (kj == kc && j < c);
            }
            perm[rank] = c;
        }
        __syncthreads();
        for (int o = tid; o < n; o += nth) {
            if (S) S[o] = s_sv[perm[o]];
            if (Sf) Sf[o] = (float)s_sv[perm[o]];
        }
        for (int e = tid; e < n * n; e += nth) {
            const int i = e / n, o = e - i * n;
            const int c = perm[o];
            const double s = s_sv[c];
            const double vio = (s > 0.0) ? s_sg[c] * gG[(int64_t)c * ld + i] / s : 0.0;
            if (V) V[(int64_t)i * ldv + o] = vio;
            if (Vf) Vf[(int64_t)i * ldv + o] = (float)vio;
            if (want_u) Wtop[(int64_t)i * k + kq + o] = d_s[i] * s_sg[c] * gV[(int64_t)c * ld + i];
        }
    }
    if (tid == 0) {
        const int32_t code = s_nonfinite ? -1 : (s_zero == 0x7fffffff ? 0 : s_zero + 1);
        // keep_info: an earlier kernel of the call may already have reported a condition
        if (!keep_info || *info == 0) *info = code;
    }
}

// Start of the block sweeps: G = R^T (column r is row r of R = D R~), J = I, the sweeps' flags 0.
__global__ void __launch_bounds__(256)
k_jacobi_init(int n, const double *__restrict__ Rt, double *__restrict__ G, double *__restrict__ Vw,
              int32_t *__restrict__ flags, int nflags)
{
    const int r = blockIdx.x;
    const double d = (Rt[(int64_t)r * n + r] >= 0.0) ? 1.0 : -1.0;
    for (int c = threadIdx.x; c < n; c += 256) {
        G[(int64_t)r * n + c] = (c >= r) ? d * Rt[(int64_t)r * n + c] : 0.0;
        Vw[(int64_t)r * n + c] = (r == c) ? 1.0 : 0.0;
    }
    if (r == 0 && (int)threadIdx.x < nflags) flags[threadIdx.x] = 0;
}

// One round of a block sweep: work-group t holds the columns of the block pair (W columns each) of
// the round-robin position t in LDS, one wave per column pair.  In a sweep's round 0 all pairs of its
// 2 W columns are rotated, in the others the W x W cross pairs.  flags[sweep] is set when a pair was
// rotated; nothing is done once a sweep has passed without.
template <int NC>
__global__ void __launch_bounds__(1024)
k_jacobi_block(int n, int W, int nblk, int round, int sweep, double *__restrict__ G,
               double *__restrict__ Vw, int32_t *flags)
{
    extern __shared__ __align__(16) double sm[];
    __shared__ double s_nrm[32];
    __shared__ int s_rot, s_far;
    if (sweep > 0 && flags[sweep - 1] == 0) return;
    const int nbp = nblk + (nblk & 1);
    const int t = blockIdx.x;
    const int b0 = rr_player(t, round, nbp), b1 = rr_player(nbp - 1 - t, round, nbp);
    const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ld = n + (n & 1), nc = 2 * W;
    double *gG = sm, *gV = sm + (size_t)nc * ld;
    // global column of local column l (n or more: none)
    auto col = [&](int l) {
        const int b = l < W ? b0 : b1;
        return b < nblk ? b * W + (l < W ? l : l - W) : n;
    };
    if (tid == 0) { s_rot = 0; s_far = 0; }
    __syncthreads();
    for (int l = w; l < nc; l += nth >> 6) {
        const int c = col(l);
        if (c >= n) continue;
        double ss = 0.0;
        for (int i = lane; i < ld; i += 64) {
            const double g = i < n ? G[(int64_t)c * n + i] : 0.0;
            gG[l * ld + i] = g;
            gV[l * ld + i] = i < n ? Vw[(int64_t)c * n + i] : 0.0;
            ss = fma(g, g, ss);
        }
        ss = wave64_sum(ss);
        if (lane == 0) {
            s_nrm[l] = ss;
            if (far_norm(ss)) s_far = 1;
        }
    }
    __syncthreads();
    const bool far = __builtin_amdgcn_readfirstlane(s_far) != 0;
    const double tol = kJacobiTol * (double)n;
    const bool full = round == 0;
    bool any = false;
    auto rounds = [&](auto FAR) {
        for (int r = 0; r < (full ? nc - 1 : W); ++r) {
            int p, q;
            if (full) {
                p = rr_player(w, r, nc);
                q = rr_player(nc - 1 - w, r, nc);
            } else {
                p = w;
                q = W + (w + r >= W ? w + r - W : w + r);
            }
            if (col(p) < n && col(q) < n)
                any |= rotate_pair<64, NC, decltype(FAR)::value>(gG + p * ld, gG + q * ld, gV + p * ld,
                                                                 gV + q * ld, ld, lane, &s_nrm[p],
                                                                 &s_nrm[q], tol * tol);
            __syncthreads();
        }
    };
    if (far) rounds(std::true_type{});
    else rounds(std::false_type{});
    if (any && lane == 0) s_rot = 1;
    __syncthreads();
    if (s_rot == 0) return;
    if (tid == 0) flags[sweep] = 1;
    for (int l = w; l < nc; l += nth >> 6) {
        const int c = col(l);
        if (c >= n) continue;
        for (int i = lane; i < n; i += 64) {
            G[(int64_t)c * n + i] = gG[l * ld + i];
            Vw[(int64_t)c * n + i] = gV[l * ld + i];
        }
    }
}

// Sweeps run by the block kernel before k_finalize takes over (which finishes what has not
// converged by then, up to kMaxSweeps): the graded and Gaussian triangles of the tests need 7 to 11.
// All their rounds are enqueued, whatever the matrix needs (no host read, so that a call can be
// captured): 112 launches at n = 101, 144 at 160, 304 at 300, 592 at 301, 1,008 at 512, as many graph
// nodes, and 0.5, 0.6, 1.3, 2.6 and 3.2 ms of host time in calls of 2.2, 3.6, 10.1, 9.7 and 22 ms on
// 2,000 rows.  At 8,000 x 160 a working round takes 31 us (a sweep's first 54), one after convergence 2.3.
constexpr int kBlockSweeps = 16;

hipError_t launch_jacobi_blocks(int n, const double *Rt, double *G, double *Vw, int32_t *flags,
                                hipStream_t st)
{
    // W columns per block: 16, or 8 where 32 columns of G and J no longer fit in LDS
    const int ld = n + (n & 1);
    const int W = sizeof(double) * 64 * (size_t)ld <= 150 * 1024 ? 16 : 8;
    const size_t lds = sizeof(double) * 4 * W * (size_t)ld;
    const int nblk = (n + W - 1) / W, nbp = nblk + (nblk & 1);
    // NC: chunks of 64 row pairs, so that only the last one can overhang the columns
    auto kern = ld <= 128 ? k_jacobi_block<1> : ld <= 256 ? k_jacobi_block<2>
                : ld <= 384 ? k_jacobi_block<3> : k_jacobi_block<4>;
    hipError_t e = ensure_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_jacobi_init, dim3((unsigned)n), dim3(256), 0, st, n, Rt, G, Vw, flags,
                       kBlockSweeps);
    for (int s = 0; s < kBlockSweeps; ++s)
        for (int r = 0; r < nbp - 1; ++r)
            hipLaunchKernelGGL(kern, dim3((unsigned)(nbp / 2)), dim3(64 * W), lds, st, n, W, nblk, r, s,
                               G, Vw, flags);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_finalize(int64_t n, const double *Rt, double *R, float *Rf, int64_t ldr,
                           double *Wtop, int k, int want_q, int want_u, double *S, float *Sf,
                           double *V, float *Vf, int64_t ldv, double *G, double *Vw,
                           int32_t *info, hipStream_t st, int keep_info)
{
    const bool svd = want_u || S != nullptr || Sf != nullptr;
    if (n > kNmaxWide) return hipErrorInvalidValue;
    // the Jacobi columns (G and J, 2 n^2 doubles) go to LDS when they fit beside the kernel's
    // static arrays (up to n = 100), else to global scratch
    const size_t need = svd ? 2 * sizeof(double) * (size_t)n * (n + (n & 1)) : 0;
    bool use_lds = false;
    auto lds_kern = (n > 96) ? k_finalize<kNmaxPad, true>
                    : (n > 64) ? k_finalize<96, true>
                    : (n > 32) ? k_finalize<64, true> : k_finalize<32, true>;
    if (svd && n <= kNmaxPad) {
        hipFuncAttributes fa;
        hipError_t e = hipFuncGetAttributes(&fa, (const void *)lds_kern);
        if (e != hipSuccess) return e;
        use_lds = need + align_up(fa.sharedSizeBytes, 16) <= kLdsPerWorkgroup;
    }
    const size_t lds = use_lds ? need : 0;
    auto kern = use_lds ? lds_kern
                : (n > kNmaxPad) ? k_finalize<kNmaxWide, false>
                : (n > 64) ? k_finalize<kNmaxPad, false> : k_finalize<64, false>;
    hipError_t e = ensure_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    // the sweeps' flags: the singular values' place in the caller's S (at least n values of four
    // bytes, n > 100 here), which is written last
    int32_t *flags = S ? (int32_t *)S : (int32_t *)Sf;
    if (svd && !use_lds) {
        if (!flags) return hipErrorInvalidValue;
        e = launch_jacobi_blocks((int)n, Rt, G, Vw, flags, st);
        if (e != hipSuccess) return e;
    }
    // one 16-lane group per column pair of a Jacobi round, whole waves, so that each round's
    // barrier waits only for waves that have work
    const int64_t pairs = (n + (n & 1)) / 2;
    const int threads = (int)std::min<int64_t>(kSvdThreads, std::max<int64_t>(64, (16 * pairs + 63) / 64 * 64));
    hipLaunchKernelGGL(kern, dim3(1), dim3(threads), lds, st, (int)n, Rt, R,
                       Rf, ldr, Wtop, k, want_q, want_u, S, Sf, V, Vf, ldv, G, Vw, info,
                       keep_info, kBlockSweeps, svd && !use_lds ? flags + kBlockSweeps - 1 : nullptr);
    return hipGetLastError();
}

}  // namespace tsqr
