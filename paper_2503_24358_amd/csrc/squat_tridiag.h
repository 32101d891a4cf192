// Top-r eigenpairs (r <= 64) of a symmetric positive semi-definite 128 x 128 matrix by the
// classical dense route, one 256-thread workgroup per matrix (Section 3.2: the
// right singular vectors and singular values of the query matrix are the
// eigenpairs of its Gram matrix):
//
//   1. Householder reduction to tridiagonal form T.  The matrix lives in the
//      REGISTERS of four wavefronts (one per SIMD), dealt out cyclically: thread
//      (team, lane l of the team of 8) holds rows team, 32 + team, 64 + team,
//      96 + team at columns l, 8 + l, .., 120 + l, so the trailing block
//      shrinks in every thread at once; per step only the product A x and the
//      next column travel through LDS (one barrier per step).
//   2. The r largest eigenvalues of T by 17-section on Sturm counts (16 trial
//      shifts per eigenvalue and round, 14 rounds from [-3, 3] ||T||): the count
//      is the number of sign changes of the three-term recurrence of the leading
//      principal minors, division-free, rescaled by a power of two every 8 terms.
//   3. Eigenvectors of T by twisted factorisations (eigenvalues closer than 1e-11 of
//      the spectrum's scale: by inverse iteration with shifts made distinct by a few
//      ulps where eigenvalues coincide: two solves per vector by Gaussian
//      elimination with partial pivoting, one lane per vector); then the Gram
//      matrix of the vectors decides whether they are orthonormal to 1e-10
//      already (separated eigenvalues), need one symmetric correction step (close
//      eigenvalues) or go through Cholesky-QR (coincident ones).
//   4. Rayleigh quotients = eigenvalues; residuals ||T x - lambda x|| checked.
//   5. Back-transformation by the stored reflectors (kept in LDS during step 1,
//      parked in global memory while steps 2-4 use that LDS block).
//
// A matrix whose result fails the checks of step 4 (never seen with fp64, kept as
// a safety net) is flagged and handed to the Jacobi kernel.  About 40 times fewer
// floating-point operations than cyclic Jacobi on the full matrix.
#pragma once

#include "squat_internal.h"
#include "squat_jacobi.h"

namespace squat {

constexpr int kTriN = 128;
constexpr int kTriRows = 4;             // matrix rows per thread in the reduction: one wavefront per SIMD, with all of its 512
                                        // registers (the first steps hold ~280; capped at 256 they spilled to scratch memory,
                                        // 10000 cycles a step instead of 3200)
constexpr int kTriThreads = kTriN / kTriRows * 8;      // a row's 128 columns are spread over 8 lanes
static_assert(kTriThreads == 256 && (kTriN / kTriRows) % 8 == 0, "whole wavefronts of 8 teams hold the matrix");
constexpr int kTriMaxR = 32;            // vectors the LDS plan holds
constexpr double kTriGap = 1e-11;       // closest eigenvalues (of the spectrum's scale) whose vectors are taken from the twisted form
constexpr double kTriPivMin = 2.0e-19;  // smallest pivot
constexpr double kTriAccept = 1e-9;     // ||T x - lambda x|| / ||T|| and |x_i . x_j| allowed before the fallback

// LDS plan, in doubles
constexpr int kTriXs = 0;               // [2][128] next column of A (double-buffered), by owner; later [128][2] (d, e^2) from the last row up
constexpr int kTriPs = 256;             // [2][128] A x, by owner
constexpr int kTriDd = 512;             // [128] diagonal of T (then normalised)
constexpr int kTriEe = 640;             // [128] sub-diagonal (then normalised)
constexpr int kTriBet = 768;            // [128] beta of every reflector
constexpr int kTriDe = 896;             // [128][2] (d_i, e_{i-1}^2) normalised, for the Sturm recurrence
constexpr int kTriLam = 1152;           // [32] eigenvalues, [32] shifts, [32] Rayleigh quotients, [32] scratch
constexpr int kTriMisc = 1280;          // [64] reductions and flags
constexpr int kTriX = 1344;             // [128][32] vectors, element-major
constexpr int kTriU0 = kTriX + 4096;    // [128][32] reciprocal pivots
constexpr int kTriU1 = kTriU0 + 4096;
constexpr int kTriU2 = kTriU1 + 4096;
constexpr int kTriS = kTriU2 + 4096;    // [32][33] Gram matrix / Cholesky factor
constexpr int kTriLdsDoubles = kTriS + 32 * 33;
constexpr size_t kTriLdsBytes = static_cast<size_t>(kTriLdsDoubles) * sizeof(double);
static_assert(kTriLdsBytes <= 160 * 1024, "LDS plan exceeds a compute unit");
static_assert(kTriX + 16384 == kTriS, "vectors and factors form one 128 KB block (reused for the reflectors)");

__device__ __forceinline__ double tri_block_max(double v, double* scratch, int tid) {
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) v = fmax(v, __shfl_xor(v, s, 64));
    __syncthreads();                                      // scratch may still be read from an earlier use
    if ((tid & 63) == 0) scratch[tid >> 6] = v;
    __syncthreads();
    double m = scratch[0];
#pragma unroll
    for (int w = 1; w < kTriThreads / 64; ++w) m = fmax(m, scratch[w]);
    return m;
}

__device__ __forceinline__ double tri_pow2(int e) {       // 2^e, -1022 <= e <= 1023
    return __hiloint2double((e + 1023) << 20, 0);
}

// Rescales a pair of consecutive minors by a power of two (the larger one to [1, 2)); returns the factor.
__device__ __forceinline__ double tri_rescale(double& p0, double& p1) {
    const double m = fmax(fabs(p0), fabs(p1));
    const int ex = ((__double2hiint(m) >> 20) & 0x7FF) - 1023;
    const double f = ex > -1000 && ex < 1000 ? tri_pow2(-ex) : 1.0;
    p0 *= f;
    p1 *= f;
    return f;
}

// Workgroup barrier that orders LDS traffic only (the Householder loop touches nothing else; the full
// barrier would also wait for the vector-memory counter).
__device__ __forceinline__ void tri_lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ double tri_readlane(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

// Sum over an aligned team of 32 lanes (two rows of 16): row sums by lane permutes, then the two rows
// trade their sums with the row-swap instruction (no trip through the LDS crossbar).
__device__ __forceinline__ double tri_sum32(double v) {
    v = team_sum<16>(v);
    const uint32_t lo = static_cast<uint32_t>(__double2loint(v)), hi = static_cast<uint32_t>(__double2hiint(v));
    const auto sl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto sh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(static_cast<int>(sh[0]), static_cast<int>(sl[0])) +
           __hiloint2double(static_cast<int>(sh[1]), static_cast<int>(sl[1]));
}

// 1 / sqrt(x) and 1 / x from the hardware approximations and Newton steps (short dependent chains: the
// library routines would sit on the critical path of every Householder step).  The approximations are good
// to 5e-8 relative (measured over 2^22 arguments across 120 binades), so two steps reach the last bit: the
// largest relative error after one step is 4e-15, after two 2.6e-16 (reciprocal: 0 against the library's
// division), and a third changes nothing.
__device__ __forceinline__ double tri_rsqrt(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const double e = fma(-x * y, y, 1.0);
        y = fma(0.5 * y, e, y);
    }
    return y;
}
__device__ __forceinline__ double tri_rcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// Lane roles inside a wavefront of the reduction: the eight lanes of a team differ in lane bits 5, 4 and 0 (column
// index l), the team in bits 3..1.  Four row sums of a team then cost four row / half swaps of the wavefront and one
// lane permute instead of three lane permutes each, and leave row r's sum in the lanes with (lane >> 4) == r.
__device__ __forceinline__ int tri_l(int lane) { return (lane >> 4) * 2 + (lane & 1); }
__device__ __forceinline__ int tri_team(int tid) { return (tid >> 6) * 8 + ((tid >> 1) & 7); }
__device__ __forceinline__ int tri_lane_of(int l) { return (l >> 1) * 16 + (l & 1); }     // a lane with column index l

__device__ __forceinline__ double tri_swap32_add(double a, double b) {      // lanes < 32: a over both halves, else b
    const auto sl = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(__double2loint(a)), static_cast<uint32_t>(__double2loint(b)), false, false);
    const auto sh = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(__double2hiint(a)), static_cast<uint32_t>(__double2hiint(b)), false, false);
    return __hiloint2double(static_cast<int>(sh[0]), static_cast<int>(sl[0])) +
           __hiloint2double(static_cast<int>(sh[1]), static_cast<int>(sl[1]));
}
__device__ __forceinline__ double tri_swap16_add(double a, double b) {      // even rows of 16 lanes: a over the row pair, odd rows: b
    const auto sl = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(__double2loint(a)), static_cast<uint32_t>(__double2loint(b)), false, false);
    const auto sh = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(__double2hiint(a)), static_cast<uint32_t>(__double2hiint(b)), false, false);
    return __hiloint2double(static_cast<int>(sh[0]), static_cast<int>(sl[0])) +
           __hiloint2double(static_cast<int>(sh[1]), static_cast<int>(sl[1]));
}
// Sum over a team, the same bits in all of its lanes (and in every team that sums the same numbers).
__device__ __forceinline__ double tri_team_sum(double v) {
#pragma clang fp contract(off)                            // a product folded into one side of an addition would round differently per lane
    v += dpp_move(v, 0);
    v = tri_swap16_add(v, v);
    return tri_swap32_add(v, v);
}

// Householder steps, grouped by the register CC = (k + 1) / 8 of the first column k1 = k + 1 that stays (a compile-time
// index).  Rows and columns are dealt out cyclically: thread (team, l) holds rows team, 32 + team, 64 + team, 96 + team
// at columns 8 c + l, c = 0 .. 15.  The trailing block then shrinks in every thread at once: registers c < CC hold
// finished columns for every lane and groups of rows below CC / 4 finished rows (both skipped at compile time).
//
// A step has ONE workgroup barrier.  Every thread carries the column being eliminated, x = A[k1.., k], in both of its
// index sets (x: its columns, xr: its rows), so A x needs no exchange; the rows' sums and column k1 of A (not yet
// updated) go to LDS, and after the barrier every wavefront forms the rest of the step from them by itself: v = x -
// alpha e_1, u = A v = A x - alpha A e_1, K = beta / 2 v'u, t = u - K v, the rank-two update A - beta (v t' + t v') of
// its registers, and the next column.  alpha and beta do not depend on the exchange and overlap the products A x.  Sums
// over a vector are taken over the eight lanes of a team (16 entries per lane): three stages, not a wavefront's six.
// Bound by instruction issue (one wavefront per SIMD, ~5 cycles an instruction) and the latency of the chain: 3200
// cycles for the first steps, 1100 for the last, 98 us for the 126 of one head, against 139 us with the column, its
// norm, A v and v'p exchanged in turn between two barriers (of one head's 290 us in all, 32 directions).
//
// The copies of an entry in different lanes and wavefronts have to stay the same to the last bit: a difference d
// between the copies of v becomes one of d |A| in the next column, relative to its size d |A| / |x|, step after step, which
// grows without bound where the columns are small (a nearly diagonal matrix).  Hence the same operations in the same
// order for rows and columns, explicit fma and no contraction.
// Entries with index <= k are zero in x, xr and in the LDS vectors (written as zeros), so finished rows and columns
// need no masks.
// LDS vectors are stored by owner, entry i at 4 (i mod 32) + i / 32, so that a thread's four rows are contiguous.
__device__ __forceinline__ int tri_row(int pos) { return 32 * (pos & 3) + (pos >> 2); }     // the entry at a position

// Step k = 8 CC + ll - 1 (column k1 = k + 1 is register CC of the lanes l == ll, row k1 register CC / 4 of one team).
// x, xr: the column in this thread's columns and rows, replaced by v; y, yr receive the next column.
template <int CC>
__device__ __forceinline__ void tri_step(double (&a)[kTriRows][16], double (&x)[16], double (&y)[16], double (&xr)[kTriRows],
                                         double (&yr)[kTriRows], int team, int l, int tid, double* L, const int ll, const int parity) {
#pragma clang fp contract(off)                            // every copy of an entry is to see the same roundings (see above)
    constexpr int R0 = CC / 4;
    const int lane = tid & 63;
    const int k1 = 8 * CC + ll, k = k1 - 1;
    double* ps = L + kTriPs + parity * kTriN;             // A x
    double* cs = L + kTriXs + parity * kTriN;             // column k + 1 of A
    const bool own_c = l == ll, own_r = 32 * R0 + team == k1, live_r = 32 * R0 + team > k;
    // ---- A x (four rows), |x|^2
    double q[kTriRows], o[kTriRows], s2[2];
    static_assert(CC < 16, "registers CC .. 15");
    constexpr int C1 = CC + 1 < 16 ? CC + 1 : CC;
#pragma unroll
    for (int r = 0; r < kTriRows; ++r) {
        q[r] = o[r] = 0.0;
        if (r < R0) continue;
        o[r] = a[r][CC];
        double q0 = a[r][CC] * x[CC], q1 = CC + 1 < 16 ? a[r][C1] * x[C1] : 0.0;
#pragma unroll
        for (int c = CC + 2; c < 16; ++c) {
            if ((c - CC) & 1) q1 = fma(a[r][c], x[c], q1);
            else q0 = fma(a[r][c], x[c], q0);
        }
        q[r] = CC + 1 < 16 ? q0 + q1 : q0;
    }
    q[R0] = live_r ? q[R0] : 0.0;
    s2[0] = x[CC] * x[CC];
    s2[1] = CC + 1 < 16 ? x[C1] * x[C1] : 0.0;
#pragma unroll
    for (int c = CC + 2; c < 16; ++c) s2[(c - CC) & 1] = fma(x[c], x[c], s2[(c - CC) & 1]);
    if (own_c) {
        o[R0] = live_r ? o[R0] : 0.0;
        *reinterpret_cast<double2*>(cs + 4 * team) = double2{o[0], o[1]};
        *reinterpret_cast<double2*>(cs + 4 * team + 2) = double2{o[2], o[3]};
    }
    double mine = tri_swap16_add(tri_swap32_add(q[0], q[2]), tri_swap32_add(q[1], q[3]));
    mine += dpp_move(mine, 0);
    ps[4 * team + (lane >> 4)] = mine;                    // (both lanes of a pair hold and write the same sum)
    // ---- the reflector's scalars: sigma = |x|^2, alpha, beta = 2 / v'v
    const double sigma = tri_team_sum(CC + 1 < 16 ? s2[0] + s2[1] : s2[0]);
    const double x0 = tri_readlane(x[CC], tri_lane_of(ll));
    // (cancellation here only matters when the rest of x is ~1e-16 |x0|^2: then the reflector is the identity to
    // working precision either way; a tiny negative result takes the identity)
    const bool live = sigma - x0 * x0 > 0.0;
    const double sq = sigma * tri_rsqrt(sigma);
    const double alpha = live ? (x0 >= 0.0 ? -sq : sq) : x0;
    const double beta = live ? tri_rcp(fma(fabs(x0), sq, sigma)) : 0.0;
    tri_lds_barrier();
    double t[16], pr[kTriRows];
#pragma unroll
    for (int c = CC; c < 16; ++c) {
        t[c] = ps[4 * (8 * (c & 3) + l) + (c >> 2)];
        y[c] = cs[4 * (8 * (c & 3) + l) + (c >> 2)];
    }
    const double p1 = ps[4 * (k1 & 31) + R0], c1 = cs[4 * (k1 & 31) + R0];
#pragma unroll
    for (int r = 0; r < kTriRows; r += 2) {
        const double2 p2 = *reinterpret_cast<const double2*>(ps + 4 * team + r);
        const double2 c2 = *reinterpret_cast<const double2*>(cs + 4 * team + r);
        pr[r] = p2.x; pr[r + 1] = p2.y;
        yr[r] = c2.x; yr[r + 1] = c2.y;
    }
    // v = x - alpha e_1 in place of x
    x[CC] -= own_c ? alpha : 0.0;
    xr[R0] -= own_r ? alpha : 0.0;
    // reflector k (the block of the later phases is free now)
    *reinterpret_cast<double2*>(L + kTriX + k * kTriN + 4 * team) = double2{xr[0], xr[1]};
    *reinterpret_cast<double2*>(L + kTriX + k * kTriN + 4 * team + 2) = double2{xr[2], xr[3]};
    // u = A v = A x - alpha A e_1;  K = beta / 2 v'u;  t = u - K v  (w = beta t)
#pragma unroll
    for (int c = CC; c < 16; ++c) t[c] = fma(-alpha, y[c], t[c]);
    double t2[2] = {x[CC] * t[CC], CC + 1 < 16 ? x[C1] * t[C1] : 0.0};
#pragma unroll
    for (int c = CC + 2; c < 16; ++c) t2[(c - CC) & 1] = fma(x[c], t[c], t2[(c - CC) & 1]);
    const double K = 0.5 * beta * tri_team_sum(CC + 1 < 16 ? t2[0] + t2[1] : t2[0]);
    const double v1 = x0 - alpha, t1 = fma(-K, v1, fma(-alpha, c1, p1));
    const double bv1 = -beta * v1, bt1 = -beta * t1;
#pragma unroll
    for (int c = CC; c < 16; ++c) t[c] = fma(-K, x[c], t[c]);
    if (tid == 0) {
        L[kTriEe + k] = alpha;
        L[kTriBet + k] = beta;
        L[kTriDd + k1] = fma(2.0 * bv1, t1, c1);
    }
    // rank-two update, and the next column in both index sets
#pragma unroll
    for (int r = R0; r < kTriRows; ++r) {
        const double ti = fma(-K, xr[r], fma(-alpha, yr[r], pr[r]));
        const double nw = -beta * ti, nv = -beta * xr[r];
        yr[r] = fma(xr[r], bt1, fma(ti, bv1, yr[r]));
#pragma unroll
        for (int c = CC; c < 16; ++c) a[r][c] = fma(nv, t[c], fma(nw, x[c], a[r][c]));
    }
#pragma unroll
    for (int c = CC; c < 16; ++c) y[c] = fma(x[c], bt1, fma(t[c], bv1, y[c]));
    y[CC] = own_c ? 0.0 : y[CC];
    yr[R0] = own_r ? 0.0 : yr[R0];
}

// The steps whose first remaining column k1 = k + 1 lies in 8 CC .. 8 CC + 7, two per trip: steps with an even k1 take
// the column from (x, xr) and leave the next in (y, yr), odd ones the other way round.
template <int CC>
__device__ __forceinline__ void tri_steps(double (&a)[kTriRows][16], double (&x)[16], double (&y)[16], double (&xr)[kTriRows],
                                          double (&yr)[kTriRows], int team, int l, int tid, double* L) {
    if constexpr (CC == 0) tri_step<CC>(a, y, x, yr, xr, team, l, tid, L, 1, 1);
#pragma nounroll
    for (int ll = CC == 0 ? 2 : 0; ll < (CC == 15 ? 6 : 8); ll += 2) {
        tri_step<CC>(a, x, y, xr, yr, team, l, tid, L, ll, 0);
        tri_step<CC>(a, y, x, yr, xr, team, l, tid, L, ll + 1, 1);
    }
    if constexpr (CC == 15) tri_step<CC>(a, x, y, xr, yr, team, l, tid, L, 6, 0);
}

// g: the matrix (row-major doubles, symmetric positive semi-definite); vws: 128 x 128 doubles of
// scratch in global memory; qhat: r rows of 128 floats = sqrt(lambda_j) v_j, eigenvalues descending;
// eig: r floats or NULL; r <= 2 kTriMaxR.  Returns (to every thread) whether the result was accepted; if not, the
// outputs are to be redone as a whole (a first batch of rows may have been written).  All kTriThreads threads of
// the block must call it; L: kTriLdsBytes of LDS, 16-byte aligned.
__device__ __forceinline__ bool tridiag_top_eigs(const double* g, double* vws, int r, float* qhat, float* eig,
                                                 double* L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int team = tri_team(tid), l = tri_l(lane);      // this thread's rows team, 32 + team, ... and columns 8 c + l
    double* misc = L + kTriMisc;

    // ---- load, scale by a power of two so that the largest entry is in [1, 2)
    double a[kTriRows][16];
#pragma unroll
    for (int r = 0; r < kTriRows; ++r) {
        const double* src = g + (kTriN / kTriRows * r + team) * kTriN + l;
#pragma unroll
        for (int c = 0; c < 16; ++c) a[r][c] = src[8 * c];
    }
    // column 0 in this thread's columns and rows (the matrix is symmetric)
    double x[16], y[16], xr[kTriRows], yr[kTriRows];
#pragma unroll
    for (int c = 0; c < 16; ++c) y[c] = g[8 * c + l];
#pragma unroll
    for (int r = 0; r < kTriRows; ++r) yr[r] = g[32 * r + team];
    double amax = 0.0;
#pragma unroll
    for (int r = 0; r < kTriRows; ++r)
#pragma unroll
        for (int c = 0; c < 16; ++c) amax = fmax(amax, fabs(a[r][c]));
    amax = tri_block_max(amax, misc, tid);
    if (!(amax > 0.0) || !(amax < 1e300)) {
        // zero matrix: zero eigenvalues, zero rows (also taken for NaN / Inf input: nothing sensible exists)
        for (int e = tid; e < r * kTriN; e += kTriThreads) qhat[e] = 0.0f;
        if (eig)
            for (int e = tid; e < r; e += kTriThreads) eig[e] = 0.0f;
        return true;
    }
    const int aexp = ((__double2hiint(amax) >> 20) & 0x7FF) - 1023;
    const int sexp = aexp < -1000 ? -1000 : (aexp > 1000 ? 1000 : aexp);
    const double down = tri_pow2(-sexp), up = tri_pow2(sexp);
#pragma unroll
    for (int r = 0; r < kTriRows; ++r)
#pragma unroll
        for (int c = 0; c < 16; ++c) a[r][c] *= down;

    // ---- 1. Householder reduction
    for (int e = tid; e < 4 * kTriN; e += kTriThreads) L[e] = 0.0;      // column and product buffers: never read uninitialised
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 16; ++c) y[c] = 8 * c + l > 0 ? y[c] * down : 0.0;
#pragma unroll
    for (int r = 0; r < kTriRows; ++r) yr[r] = 32 * r + team > 0 ? yr[r] * down : 0.0;
    if (tid == 0) L[kTriDd] = a[0][0];
    tri_steps<0>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<1>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<2>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<3>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<4>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<5>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<6>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<7>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<8>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<9>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<10>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<11>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<12>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<13>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<14>(a, x, y, xr, yr, team, l, tid, L);
    tri_steps<15>(a, x, y, xr, yr, team, l, tid, L);
    // the last 2 x 2 block: its first diagonal entry came with the last step, the next column is e_126, and the corner
    // is in the last team's last row
    if (team == 31 && l == 7) {
        L[kTriDd + kTriN - 1] = a[kTriRows - 1][15];
        L[kTriEe + kTriN - 2] = y[15];
        L[kTriEe + kTriN - 1] = 0.0;
        L[kTriBet + kTriN - 2] = 0.0;
        L[kTriBet + kTriN - 1] = 0.0;
    }
    __syncthreads();
    // the reflectors leave LDS (their block is needed for the vectors and factors) and come back for step 5
    for (int e = tid * 2; e < (kTriN - 2) * kTriN; e += 2 * kTriThreads)
        *reinterpret_cast<double2*>(vws + e) = *reinterpret_cast<const double2*>(L + kTriX + e);

    // ---- normalise T to max |entry| = 1
    double tmax = 0.0;
    if (tid < kTriN) tmax = fmax(fabs(L[kTriDd + tid]), fabs(L[kTriEe + tid]));
    tmax = tri_block_max(tmax, misc, tid);                // > 0: the trace is preserved
    const double tinv = 1.0 / tmax;
    __syncthreads();
    if (tid < kTriN) {
        const double dn = L[kTriDd + tid] * tinv, en = L[kTriEe + tid] * tinv;
        L[kTriDd + tid] = dn;
        L[kTriEe + tid] = en;
        L[kTriDe + 2 * tid] = dn;
        if (tid + 1 < kTriN) L[kTriDe + 2 * (tid + 1) + 1] = en * en;
        if (tid == 0) L[kTriDe + 1] = 0.0;
        // the same from the last row up (the buffers of the reduction are free now)
        L[kTriXs + 2 * (kTriN - 1 - tid)] = dn;
        L[kTriXs + 2 * (kTriN - 1 - tid) + 1] = tid + 1 < kTriN ? en * en : 0.0;
    }
    __syncthreads();

    // Steps 2-5 take the eigenpairs in batches of kTriMaxR, largest first (the LDS plan holds that many vectors): r <= 32
    // is one batch; for more, T and the reflectors serve every batch.  (Two inlined copies of the batch rather than
    // a loop around one: inside a loop the compiler spills a hundred registers.)
    double lam_edge = 0.0;                                // smallest eigenvalue of the batch before
    auto batch = [&](const int joff, const int rb) -> bool {
        // ---- 2. the rb largest eigenvalues by multisection on Sturm counts.  A power-of-two team of threads per eigenvalue,
        // NP trial shifts per thread; `points` = team size x NP trial shifts divide a bracket into points + 1 parts.
        auto search = [&](auto np_tag, const int team_size, const int rounds) {
            constexpr int NP = decltype(np_tag)::value;
            const int j = tid / team_size, sub = tid & (team_size - 1);
            if (j >= rb) return;
            const int points = team_size * NP;
            const double inv_parts = 1.0 / (points + 1);
            const int below_target = kTriN - 1 - (joff + j);  // eigenvalue joff + j (descending) has this many below it
            const unsigned long long team_mask = team_size == 64 ? ~0ull : ((1ull << team_size) - 1ull) << (lane & ~(team_size - 1));
            double lo = -3.0001, hi = 3.0001;
            const double* de = L + kTriDe;
            for (int round = 0; round < rounds; ++round) {
                asm volatile("" ::: "memory");                // keep the 128 LDS reads inside the round (not hoisted into registers)
                const double step = (hi - lo) * inv_parts;
                double x[NP], p0[NP], p1[NP];
                uint32_t signs[NP];
                int cnt[NP];
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    x[q] = fma(step, static_cast<double>(sub + q * team_size + 1), lo);
                    p0[q] = 1.0;
                    p1[q] = de[0] - x[q];
                    // The signs of the minors are shifted into a register, newest at bit 0 (one instruction per term);
                    // a block's sign changes are then the ones of (signs ^ signs >> 1) over its terms.  The sign of
                    // p_0 = 1 is 0, so the first minor's own sign is a change.
                    signs[q] = static_cast<uint32_t>(__double2hiint(p1[q])) >> 31;
                    cnt[q] = static_cast<int>(signs[q]);
                }
                auto block = [&](int b, auto nt_tag) {
                    constexpr int NTERMS = decltype(nt_tag)::value;
#pragma unroll
                    for (int u = 0; u < NTERMS; ++u) {
                        const double2 t = *reinterpret_cast<const double2*>(de + 2 * (b + u));
#pragma unroll
                        for (int q = 0; q < NP; ++q) {
                            const double p2 = fma(t.x - x[q], p1[q], -(t.y * p0[q]));
                            signs[q] = __builtin_amdgcn_alignbit(signs[q], static_cast<uint32_t>(__double2hiint(p2)), 31);
                            p0[q] = p1[q];
                            p1[q] = p2;
                        }
                    }
#pragma unroll
                    for (int q = 0; q < NP; ++q) {
                        cnt[q] += __popc((signs[q] ^ (signs[q] >> 1)) & ((1u << NTERMS) - 1u));
                        tri_rescale(p0[q], p1[q]);
                    }
                };
                static_assert((kTriN - 1) % 8 == 7, "15 blocks of 8 terms and one of 7");
                for (int b = 1; b + 8 <= kTriN; b += 8) block(b, std::integral_constant<int, 8>{});
                block(kTriN - 7, std::integral_constant<int, 7>{});
                // the team's points are ascending: those with count <= target are a prefix
                int nb = 0;
#pragma unroll
                for (int q = 0; q < NP; ++q) nb += __popcll(__ballot(cnt[q] <= below_target) & team_mask);
                const double nlo = nb == 0 ? lo : fma(step, static_cast<double>(nb), lo);
                const double nhi = nb == points ? hi : fma(step, static_cast<double>(nb + 1), lo);
                lo = nlo;
                hi = nhi;
            }
            if (sub == 0) L[kTriLam + j] = 0.5 * (lo + hi);
        };
        // (parts^rounds > 6 x 2^53)
        if (rb > 16)
            search(std::integral_constant<int, 2>{}, 8, 14);
        else if (rb > 8)
            search(std::integral_constant<int, 1>{}, 16, 14);
        else if (rb > 4)
            search(std::integral_constant<int, 1>{}, 32, 12);
        else
            search(std::integral_constant<int, 1>{}, 64, 10);
        __syncthreads();
        // A later batch stands on its own only if its eigenvalues are clear of the batch before (vectors of eigenvalues
        // closer than this could share a subspace, which only a joint orthonormalisation would see)
        if (joff > 0 && !(lam_edge - L[kTriLam] >= 1e-7)) return false;      // uniform
        lam_edge = L[kTriLam + rb - 1];

        // ---- 3. eigenvectors of T.  Eigenvalues at least kTriGap apart (of the spectrum's scale): twisted factorisation.
        // The leading minors P_i of T - lambda (top down) and the trailing ones Q_i (bottom up) are two three-term
        // recurrences, one lane each; their ratios are the pivots D+_i = P_{i+1} / P_i and D-_i of the LDL' and UDU'
        // factorisations.  With gamma_i = D+_i + D-_i - (d_i - lambda), smallest in size at row k, the vector with
        // z_k = 1 and z_i = -(e_i / D+_i) z_{i+1} above, z_i = -(e_{i-1} / D-_i) z_{i-1} below has the residual
        // |gamma_k| / |z| (Parlett and Dhillon, "Fernando's solution to Wilkinson's problem", 1997): one pass of two
        // multiply-adds per row, and everything after it is spread over all threads (eight per vector).  The inverse
        // iteration below, one lane per vector through two solves with a reciprocal per row, took 48 us of one head's
        // 300; this takes ~3.  It is kept for eigenvalues closer than that, whose vectors come out of the twisted form
        // nearly parallel, while it starts from independent vectors.
        bool close = false;
        {
            const double gap = lane + 1 < rb ? L[kTriLam + lane] - L[kTriLam + lane + 1] : 1.0;
            close = __ballot(!(gap >= kTriGap)) != 0ull;  // every wavefront sees the same
        }
        if (!close) {
            if (tid < 64) {
                const int j = tid & 31;
                const bool rising = tid >= 32;                  // bottom-up half
                const double lam = L[kTriLam + (j < rb ? j : rb - 1)];
                const double* src = L + (rising ? kTriXs : kTriDe);      // (d, e^2) in the order of the recurrence
                double* dst = L + (rising ? kTriU1 : kTriU0) + j; // dst[32 i] = minor i + 1
                double p0 = 1.0, p1 = src[0] - lam;
                if (fabs(p1) < kTriPivMin) p1 = kTriPivMin;
                dst[0] = p1;
                auto block = [&](int m0, auto nt_tag) {
                    constexpr int NT = decltype(nt_tag)::value;
#pragma unroll
                    for (int u = 0; u < NT; ++u) {
                        const double2 t = *reinterpret_cast<const double2*>(src + 2 * (m0 + u));
                        double p2 = fma(t.x - lam, p1, -(t.y * p0));
                        if (fabs(p2) < kTriPivMin * fabs(p1)) p2 = kTriPivMin * p1;      // a pivot below the threshold: the threshold
                        dst[32 * (m0 + u)] = p2;
                        p0 = p1;
                        p1 = p2;
                    }
                    tri_rescale(p0, p1);                      // (the stored minors keep the old scale: redone below)
                };
                block(1, std::integral_constant<int, 7>{});
                for (int m0 = 8; m0 < kTriN; m0 += 8) block(m0, std::integral_constant<int, 8>{});
            }
            __syncthreads();
            // thread (j, sg): rows 16 sg .. 16 sg + 15 of vector j
            constexpr int RS = kTriN / 8;
            const int j = tid & 31, sg = tid >> 5;
            const double lam = L[kTriLam + (j < rb ? j : rb - 1)];
            double rp[RS], rm[RS];                            // -e_i / D+_i and -e_{i-1} / D-_i
            double gbest = 1e300;
            int kbest = 16 * sg;
            {
                double dp[RS];
                const double* P = L + kTriU0 + j;
                const double* Q = L + kTriU1 + j;
#pragma unroll
                for (int h = 0; h < 2; ++h) {                 // blocks of 8 minors share a scale
                    const int i0 = 16 * sg + 8 * h;
                    double pa = 1.0;                          // P_{i0}, in the scale of its block
                    if (i0 > 0) {
                        double pb = P[32 * (i0 - 2)];
                        pa = P[32 * (i0 - 1)];
                        tri_rescale(pb, pa);
                    }
                    double inv = tri_rcp(pa);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int i = 8 * h + u;
                        const double pn = P[32 * (i0 + u)];
                        dp[i] = pn * inv;
                        inv = tri_rcp(pn);
                        rp[i] = -L[kTriEe + i0 + u] * (pa * inv);
                        pa = pn;
                    }
                }
#pragma unroll
                for (int h = 1; h >= 0; --h) {                // bottom up: row i is minor 127 - i
                    const int m0 = kTriN - 8 - (16 * sg + 8 * h);
                    double qa = 1.0;
                    if (m0 > 0) {
                        double qb = Q[32 * (m0 - 2)];
                        qa = Q[32 * (m0 - 1)];
                        tri_rescale(qb, qa);
                    }
                    double inv = tri_rcp(qa);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int i = 8 * h + 7 - u, row = 16 * sg + i;
                        const double qn = Q[32 * (m0 + u)];
                        const double dm = qn * inv;
                        inv = tri_rcp(qn);
                        rm[i] = row > 0 ? -L[kTriEe + row - 1] * (qa * inv) : 0.0;
                        qa = qn;
                        const double ga = fabs(dp[i] + dm - (L[kTriDd + row] - lam));
                        if (ga < gbest) { gbest = ga; kbest = row; }
                    }
                }
            }
            double* G = L + kTriX;                            // [8][32] smallest |gamma|, its row, products of a segment, sums
            G[tid] = gbest;
            G[256 + tid] = static_cast<double>(kbest);
            __syncthreads();
            int k = 0;
            {
                double best = 2e300;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const double v = G[32 * q + j];
                    if (v < best) { best = v; k = static_cast<int>(G[256 + 32 * q + j]); }
                }
            }
            // products of the segment's factors, away from row k
            double down_p = 1.0, up_p = 1.0;
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                down_p *= 16 * sg + i > k ? rm[i] : 1.0;
                up_p *= 16 * sg + i < k ? rp[i] : 1.0;
            }
            G[512 + tid] = up_p;
            G[768 + tid] = down_p;
            __syncthreads();
            double c_up = 1.0, c_down = 1.0;                  // z next to this segment's last / first row
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                c_up *= q > sg ? G[512 + 32 * q + j] : 1.0;
                c_down *= q < sg ? G[768 + 32 * q + j] : 1.0;
            }
            double z[RS], ss = 0.0;
#pragma unroll
            for (int i = RS - 1; i >= 0; --i) {
                c_up *= 16 * sg + i < k ? rp[i] : 1.0;
                z[i] = c_up;
            }
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                c_down *= 16 * sg + i > k ? rm[i] : 1.0;
                z[i] = 16 * sg + i > k ? c_down : z[i];
                ss = fma(z[i], z[i], ss);
            }
            G[1024 + tid] = ss;
            __syncthreads();
            double total = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) total += G[1024 + 32 * q + j];
            const double nrm = 1.0 / sqrt(total);
            __syncthreads();                                  // G is part of X
#pragma unroll
            for (int i = 0; i < RS; ++i) L[kTriX + 32 * (16 * sg + i) + j] = z[i] * nrm;
        } else {
            // inverse iteration, one lane per vector
            if (tid == 0) {
                const double sep = 10.0 * 2.220446049250313e-16;  // coincident eigenvalues get shifts a few ulps apart
                double prev = L[kTriLam];
                L[kTriLam + 32] = prev;
                for (int j = 1; j < rb; ++j) {
                    double s = L[kTriLam + j];
                    s = s > prev - sep ? prev - sep : s;
                    L[kTriLam + 32 + j] = s;
                    prev = s;
                }
            }
            // columns rb .. 31 are padding (unit vectors, never used)
            for (int e = tid; e < kTriN * 32; e += kTriThreads) {
                const int row = e >> 5, colj = e & 31;
                // start vectors: a fixed pseudo-random pattern in (-1, 1)
                uint32_t h = static_cast<uint32_t>(row) * 2654435761u + static_cast<uint32_t>(colj) * 40503u + 12345u;
                h ^= h >> 15;
                h *= 2246822519u;
                h ^= h >> 13;
                const double rnd = (static_cast<double>(h >> 8) + 0.5) * (2.0 / 16777216.0) - 1.0;
                L[kTriX + e] = colj < rb ? rnd : (row == colj ? 1.0 : 0.0);
            }
            __syncthreads();
            if (tid < rb) {
                const int j = tid;
                const double shift = L[kTriLam + 32 + j];
                    const double* dn = L + kTriDd;
                const double* en = L + kTriEe;
                double* X = L + kTriX + j;
                double* U0 = L + kTriU0 + j;
                double* U1 = L + kTriU1 + j;
                double* U2 = L + kTriU2 + j;
                double scale = 1.0;
                for (int it = 0; it < 2; ++it) {
                    // forward elimination with row interchanges, applied to the right-hand side on the fly
                    double ca = dn[0] - shift, cc = en[0], cf = 0.0, cb = X[0] * scale;
                    for (int row = 0; row < kTriN - 1; ++row) {
                        const double na = en[row], nc = dn[row + 1] - shift, nf = row + 1 < kTriN - 1 ? en[row + 1] : 0.0;
                        const double nb = X[32 * (row + 1)] * scale;
                        const bool keep = fabs(ca) >= fabs(na);
                        double pa = keep ? ca : na, pc = keep ? cc : nc, pf = keep ? cf : nf, pb = keep ? cb : nb;
                        const double oa = keep ? na : ca, oc = keep ? nc : cc, of = keep ? nf : cf, ob = keep ? nb : cb;
                        if (fabs(pa) < kTriPivMin) pa = pa < 0.0 ? -kTriPivMin : kTriPivMin;
                        const double inv = tri_rcp(pa);
                        const double mlt = oa * inv;
                        U0[32 * row] = inv;
                        U1[32 * row] = pc;
                        U2[32 * row] = pf;
                        X[32 * row] = pb;
                        ca = fma(-mlt, pc, oc);
                        cc = fma(-mlt, pf, of);
                        cf = 0.0;
                        cb = fma(-mlt, pb, ob);
                    }
                    if (fabs(ca) < kTriPivMin) ca = ca < 0.0 ? -kTriPivMin : kTriPivMin;
                    // back substitution
                    double x2 = 0.0, x1 = cb * tri_rcp(ca), big = fabs(x1);
                    X[32 * (kTriN - 1)] = x1;
                    for (int row = kTriN - 2; row >= 0; --row) {
                        const double x = (X[32 * row] - U1[32 * row] * x1 - U2[32 * row] * x2) * U0[32 * row];
                        X[32 * row] = x;
                        big = fmax(big, fabs(x));
                        x2 = x1;
                        x1 = x;
                    }
                    scale = big > 0.0 && big < 1e300 ? 1.0 / big : 1.0;
                }
                // unit 2-norm
                double s2 = 0.0;
                for (int row = 0; row < kTriN; ++row) {
                    const double x = X[32 * row] * scale;
                    s2 = fma(x, x, s2);
                }
                const double nrm = scale * (s2 > 0.0 ? 1.0 / sqrt(s2) : 0.0);
                for (int row = 0; row < kTriN; ++row) X[32 * row] *= nrm;
            }
        }
        __syncthreads();
        // ---- orthonormality: Gram matrix of the 32 columns; Cholesky-QR (twice) only if it is not the identity
        double* S = L + kTriS;
        bool ok = true;
        for (int pass = 0; pass < 3; ++pass) {
            double dev = 0.0;
            if (tid < 256) {
                const int a2 = tid >> 4, b2 = tid & 15;
                double s00 = 0.0, s01 = 0.0, s10 = 0.0, s11 = 0.0;
                for (int row = 0; row < kTriN; ++row) {
                    const double2 xa = *reinterpret_cast<const double2*>(L + kTriX + 32 * row + 2 * a2);
                    const double2 xb = *reinterpret_cast<const double2*>(L + kTriX + 32 * row + 2 * b2);
                    s00 = fma(xa.x, xb.x, s00);
                    s01 = fma(xa.x, xb.y, s01);
                    s10 = fma(xa.y, xb.x, s10);
                    s11 = fma(xa.y, xb.y, s11);
                }
                S[(2 * a2) * 33 + 2 * b2] = s00;
                S[(2 * a2) * 33 + 2 * b2 + 1] = s01;
                S[(2 * a2 + 1) * 33 + 2 * b2] = s10;
                S[(2 * a2 + 1) * 33 + 2 * b2 + 1] = s11;
                // only the rb real columns count (the padding columns are never used)
                const double i00 = a2 == b2 ? 1.0 : 0.0;
                const bool ra0 = 2 * a2 < rb, ra1 = 2 * a2 + 1 < rb, rb0 = 2 * b2 < rb, rb1 = 2 * b2 + 1 < rb;
                dev = fmax(fmax(ra0 && rb0 ? fabs(s00 - i00) : 0.0, ra1 && rb1 ? fabs(s11 - i00) : 0.0),
                           fmax(ra0 && rb1 ? fabs(s01) : 0.0, ra1 && rb0 ? fabs(s10) : 0.0));
            }
            dev = tri_block_max(dev, misc, tid);
            if (!(dev == dev)) ok = false;
            if (dev <= 1e-10 || !ok) break;
            if (pass == 2) {
                ok = dev <= kTriAccept;
                break;
            }
            if (dev <= 1e-5) {
                // nearly orthonormal (close eigenvalues, not coincident ones): one symmetric step
                // X <- X (3/2 I - 1/2 S) squares the deviation
                constexpr int NP = kTriN * 8 / kTriThreads;    // row passes per thread
                const int j0 = 4 * (tid & 7);
                double out[NP][4];
#pragma unroll
                for (int ps2 = 0; ps2 < NP; ++ps2) {
                    const double* xr = L + kTriX + 32 * ((tid >> 3) + ps2 * (kTriThreads / 8));
#pragma unroll
                    for (int c = 0; c < 4; ++c) out[ps2][c] = 0.0;
                    for (int k2 = 0; k2 < rb; ++k2) {
                        const double xk = xr[k2];
#pragma unroll
                        for (int c = 0; c < 4; ++c) out[ps2][c] = fma(xk, S[k2 * 33 + j0 + c], out[ps2][c]);
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c) out[ps2][c] = fma(-0.5, out[ps2][c], 1.5 * xr[j0 + c]);
                }
                __syncthreads();
#pragma unroll
                for (int ps2 = 0; ps2 < NP; ++ps2)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (j0 + c < rb) L[kTriX + 32 * ((tid >> 3) + ps2 * (kTriThreads / 8)) + j0 + c] = out[ps2][c];
                __syncthreads();
                continue;
            }
            // Cholesky S = C C' in place (lower triangle), one wavefront, lane = row
            if (wave == 0) {
                int bad = 0;
                for (int j = 0; j < rb; ++j) {
                    double acc = 0.0;
                    if (lane < rb && lane >= j) {
                        acc = S[lane * 33 + j];
                        for (int k2 = 0; k2 < j; ++k2) acc = fma(-S[lane * 33 + k2], S[j * 33 + k2], acc);
                    }
                    const double piv = __shfl(acc, j, 64);
                    if (!(piv > 1e-280)) bad = 1;
                    const double rs = bad ? 0.0 : 1.0 / sqrt(piv);
                    if (lane < rb && lane >= j) S[lane * 33 + j] = lane == j ? rs : acc * rs;      // diagonal: 1 / C_jj
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
                if (lane == 0) misc[32] = bad ? 1.0 : 0.0;
            }
            __syncthreads();
            if (misc[32] != 0.0) {
                ok = false;
                break;
            }
            // X <- X C^-T : row by row, y_j = (x_j - sum_{k<j} C_jk y_k) / C_jj
            if (tid < kTriN) {
                double* xr = L + kTriX + 32 * tid;
                double y[32];
#pragma unroll
                for (int j = 0; j < 32; ++j) {
                    if (j < rb) {                              // uniform
                        double acc = xr[j];
#pragma unroll
                        for (int k2 = 0; k2 < j; ++k2) acc = fma(-S[j * 33 + k2], y[k2], acc);
                        y[j] = acc * S[j * 33 + j];
                    }
                }
#pragma unroll
                for (int j = 0; j < 32; ++j)
                    if (j < rb) xr[j] = y[j];
            }
            __syncthreads();
        }

        // ---- 4. Rayleigh quotients and residuals: team of 32 lanes per vector, 4 elements per lane, NV
        // vectors per thread
        constexpr int NV = 32 * 32 / kTriThreads;
        const int sub = tid & 31;
        double xv[NV][4];
        {
            double worst = 0.0;
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const int vj = (tid >> 5) + q * (kTriThreads / 32);
                double num = 0.0, den = 0.0;
                double yv[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int row = sub + 32 * m;
                    const double x = L[kTriX + 32 * row + vj];
                    const double xm = row > 0 ? L[kTriX + 32 * (row - 1) + vj] : 0.0;
                    const double xp = row < kTriN - 1 ? L[kTriX + 32 * (row + 1) + vj] : 0.0;
                    const double em = row > 0 ? L[kTriEe + row - 1] : 0.0;
                    const double y = fma(L[kTriDd + row], x, fma(em, xm, L[kTriEe + row] * xp));
                    xv[q][m] = x;
                    yv[m] = y;
                    num = fma(x, y, num);
                    den = fma(x, x, den);
                }
                num = tri_sum32(num);
                den = tri_sum32(den);
                const double rq = den > 0.0 ? num / den : 0.0;
                double res = 0.0;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const double t = yv[m] - rq * xv[q][m];
                    res = fma(t, t, res);
                }
                res = tri_sum32(res);
                if (sub == 0) L[kTriLam + 64 + vj] = rq;
                double w = vj < rb ? sqrt(res) : 0.0;
                if (!(w == w)) w = 1e300;
                worst = fmax(worst, w);
            }
            worst = tri_block_max(worst, misc, tid);
            if (!(worst <= kTriAccept)) ok = false;
        }
        if (!ok) return false;                                // uniform: every thread saw the same flags

        // ---- 5. back-transformation: team of 16 lanes per vector, lane s holds the elements at positions s, s + 16, ...,
        // s + 112 of NB vectors (two where the batch has more than 16).  Per reflector and lane: a dot product over 8
        // elements per vector, a sum over the 16 lanes, 8 multiply-adds per vector; the next reflector's entries are
        // fetched meanwhile.  The vectors are read from LDS in this layout before the reflectors come back from global
        // memory into their block.
        auto back = [&](auto nb_tag) {
            constexpr int NB = decltype(nb_tag)::value;
            const int bvj = tid >> 4, bs = tid & 15;
            double xb[NB][8];
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int m = 0; m < 8; ++m) xb[q][m] = L[kTriX + 32 * tri_row(bs + 16 * m) + bvj + 16 * q];
            __syncthreads();
            __threadfence_block();
            double* V = L + kTriX;
            // (unrolled, so that the loads of several trips are in flight together: one trip at a time, each of the
            // trips waits out a whole global-memory round trip)
#pragma unroll 16
            for (int e = tid * 2; e < (kTriN - 2) * kTriN; e += 2 * kTriThreads)
                *reinterpret_cast<double2*>(V + e) = *reinterpret_cast<const double2*>(vws + e);
            __syncthreads();
            double vn[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) vn[m] = V[(kTriN - 3) * kTriN + bs + 16 * m];
            // (a wavefront holds four vectors per q: one whose vectors are all padding skips the loop)
            for (int k = 4 * wave < rb ? kTriN - 3 : -1; k >= 0; --k) {
                const double beta = L[kTriBet + k];
                double v[8];
#pragma unroll
                for (int m = 0; m < 8; ++m) v[m] = vn[m];
                if (k > 0) {
#pragma unroll
                    for (int m = 0; m < 8; ++m) vn[m] = V[(k - 1) * kTriN + bs + 16 * m];
                }
                if (beta == 0.0) continue;                    // uniform
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    double s0 = 0.0, s1 = 0.0;
#pragma unroll
                    for (int m = 0; m < 8; m += 2) {
                        s0 = fma(v[m], xb[q][m], s0);
                        s1 = fma(v[m + 1], xb[q][m + 1], s1);
                    }
                    const double sc = team_sum<16>(s0 + s1) * beta;
#pragma unroll
                    for (int m = 0; m < 8; ++m) xb[q][m] = fma(-sc, v[m], xb[q][m]);
                }
            }

            // ---- output: rank by eigenvalue, sign so that the largest component is positive, rows sqrt(lambda) v
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int vj = bvj + 16 * q;
                if (vj >= rb) continue;                       // uniform per team of 16 lanes
                const double lam = L[kTriLam + 64 + vj];
                int rank = 0;
                for (int o = 0; o < rb; ++o) {
                    const double lo = L[kTriLam + 64 + o];
                    rank += (lo > lam) || (lo == lam && o < vj);
                }
                double best = -1.0, bestv = 0.0;
                int besti = kTriN;
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const double av = fabs(xb[q][m]);
                    const int row = tri_row(bs + 16 * m);
                    if (av > best || (av == best && row < besti)) { best = av; bestv = xb[q][m]; besti = row; }
                }
#pragma unroll
                for (int off = 8; off > 0; off >>= 1) {
                    const double ob = __shfl_xor(best, off, 64);
                    const double ov = __shfl_xor(bestv, off, 64);
                    const int oi = __shfl_xor(besti, off, 64);
                    if (ob > best || (ob == best && oi < besti)) { best = ob; bestv = ov; besti = oi; }
                }
                const double lam_true = fmax(lam, 0.0) * tmax * up;
                const double sc = (bestv < 0.0 ? -1.0 : 1.0) * sqrt(lam_true);
                float* dst = qhat + (joff + rank) * kTriN;
#pragma unroll
                for (int m = 0; m < 8; ++m) dst[tri_row(bs + 16 * m)] = static_cast<float>(xb[q][m] * sc);
                if (eig && bs == 0) eig[joff + rank] = static_cast<float>(lam_true);
            }
        };
        if (rb > 16)
            back(std::integral_constant<int, 2>{});
        else
            back(std::integral_constant<int, 1>{});
        __syncthreads();                                  // the next batch reuses every LDS block
        return true;
    };
    if (!batch(0, r < kTriMaxR ? r : kTriMaxR)) return false;
    if (r > kTriMaxR) {
        if (!batch(kTriMaxR, r - kTriMaxR)) return false;
    }
    return true;
}

}  // namespace squat
