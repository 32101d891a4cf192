// Top-r eigenpairs (r <= 64) of a symmetric positive semi-definite 128 x 128 matrix by the
// classical dense route, one 256-thread workgroup per matrix (Section 3.2: the
// right singular vectors and singular values of the query matrix are the
// eigenpairs of its Gram matrix):
//
//   1. Householder reduction to tridiagonal form T.  The matrix lives in the
//      REGISTERS of four wavefronts (one per SIMD): a wavefront holds the rows of
//      its own number modulo 4, two lanes a row, one the even, one the odd
//      columns, so the trailing block shrinks in every wavefront at once and a
//      product with a vector stays in the lane; per step only the product A x, the
//      next column and one number per wavefront travel through LDS (one barrier);
//      the last 31 steps on one wavefront, without.
//   2. The r largest eigenvalues of T by Sturm counts (a team of threads per
//      eigenvalue, a trial shift each): the count
//      is the number of sign changes of the three-term recurrence of the leading
//      principal minors, division-free, rescaled by a power of two every 8 terms;
//      once a bracket holds one eigenvalue the trial shifts follow the zero of a
//      linear fraction through its ends and a third shift.
//   3. Eigenvectors of T by twisted factorisations (eigenvalues closer than 1e-11 of
//      the spectrum's scale: by inverse iteration with shifts made distinct by a few
//      ulps where eigenvalues coincide: two solves per vector by Gaussian
//      elimination with partial pivoting, one lane per vector); then the Gram
//      matrix of the vectors decides whether they are orthonormal to 1e-10
//      already (separated eigenvalues), need one symmetric correction step (close
//      eigenvalues) or go through Cholesky-QR (coincident ones).
//   4. Rayleigh quotients = eigenvalues; residuals ||T x - lambda x|| checked.
//   5. Back-transformation in blocks of 16 reflectors on the matrix cores (their
//      operands are formed beside the end of step 1 and after it, while the
//      reflectors are in LDS, and wait
//      in global memory while steps 2-4 use that LDS block).
//
// A matrix whose result fails the checks of step 4 (never seen with fp64, kept as
// a safety net) is handed to the Jacobi routine of squat_jacobi.h.  About 40 times fewer
// floating-point operations than cyclic Jacobi on the full matrix.
#pragma once

#include "squat_internal.h"
#include "squat_jacobi.h"

namespace squat {

constexpr int kTriN = 128;
constexpr int kTriThreads = 256;        // one wavefront per SIMD, with all of its 512 registers
constexpr int kTriMaxR = 32;            // vectors the LDS plan holds
constexpr double kTriGap = 1e-11;       // closest eigenvalues (of the spectrum's scale) whose vectors are taken from the twisted form
constexpr double kTriTiny = 1e-290;     // |x|^2 below which a column counts as zero
constexpr double kTriPivMin = 2.0e-19;  // smallest pivot
constexpr double kTriBound = 3.0001;     // > the largest eigenvalue of a tridiagonal matrix with entries of at most 1
constexpr double kTriPart = 2.0 * kTriBound / 257.0;
constexpr double kTriWidth = 4.5e-16;   // width of an eigenvalue's bracket (one unit in the last place of numbers from 2 to 4)
constexpr double kTriAccept = 1e-9;     // ||T x - lambda x|| / ||T|| and |x_i . x_j| allowed before the fallback
#ifndef SQUAT_TRI_REFUSED               // matrices refused all the same, by the exponent of their largest entry: a build for tests has some
#define SQUAT_TRI_REFUSED(exponent) false
#endif

// LDS plan, in doubles
constexpr int kTriSs = 0;               // [2][4][64] in the reduction: the wavefronts' parts of x'A x (lanes 16 .. 31)
constexpr int kTriXs = 0;               // [128][2] later: (d, e^2) from the last row up
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
constexpr int kTriS = kTriU2 + 4096;    // [32][33] Gram matrix / Cholesky factor, or [8][16][17] the blocks' T factors
constexpr int kTriPs = kTriS;           // in the reduction: [2][128] A x
constexpr int kTriCs = kTriS + 256;     // and [2][128] the next column of A
constexpr int kTriTLd = 17;
constexpr int kTriLdsDoubles = kTriS + 8 * 16 * kTriTLd;
constexpr size_t kTriLdsBytes = static_cast<size_t>(kTriLdsDoubles) * sizeof(double);
constexpr int kTriWsPerWave = 9 * 8 * 64;              // operands of the back-transformation, per wavefront, and per matrix:
constexpr int kTriWsDoubles = kTriThreads / 64 * kTriWsPerWave;
constexpr int kTriVLd = 130;            // reflector k at kTriX + 130 k in the reduction (over the vectors and factors, not in use yet);
                                        // 130: the 16 reflectors of a matrix operand fall on different banks
constexpr int kTriTail = 96;            // first column of the reduction's last steps, on one wavefront
constexpr int kTriTailW = kTriS + 512;  // [32][33] its matrix, [32] the column in hand
constexpr int kTriTailLd = 33;
static_assert(512 + 32 * kTriTailLd + 32 <= 8 * 16 * kTriTLd, "aliased blocks");
static_assert(kTriLdsBytes <= 160 * 1024, "LDS plan exceeds a compute unit");
static_assert((kTriN - 2) * kTriVLd <= 4 * 4096 && 32 * 33 <= 8 * 16 * kTriTLd, "aliased blocks");

typedef double double4v __attribute__((ext_vector_type(4)));

// Max over the workgroup (by lane permutes and swaps inside a wavefront: no trips through the LDS crossbar).
__device__ __forceinline__ double tri_block_max(double v, double* scratch, int tid) {
#pragma unroll
    for (int sel = 0; sel < 4; ++sel) v = fmax(v, dpp_move(v, sel));
    {
        const uint32_t lo = static_cast<uint32_t>(__double2loint(v)), hi = static_cast<uint32_t>(__double2hiint(v));
        const auto sl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto sh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        v = fmax(__hiloint2double(static_cast<int>(sh[0]), static_cast<int>(sl[0])),
                 __hiloint2double(static_cast<int>(sh[1]), static_cast<int>(sl[1])));
    }
    {
        const uint32_t lo = static_cast<uint32_t>(__double2loint(v)), hi = static_cast<uint32_t>(__double2hiint(v));
        const auto sl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto sh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        v = fmax(__hiloint2double(static_cast<int>(sh[0]), static_cast<int>(sl[0])),
                 __hiloint2double(static_cast<int>(sh[1]), static_cast<int>(sl[1])));
    }
    __syncthreads();                                      // scratch may still be read from an earlier use
    if ((tid & 63) == 0) scratch[tid >> 6] = v;
    __syncthreads();
    double m = scratch[0];
#pragma unroll
    for (int w = 1; w < kTriThreads / 64; ++w) m = fmax(m, scratch[w]);
    return m;
}

// Waits for the LDS reads issued so far, once: the reads that follow are then the only ones the compiler has to count.
__device__ __forceinline__ void tri_lds_wait() { __builtin_amdgcn_s_waitcnt(0xC07F); }      // lgkmcnt(0), nothing else

__device__ __forceinline__ double tri_pow2(int e) {       // 2^e, -1022 <= e <= 1023
    return __hiloint2double((e + 1023) << 20, 0);
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

// 1 / sqrt(x) and 1 / x from the hardware approximations, good to 5e-8 relative, and one step of the series in the remaining
// error up to its cube (short dependent chains: the library routines would sit on the critical path of every Householder
// step).  Largest relative errors over 2^22 arguments across 120 binades: 1.4e-16 and 1.1e-16 (two Newton steps: 2.6e-16).
__device__ __forceinline__ double tri_rsqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);                 // 1 / sqrt(x) = y (1 + e / 2 + 3 e^2 / 8 + 5 e^3 / 16 + ..)
    return fma(y * e, fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ double tri_rcp(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);                     // 1 / x = y (1 + e + e^2 + e^3 + ..)
    return fma(y, fma(e, e, e), y);
}

// Sum over the two halves of a wavefront / over pairs of 16 lanes, of two numbers at once.
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

// ---- multiply-adds whose first factor is one lane's number for each row of 16 lanes (v_fmac_f64 with row_newbcast; at the
// rate of the plain one).  Eight registers of matrix columns a[8] meet the lanes 0..7 (HI: 8..15) of x; the first M of them
// are left out.  A lane permute must not read a register in the two cycles behind the instruction that wrote it, which the
// compiler does not see here: each block waits first.
#define TRI_FM(D, S, A, J) "v_fmac_f64_dpp " D ", " S ", " A " row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
#define TRI_BLOCK(P0, P1, P2, P3, ...)                                   \
    do {                                                                 \
        if constexpr (M == 0) asm("s_nop 1\n\t" P0 P1 P2 P3 __VA_ARGS__); \
        else if constexpr (M == 2) asm("s_nop 1\n\t" P1 P2 P3 __VA_ARGS__); \
        else if constexpr (M == 4) asm("s_nop 1\n\t" P2 P3 __VA_ARGS__); \
        else asm("s_nop 1\n\t" P3 __VA_ARGS__);                          \
    } while (0)

// q0 + q1 += a x
#define TRI_MV(B0, B1, J0, J1) TRI_FM("%0", "%2", B0, J0) TRI_FM("%1", "%2", B1, J1)
#define TRI_MV_OPS : "+v"(q0), "+v"(q1) : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7])
template <bool HI, int M>
__device__ __forceinline__ void tri_mv(double& q0, double& q1, double x, const double* a) {
    if constexpr (!HI)
        TRI_BLOCK(TRI_MV("%3", "%4", 0, 1), TRI_MV("%5", "%6", 2, 3), TRI_MV("%7", "%8", 4, 5), TRI_MV("%9", "%10", 6, 7), TRI_MV_OPS);
    else
        TRI_BLOCK(TRI_MV("%3", "%4", 8, 9), TRI_MV("%5", "%6", 10, 11), TRI_MV("%7", "%8", 12, 13), TRI_MV("%9", "%10", 14, 15), TRI_MV_OPS);
}
// a += nv u + nt v
#define TRI_UP(B0, B1, J0, J1) TRI_FM(B0, "%8", "%10", J0) TRI_FM(B1, "%8", "%10", J1) TRI_FM(B0, "%9", "%11", J0) TRI_FM(B1, "%9", "%11", J1)
#define TRI_UP_OPS : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]) \
    : "v"(u), "v"(v), "v"(nv), "v"(nt)
template <bool HI, int M>
__device__ __forceinline__ void tri_up(double* a, double u, double v, double nv, double nt) {
    if constexpr (!HI)
        TRI_BLOCK(TRI_UP("%0", "%1", 0, 1), TRI_UP("%2", "%3", 2, 3), TRI_UP("%4", "%5", 4, 5), TRI_UP("%6", "%7", 6, 7), TRI_UP_OPS);
    else
        TRI_BLOCK(TRI_UP("%0", "%1", 8, 9), TRI_UP("%2", "%3", 10, 11), TRI_UP("%4", "%5", 12, 13), TRI_UP("%6", "%7", 14, 15), TRI_UP_OPS);
}
#undef TRI_FM
#undef TRI_BLOCK
#undef TRI_MV
#undef TRI_MV_OPS
#undef TRI_UP
#undef TRI_UP_OPS

// Householder steps.  Wavefront w holds the rows 4 m + w, m = lane & 31, lane (h = lane >> 5, m) the columns 2 j + h, j = 0 ..
// 63, of its row.  The vectors of a step are kept twice: by columns (register e of lane (h, i = lane & 15): entry 32 e + 2 i +
// h, the same in every wavefront and in both rows of 16 lanes of a half), and the entry of the lane's own row.  A product with
// a vector by columns takes its factors by broadcast inside the rows of 16 lanes, in the instruction itself.
//
// A step (k1 = k + 1 is the first column that stays) has ONE workgroup barrier.  Before it: p = A x for the wavefront's rows
// (one sum over the halves), the wavefront's part of x'A x, and |x|^2; p, that part and column k1 of A (not yet updated; one
// half of the lanes holds it, the other writes p in the same instruction) go to LDS.  After it every wavefront forms the rest
// by itself: v = x - alpha e_1, u = A v = p - alpha A e_1, v'u = x'p - 2 alpha p_1 + alpha^2 a_11 (which costs no second sum
// over the lanes), K = beta / 2 v'u, t = u - K v, the rank-two update A - beta (v t' + t v') = A - beta (v u' + (u - 2 K v) v')
// of its rows, and the next column.  alpha and beta do not depend on the exchange.
// Bound by instruction issue (one wavefront per SIMD, four cycles an instruction, fp64 or not, dependent or not) and, with the
// blocks getting small, by the barrier and the exchange: 300 instructions and 1800 cycles a step at the start, 200 and
// 1180 with 32 columns left, where the last steps take another form (below); of one head 61 us for these 95, 10.6 for the last 31 and
// the hand-over to them.  Before, every thread held four rows at 16 columns and 20 entries of each vector
// (16 by columns, a copy in each of a wavefront's eight teams, and 4 by rows), the sum x'u followed the exchange, and a step was
// 556 and 152 instructions: 99 us.  What did not help: the same with two rows a lane and the sums over the wavefronts formed
// by the readers (79 us; LDS), all steps unrolled (same time a step, the compiler spills), the scalars in front of the barrier.
// Writes of many lanes to one LDS address cost 200 cycles a step: every lane has a place of its own, and T stays in registers.
//
// The copies of an entry in different lanes and wavefronts have to stay the same to the last bit: a difference d
// between the copies of v becomes one of d |A| in the next column, relative to its size d |A| / |x|, step after step, which
// grows without bound where the columns are small (a nearly diagonal matrix).  Hence the same operations in the same
// order for rows and columns, explicit fma and no contraction.
// Entries with index <= k are zero in x; finished rows and the finished columns that share a block of registers with others
// are updated too (with finite numbers: a finished row is only turned by the reflectors) and never used.
struct TriLane {
    int lane, wave, row, col;                             // col: 2 i + h
    int pos[2];                                           // where this lane writes its row in an odd / even step: p or column k1
    int rowpos;                                           // its row's place in a vector by columns
};

// A vector by columns in LDS: entry 32 e + 2 i + h, pairs of e beside each other.
__device__ __forceinline__ int tri_pos(int entry) { return (entry >> 6) * 64 + (entry & 31) * 2 + ((entry >> 5) & 1); }

// Steps with k1 = 8 G + ll: registers 4 G + ll / 2 of the lanes with h = ll & 1 hold column k1.  xr, xc: the column, replaced by
// the next one.
template <int G, int S>                                   // S = ll & 1
__device__ __forceinline__ void tri_step(double (&a)[64], double& xr, double (&xc)[4], const TriLane& id, double (&T)[3],
                                         double* const vp, double* L, const int ll) {
#pragma clang fp contract(off)                            // every copy of an entry is to see the same roundings (see above)
    constexpr int R = G / 4, B0 = G / 2, M = G % 2 * 4;
    const int k1 = 8 * G + ll, src = 32 * S + ((4 * G + (ll >> 1)) & 15);      // (a lane that holds column k1)
    const double* ps = L + kTriPs + S * kTriN;            // A x
    const double* cs = L + kTriCs + S * kTriN;            // column k1 of A
    double* sp = L + kTriSs + S * 256 + 16;               // the parts of x'A x, 64 doubles apart
    // ---- A x for the wavefront's rows
    double q0 = 0.0, q1 = 0.0;
    tri_mv<B0 % 2 == 1, M>(q0, q1, xc[B0 / 2], a + 8 * B0);
    if constexpr (B0 < 7) tri_mv<(B0 + 1) % 2 == 1, 0>(q0, q1, xc[(B0 + 1) / 2 & 3], a + 8 * ((B0 + 1) & 7));
    if constexpr (B0 < 6) tri_mv<(B0 + 2) % 2 == 1, 0>(q0, q1, xc[(B0 + 2) / 2 & 3], a + 8 * ((B0 + 2) & 7));
    if constexpr (B0 < 5) tri_mv<(B0 + 3) % 2 == 1, 0>(q0, q1, xc[(B0 + 3) / 2 & 3], a + 8 * ((B0 + 3) & 7));
    if constexpr (B0 < 4) tri_mv<(B0 + 4) % 2 == 1, 0>(q0, q1, xc[(B0 + 4) / 2 & 3], a + 8 * ((B0 + 4) & 7));
    if constexpr (B0 < 3) tri_mv<(B0 + 5) % 2 == 1, 0>(q0, q1, xc[(B0 + 5) / 2 & 3], a + 8 * ((B0 + 5) & 7));
    if constexpr (B0 < 2) tri_mv<(B0 + 6) % 2 == 1, 0>(q0, q1, xc[(B0 + 6) / 2 & 3], a + 8 * ((B0 + 6) & 7));
    if constexpr (B0 < 1) tri_mv<(B0 + 7) % 2 == 1, 0>(q0, q1, xc[(B0 + 7) / 2 & 3], a + 8 * ((B0 + 7) & 7));
    q0 = q0 + q1;
    q0 = tri_swap32_add(q0, q0);
    const double k0 = a[4 * G], k2 = a[4 * G + 1], k4 = a[4 * G + 2], k6 = a[4 * G + 3];
    const double ck = ll < 4 ? (ll < 2 ? k0 : k2) : (ll < 6 ? k4 : k6);
    L[id.pos[S]] = id.lane >> 5 == S ? ck : q0;
    double s2 = xc[3] * xc[3];
#pragma unroll
    for (int e = R; e < 3; ++e) s2 = fma(xc[e], xc[e], s2);
    double z = tri_swap16_add(s2, xr * q0);               // even rows of 16 lanes: 2 |x|^2 of the half, odd ones: x'A x
#pragma unroll
    for (int sel = 0; sel < 4; ++sel) z += dpp_move(z, sel);
    sp[64 * id.wave + id.lane - 16] = z;                  // (a place for every lane: writes of many lanes to one are slow)
    const double sigma2 = tri_readlane(z, 0) + tri_readlane(z, 32), x0 = tri_readlane(xc[R], src);
    tri_lds_barrier();
    double p[4], c[4];
#pragma unroll
    for (int e = R & 2; e < 4; e += 2) {
        if constexpr (R == 3) {
            p[3] = ps[64 + 2 * id.col + 1];
            c[3] = cs[64 + 2 * id.col + 1];
        } else {
            const double2 pe = *reinterpret_cast<const double2*>(ps + 32 * e + 2 * id.col);
            const double2 ce = *reinterpret_cast<const double2*>(cs + 32 * e + 2 * id.col);
            p[e] = pe.x; p[e + 1] = pe.y;
            c[e] = ce.x; c[e + 1] = ce.y;
        }
    }
    const double pr = ps[id.rowpos], cr = cs[id.rowpos];
    const double s0 = sp[0], s1 = sp[64], s2b = sp[128], s3 = sp[192];
    __builtin_amdgcn_sched_barrier(0);                    // the scalars are formed while these are on their way
    // ---- the reflector's scalars: sigma = |x|^2, al = -alpha, beta = 2 / v'v.  A column of nothing (|x| < 1e-145, of entries
    // of at most 2) takes the identity; alpha is then of that size as well.
    const double sg = fma(0.5, sigma2, kTriTiny);
    const double al = copysign(sg * tri_rsqrt(sg), x0);
    const double binv = tri_rcp(fma(fabs(x0), fabs(al), sg));
    const double beta = sigma2 > kTriTiny ? binv : 0.0;
    __builtin_amdgcn_sched_barrier(0);
    // u = A v
    double u[4];
#pragma unroll
    for (int e = R; e < 4; ++e) u[e] = fma(al, c[e], p[e]);
    const double ur = fma(al, cr, pr);
    const double u1 = tri_readlane(u[R], src), c1 = tri_readlane(c[R], src);
    const double vu = fma(al, fma(-al, c1, u1 + u1), (s0 + s1) + (s2b + s3));
    const double K2 = beta * vu;                          // 2 K
    const double v1 = x0 + al;
    const double bv1 = -beta * v1, bt1 = -beta * fma(-K2, v1, u1);
    // v = x - alpha e_1 in place of x
    const bool own = id.row == k1;
    xr = own ? v1 : xr;
    xc[R] = id.col == (k1 & 31) ? v1 : xc[R];
    vp[ll * kTriVLd] = xr;                                // reflector k (the block of the later phases is free now)
    // rank-two update, and the next column.  (What is finished gets the high half of a zero: a number below 1e-313.)
    const double nv = -beta * xr, nt = -beta * fma(-K2, xr, ur);
    xr = fma(xr, bt1, fma(ur, bv1, cr));
    // the lanes of row k1 keep T's entries d_k1 and -e_k, and beta
    T[0] = own ? xr : T[0];
    T[1] = own ? al : T[1];
    T[2] = own ? beta : T[2];
    xr = __hiloint2double(id.row > k1 ? __double2hiint(xr) : 0, __double2loint(xr));
    double vc[4];
#pragma unroll
    for (int e = R; e < 4; ++e) {
        vc[e] = xc[e];
        xc[e] = fma(xc[e], bt1, fma(u[e], bv1, c[e]));
    }
    xc[R] = __hiloint2double(id.col > (k1 & 31) ? __double2hiint(xc[R]) : 0, __double2loint(xc[R]));
    tri_up<B0 % 2 == 1, M>(a + 8 * B0, u[B0 / 2], vc[B0 / 2], nv, nt);
    if constexpr (B0 < 7) tri_up<(B0 + 1) % 2 == 1, 0>(a + 8 * ((B0 + 1) & 7), u[(B0 + 1) / 2 & 3], vc[(B0 + 1) / 2 & 3], nv, nt);
    if constexpr (B0 < 6) tri_up<(B0 + 2) % 2 == 1, 0>(a + 8 * ((B0 + 2) & 7), u[(B0 + 2) / 2 & 3], vc[(B0 + 2) / 2 & 3], nv, nt);
    if constexpr (B0 < 5) tri_up<(B0 + 3) % 2 == 1, 0>(a + 8 * ((B0 + 3) & 7), u[(B0 + 3) / 2 & 3], vc[(B0 + 3) / 2 & 3], nv, nt);
    if constexpr (B0 < 4) tri_up<(B0 + 4) % 2 == 1, 0>(a + 8 * ((B0 + 4) & 7), u[(B0 + 4) / 2 & 3], vc[(B0 + 4) / 2 & 3], nv, nt);
    if constexpr (B0 < 3) tri_up<(B0 + 5) % 2 == 1, 0>(a + 8 * ((B0 + 5) & 7), u[(B0 + 5) / 2 & 3], vc[(B0 + 5) / 2 & 3], nv, nt);
    if constexpr (B0 < 2) tri_up<(B0 + 6) % 2 == 1, 0>(a + 8 * ((B0 + 6) & 7), u[(B0 + 6) / 2 & 3], vc[(B0 + 6) / 2 & 3], nv, nt);
    if constexpr (B0 < 1) tri_up<(B0 + 7) % 2 == 1, 0>(a + 8 * ((B0 + 7) & 7), u[(B0 + 7) / 2 & 3], vc[(B0 + 7) / 2 & 3], nv, nt);
}

// The steps whose first remaining column k1 = k + 1 lies in 8 G .. 8 G + 7, two per trip (the LDS buffers alternate).
template <int G>
__device__ __forceinline__ void tri_steps(double (&a)[64], double& xr, double (&xc)[4], const TriLane& id, double (&T)[3], double* L) {
    double* const vp = L + kTriX + (8 * G - 1) * kTriVLd + id.row;
    if constexpr (G == 0) tri_step<G, 1>(a, xr, xc, id, T, vp, L, 1);
#pragma nounroll
    for (int ll = G == 0 ? 2 : 0; ll < 8; ll += 2) {
        tri_step<G, 0>(a, xr, xc, id, T, vp, L, ll);
        tri_step<G, 1>(a, xr, xc, id, T, vp, L, ll + 1);
    }
}

// The last steps, k1 = 96 .. 126, on one wavefront and without LDS or barriers: with 32 columns left, lanes l and l + 32 hold row
// 96 + rho, rho = 2 (l & 15) + (l >> 4 & 1), the lower half its even columns, the upper one the odd ones.  The sums of a row's two
// halves are then in both of them, and a vector by rows becomes one by columns (lane (h, i): column 2 i + h, in both rows of
// 16 lanes of the half) by one swap of rows of 16 lanes.  Everything else as above.
// Bound by instruction issue: 178 instructions a step, 130 at the end, against 200 and 160 with the barrier and the exchange (~300
// cycles) on top.  Build of the subspace with them | now, us: one head 122.5 | 119.8, 8 heads x 4 131.5 | 128.5, 256 heads 151.6 |
// 148.2.  The same from 64 columns on (a lane per row): 125; the four wavefronts' share of the products is worth their barrier there.
template <int S>                                          // v of the lower (upper) half, in both
__device__ __forceinline__ double tri_both(double v) {
    const auto sl = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(__double2loint(v)), static_cast<uint32_t>(__double2loint(v)), false, false);
    const auto sh = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(__double2hiint(v)), static_cast<uint32_t>(__double2hiint(v)), false, false);
    return __hiloint2double(static_cast<int>(sh[S]), static_cast<int>(sl[S]));
}
__device__ __forceinline__ double tri_columns(double v, bool lower) {
    const auto sl = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(__double2loint(v)), static_cast<uint32_t>(__double2loint(v)), false, false);
    const auto sh = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(__double2hiint(v)), static_cast<uint32_t>(__double2hiint(v)), false, false);
    return __hiloint2double(static_cast<int>(lower ? sh[0] : sh[1]), static_cast<int>(lower ? sl[0] : sl[1]));
}
template <int G, int S>                                   // k1 = 96 + 8 G + ll, S = ll & 1
__device__ __forceinline__ void tri_tail_step(double (&a)[16], double& xr, double& xc, int lane, int rho, double (&T)[3],
                                              double* const vp, const int ll) {
#pragma clang fp contract(off)
    constexpr int B0 = G / 2, M = G % 2 * 4;
    const int at = 4 * G + (ll >> 1), src = 16 * S + at;  // column k1: registers `at` of the half S; its row: lanes src, src + 32
    double q0 = 0.0, q1 = 0.0;
    tri_mv<B0 == 1, M>(q0, q1, xc, a + 8 * B0);
    if constexpr (B0 < 1) tri_mv<true, 0>(q0, q1, xc, a + 8);
    q0 = q0 + q1;
    const double p = tri_swap32_add(q0, q0);
    const double k0 = a[4 * G], k2 = a[4 * G + 1], k4 = a[4 * G + 2], k6 = a[4 * G + 3];
    const double c = tri_both<S>(ll < 4 ? (ll < 2 ? k0 : k2) : (ll < 6 ? k4 : k6));
    double z = tri_swap16_add(xr * xr, xr * p);           // even rows of 16 lanes: |x|^2, odd ones: x'A x
#pragma unroll
    for (int sel = 0; sel < 4; ++sel) z += dpp_move(z, sel);
    const double sigma2 = tri_readlane(z, 0), xax = tri_readlane(z, 16), x0 = tri_readlane(xr, src);
    const double sg = sigma2 + kTriTiny;
    const double al = copysign(sg * tri_rsqrt(sg), x0);
    const double binv = tri_rcp(fma(fabs(x0), fabs(al), sg));
    const double beta = sigma2 > kTriTiny ? binv : 0.0;
    const double u = fma(al, c, p);
    const double u1 = tri_readlane(u, src), c1 = tri_readlane(c, src);
    const double vu = fma(al, fma(-al, c1, u1 + u1), xax);
    const double K2 = beta * vu;
    const double v1 = x0 + al;
    const double bv1 = -beta * v1, bt1 = -beta * fma(-K2, v1, u1);
    const bool own = (lane & 31) == src;
    xr = own ? v1 : xr;
    const double vc = (lane & 47) == 32 * S + at ? v1 : xc;
    vp[ll * kTriVLd] = xr;
    const double nv = -beta * xr, nt = -beta * fma(-K2, xr, u);
    xr = fma(xr, bt1, fma(u, bv1, c));
    T[0] = own ? xr : T[0];
    T[1] = own ? al : T[1];
    T[2] = own ? beta : T[2];
    xr = __hiloint2double(rho > 8 * G + ll ? __double2hiint(xr) : 0, __double2loint(xr));
    xc = tri_columns(xr, lane < 32);
    const double uc = tri_columns(u, lane < 32);
    tri_up<B0 == 1, M>(a + 8 * B0, uc, vc, nv, nt);
    if constexpr (B0 < 1) tri_up<true, 0>(a + 8, uc, vc, nv, nt);
}
template <int G>
__device__ __forceinline__ void tri_tail_steps(double (&a)[16], double& xr, double& xc, int lane, int rho, double (&T)[3], double* L) {
    double* const vp = L + kTriX + (kTriTail + 8 * G - 1) * kTriVLd + kTriTail + rho;
#pragma nounroll
    for (int ll = 0; ll < (G == 3 ? 6 : 8); ll += 2) {
        tri_tail_step<G, 0>(a, xr, xc, lane, rho, T, vp, ll);
        tri_tail_step<G, 1>(a, xr, xc, lane, rho, T, vp, ll + 1);
    }
    if constexpr (G == 3) tri_tail_step<G, 0>(a, xr, xc, lane, rho, T, vp, 6);
}

// Eight terms of the three-term recurrence of the leading principal minors of T - x, p_{i+1} = (d_i - x) p_i - e_{i-1}^2
// p_{i-1}, for the rows whose d_i and -e_{i-1}^2 are held by the lanes 0 .. 7 (HI: 8 .. 15) of each row of 16 lanes; nx = -x.
// (x p_i is rounded, d_i p_i is not: an error of x by half a unit in its last place.)  PIV: piv p_i is added, so that no minor
// vanishes against the one before it.
#define TRI_BC " row_newbcast:"
#define TRI_FULL " row_mask:0xf bank_mask:0xf\n\t"
#define TRI_T0(P2, P1, P0, J, W) "v_mul_f64 " P2 ", %10, " P1 "\n\t" W "v_fmac_f64_dpp " P2 ", %11, " P1 TRI_BC #J TRI_FULL "v_fmac_f64_dpp " P2 ", %12, " P0 TRI_BC #J TRI_FULL
#define TRI_T1(P2, P1, P0, J, W) TRI_T0(P2, P1, P0, J, W) "v_fmac_f64_e32 " P2 ", %13, " P1 "\n\t"
#define TRI_EIGHT(T, J0, J1, J2, J3, J4, J5, J6, J7)                                                                                \
    asm(T("%0", "%8", "%9", J0, "s_nop 0\n\t") T("%1", "%0", "%8", J1, "") T("%2", "%1", "%0", J2, "") T("%3", "%2", "%1", J3, "")  \
        T("%4", "%3", "%2", J4, "") T("%5", "%4", "%3", J5, "") T("%6", "%5", "%4", J6, "") T("%7", "%6", "%5", J7, "")             \
        : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3]), "=&v"(p[4]), "=&v"(p[5]), "=&v"(p[6]), "=&v"(p[7])                    \
        : "v"(p1), "v"(p0), "v"(nx), "v"(d), "v"(e), "v"(piv))
template <bool HI, bool PIV>
__device__ __forceinline__ void tri_eight(double (&p)[8], double p0, double p1, double nx, double d, double e, double piv) {
    if constexpr (!HI && !PIV) TRI_EIGHT(TRI_T0, 0, 1, 2, 3, 4, 5, 6, 7);
    else if constexpr (!PIV) TRI_EIGHT(TRI_T0, 8, 9, 10, 11, 12, 13, 14, 15);
    else if constexpr (!HI) TRI_EIGHT(TRI_T1, 0, 1, 2, 3, 4, 5, 6, 7);
    else TRI_EIGHT(TRI_T1, 8, 9, 10, 11, 12, 13, 14, 15);
}
#undef TRI_BC
#undef TRI_FULL
#undef TRI_T0
#undef TRI_T1
#undef TRI_EIGHT

// Rescales a pair of consecutive minors by a power of two (the larger one to [1/2, 1)); returns the exponent taken out.
__device__ __forceinline__ int tri_rescale(double& p0, double& p1) {
    double m;
    asm("v_max_f64 %0, |%1|, |%2|" : "=v"(m) : "v"(p0), "v"(p1));
    const int ex = __builtin_amdgcn_frexp_exp(m);         // (0 for a zero, an infinity or a NaN)
    p0 = __builtin_ldexp(p0, -ex);
    p1 = __builtin_ldexp(p1, -ex);
    return ex;
}

// Sturm count (sign changes of the minors) and last minor p1 2^ex of T - x; d, e: lane i of a row of 16 lanes holds the rows
// 16 b + i.  Four instructions a term (with T read from LDS, one 16-byte read a term, they were eight: 46 cycles a term where
// this takes 21 with its share of the rescaling and counting).
__device__ __forceinline__ void tri_minors(const double (&d)[8], const double (&e)[8], double x, double& p1, int& cnt, int& ex) {
    double p0 = 0.0;
    uint32_t signs = 0;                                   // newest at bit 0; that of p_0 = 1 is 0
    p1 = 1.0;
    cnt = ex = 0;
    auto eight = [&](int b, auto hi_tag) __attribute__((always_inline)) {
        double p[8];
        tri_eight<decltype(hi_tag)::value, false>(p, p0, p1, -x, d[b], e[b], 0.0);
#pragma unroll
        for (int u = 0; u < 8; ++u) signs = __builtin_amdgcn_alignbit(signs, static_cast<uint32_t>(__double2hiint(p[u])), 31);
        p0 = p[6];
        p1 = p[7];
        ex += tri_rescale(p0, p1);
    };
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        eight(b, std::false_type{});
        eight(b, std::true_type{});
        cnt += __popc((signs ^ (signs >> 1)) & 0xFFFFu);
    }
}

// g: the matrix (row-major doubles, symmetric positive semi-definite); vws: kTriWsDoubles doubles of
// scratch in global memory; qhat: r rows of 128 floats = sqrt(lambda_j) v_j, eigenvalues descending;
// eig: r floats or NULL; r <= 2 kTriMaxR.  Returns (to every thread) whether the result was accepted; if not, the
// outputs are to be redone as a whole (a first batch of rows may have been written).  All kTriThreads threads of
// the block must call it; L: kTriLdsBytes of LDS, 16-byte aligned.
__device__ __forceinline__ bool tridiag_top_eigs(const double* g, double* vws, int r, float* qhat, float* eig,
                                                 double* L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double* misc = L + kTriMisc;

    // ---- load (a column is read as the row of the same number: 512 bytes of a wavefront's load lie side by side), scale by a
    // power of two so that the largest entry is in [1, 2)
    TriLane id;
    id.lane = lane;
    id.wave = wave;
    id.row = 4 * (lane & 31) + wave;
    id.col = 2 * (lane & 15) + (lane >> 5);
    id.rowpos = tri_pos(id.row);
    id.pos[0] = (lane >> 5 == 0 ? kTriCs : kTriPs) + id.rowpos;
    id.pos[1] = (lane >> 5 == 1 ? kTriCs : kTriPs) + kTriN + id.rowpos;
    double a[64], xr = g[id.row], xc[4];                  // (xr, xc: column 0)
#pragma unroll
    for (int j = 0; j < 64; ++j) a[j] = g[(2 * j + (lane >> 5)) * kTriN + id.row];
#pragma unroll
    for (int e = 0; e < 4; ++e) xc[e] = g[32 * e + id.col];
    double amax = 0.0;
#pragma unroll
    for (int j = 0; j < 64; ++j) amax = fmax(amax, fabs(a[j]));
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
    for (int j = 0; j < 64; ++j) a[j] *= down;

    // ---- 1. Householder reduction
    __syncthreads();                                      // (everyone is past amax's scratch)
    const double d0 = a[0];
    xr = id.row > 0 ? xr * down : 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) xc[e] = 32 * e + id.col > 0 ? xc[e] * down : 0.0;
    double T[3] = {0.0, 0.0, 0.0};
    tri_steps<0>(a, xr, xc, id, T, L);
    tri_steps<1>(a, xr, xc, id, T, L);
    tri_steps<2>(a, xr, xc, id, T, L);
    tri_steps<3>(a, xr, xc, id, T, L);
    tri_steps<4>(a, xr, xc, id, T, L);
    tri_steps<5>(a, xr, xc, id, T, L);
    tri_steps<6>(a, xr, xc, id, T, L);
    tri_steps<7>(a, xr, xc, id, T, L);
    tri_steps<8>(a, xr, xc, id, T, L);
    tri_steps<9>(a, xr, xc, id, T, L);
    tri_steps<10>(a, xr, xc, id, T, L);
    tri_steps<11>(a, xr, xc, id, T, L);
    // ---- operands of the back-transformation, while the reflectors are in LDS.  The reflectors are taken in blocks of 16,
    // H_{16 b} ... H_{16 b + 15} = I - V T V' with T upper triangular, T_mm = beta_m, T_{0..m-1, m} = -beta_m T (V'v_m).
    // Wavefront w keeps the row tiles w and 7 - w (16 rows each) of the vectors; as the first rows of a block's
    // reflectors are zero, tile t meets the blocks b <= t only.  Per (tile, block): V' as the A operand of V'X (4
    // registers) and -(V T)' likewise for X - (V T)(V'X); both wait in global memory, as the lanes hold them, until step 5
    // (kept in registers meanwhile they slow steps 2-4 down: 40 k cycles more in the search).  v_mfma_f64_16x16x4_f64: A lane (i = lane & 15, k = lane >> 4), B lane (j = lane & 15, k = lane >> 4), result
    // lane (j = lane & 15), register q: row (lane >> 4) + 4 q, i.e. a result is the B operand of the next product as it is.
    // The blocks 0 .. 4, whose reflectors are there by then, are the work of wavefronts 1 .. 3 beside the last steps; of the
    // others a wavefront takes one each behind them (6 pairs of 36).  A block's T and pairs stay with one wavefront, so that no
    // barrier stands between.  All behind the steps, 15 k cycles, against 7 k: build of the subspace, us, one head 119.9 | 116.6,
    // 32 heads 132.8 | 129.3, 256 heads 147.4 | 145.3.
    const int mi = lane & 15, mk = lane >> 4;
    // [wavefront][9 (tile, block) pairs: tile 7 - wave with blocks 0 .. 7 - wave, tile `wave` with blocks 0 .. wave]
    // [registers 0 1, 2 3 of V', of -(V T)'][64][2]
    double2* const vmine = reinterpret_cast<double2*>(vws + wave * kTriWsPerWave);
    auto block_operands = [&](const int bA, const int bB) __attribute__((always_inline)) {      // of one or two blocks; uniform
        const double* V = L + kTriX;
        double* TS = L + kTriS;
        for (int b = bA;; b = bB) {                           // V'V
            const bool real = 16 * b + mi < kTriN - 2;        // reflectors 126 and 127 do not exist
            const double* v = V + (real ? 16 * b + mi : 0) * kTriVLd;
            double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
            for (int m = 4 * b; m < kTriN / 4; ++m) {
                double x = v[4 * m + mk];
                x = real ? x : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, x, acc, 0, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) TS[(16 * b + mk + 4 * q) * kTriTLd + mi] = acc[q];
            if (b == bB) break;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // T, a row per lane (lanes 0 .. 15: block bA, 16 .. 31: block bB)
        {
            const int b = (lane & 16) ? bB : bA;
            double* S = TS + 16 * b * kTriTLd;
            double t[16];
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                double sum = 0.0;
#pragma unroll
                for (int q = 0; q < m; ++q) sum = fma(t[q], S[q * kTriTLd + m], sum);
                const double bt = L[kTriBet + 16 * b + m];
                t[m] = m == mi ? bt : (m > mi ? -bt * sum : 0.0);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (lane < 32) {
#pragma unroll
                for (int m = 0; m < 16; ++m) S[mi * kTriTLd + m] = t[m];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int b = bA;; b = bB) {
            const bool real = 16 * b + mi < kTriN - 2;
            const double* vk = V + (real ? 16 * b + mi : 0) * kTriVLd;
#pragma unroll 3
            for (int tile = b; tile < 8; ++tile) {
                const int owner = tile < 4 ? tile : 7 - tile;
                double2* const dst = reinterpret_cast<double2*>(vws + owner * kTriWsPerWave) + (tile < 4 ? 8 - tile + b : b) * (4 * 64);
                double4v acc = {0.0, 0.0, 0.0, 0.0};
                double x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x[q] = vk[16 * tile + 4 * q + mk];
                    x[q] = real ? x[q] : 0.0;
                    const bool kreal = 16 * b + 4 * q + mk < kTriN - 2;
                    double y = V[(kreal ? 16 * b + 4 * q + mk : 0) * kTriVLd + 16 * tile + mi];
                    y = kreal ? y : 0.0;
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(TS[(16 * b + 4 * q + mk) * kTriTLd + mi], y, acc, 0, 0, 0);
                }
                dst[lane] = double2{x[0], x[1]};
                dst[64 + lane] = double2{x[2], x[3]};
                dst[128 + lane] = double2{-acc[0], -acc[1]};
                dst[192 + lane] = double2{-acc[2], -acc[3]};
            }
            if (b == bB) break;
        }
    };

    // the last 32 rows to wavefront 0; meanwhile the others clear what its reflectors have above
    {
        double* const W = L + kTriTailW;
        double* const X = W + 32 * kTriTailLd;
        if ((lane & 31) >= kTriTail / 4) {
            const int row = id.row - kTriTail;
#pragma unroll
            for (int j = 0; j < 16; ++j) W[row * kTriTailLd + 2 * j + (lane >> 5)] = a[kTriTail / 2 + j];
            X[row] = xr;                                  // (both halves have it)
        }
        // T and the reflectors' beta, of the rows before those
        if (id.row == 0) {
            if (lane == 0) L[kTriDd] = d0;
        } else if (id.row < kTriTail) {
            L[kTriDd + id.row] = T[0];
            L[kTriEe + id.row - 1] = -T[1];
            L[kTriBet + id.row - 1] = T[2];
        }
        __syncthreads();
        const int rho = 2 * (lane & 15) + (lane >> 4 & 1);
        double t[16], x = 0.0, y = 0.0;
        if (wave == 0) {
#pragma unroll
            for (int j = 0; j < 16; ++j) t[j] = W[rho * kTriTailLd + 2 * j + (lane >> 5)];
            x = X[rho];
            y = X[id.col];
        }
        __syncthreads();                                  // (the blocks' T factors go where W was)
        if (wave == 0) {
            double T2[3] = {0.0, 0.0, 0.0};
            tri_tail_steps<0>(t, x, y, lane, rho, T2, L);
            tri_tail_steps<1>(t, x, y, lane, rho, T2, L);
            tri_tail_steps<2>(t, x, y, lane, rho, T2, L);
            tri_tail_steps<3>(t, x, y, lane, rho, T2, L);
            // T and the reflectors' beta: rows up to 126 from their steps; of the last 2 x 2 block the next column is e_126, and
            // the corner is in the last row's last column
            const int row = kTriTail + rho;
            if (row < kTriN - 1) {
                L[kTriDd + row] = T2[0];
                L[kTriEe + row - 1] = -T2[1];
                L[kTriBet + row - 1] = T2[2];
            } else if (lane == 63) {
                L[kTriDd + kTriN - 1] = t[15];
                L[kTriEe + kTriN - 2] = x;
                L[kTriEe + kTriN - 1] = 0.0;
                L[kTriBet + kTriN - 2] = 0.0;
                L[kTriBet + kTriN - 1] = 0.0;
            }
        } else {
            for (int e = tid - 64; e < (kTriN - 1 - kTriTail) * (kTriTail / 2); e += kTriThreads - 64) {
                const int k = e / (kTriTail / 2), m = e % (kTriTail / 2);
                *reinterpret_cast<double2*>(L + kTriX + (kTriTail - 1 + k) * kTriVLd + 2 * m) = double2{0.0, 0.0};
            }
            block_operands(wave - 1, wave == 1 ? 0 : 6 - wave);      // 0; 1, 4; 2, 3
        }
    }
    __syncthreads();
    if (wave < 3) block_operands(5 + wave, 5 + wave);
    __syncthreads();

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
    auto batch = [&](const int joff, const int rb) __attribute__((always_inline)) -> bool {
        // ---- 2. the rb largest eigenvalues, bracketed by Sturm counts.  A power-of-two team of threads per eigenvalue, a
        // trial shift each; every round keeps the part of the bracket between two neighbouring trial
        // shifts that holds the eigenvalue.  The trial shifts divide the bracket evenly while it holds several eigenvalues.
        // Once it holds one, the last minor (the characteristic polynomial) changes sign in it and its values at the two
        // ends and at the next shift are known: the shifts then sit around the zero of the linear fraction (x - z) / (a x + b)
        // through the three (of the line through the two where that falls outside), at distances that fall from 1/8 of
        // the bracket by equal factors to 2^-27 or less, so a round gains as many digits as that estimate has and the count
        // alone still decides.  A round whose estimate was no good (the bracket not an eighth) is followed by an even one.  5 to 7
        // rounds for 16 eigenvalues (16 shifts each), 8 to 10 for 32 (8 shifts each): 26 k and 34 k cycles, the shared round included.
        // (Even division throughout, 17 parts in 14 rounds: 75 k and 113 k; the zero of the line alone, 9 rounds: 53 k and 76 k with T
        // read from LDS, 36 k and 61 k with T in lanes.)
        double td[8], te[8];                                  // T for the counts: lane i of a row of 16 lanes holds rows 16 b + i
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const double2 t = *reinterpret_cast<const double2*>(L + kTriDe + 2 * (16 * b + mi));
            td[b] = t.x;
            te[b] = -t.y;
        }
        {
            // shared round: 256 shifts over [-kTriBound, kTriBound], one per thread, serve every eigenvalue
            const double x = fma(kTriPart, static_cast<double>(tid + 1), -kTriBound);
            double p1;
            int cnt, ex;
            tri_minors(td, te, x, p1, cnt, ex);
            L[kTriU0 + tid] = p1;
            reinterpret_cast<int2*>(L + kTriU1)[tid] = int2{cnt, ex};
            __syncthreads();
        }
        {
            const int team_log2 = rb > 16 ? 3 : (rb > 8 ? 4 : (rb > 4 ? 5 : 6)), points = 1 << team_log2, sub = tid & (points - 1);
            const int j = (tid >> team_log2) < rb ? tid >> team_log2 : rb - 1;     // (spare teams repeat the last: all lanes take part)
            const int half = points / 2, fall = 64 >> team_log2;
            const double inv_parts = 1.0 / (points + 1);
            const int below_target = kTriN - 1 - (joff + j);  // eigenvalue joff + j (descending) has this many below it
            const int lane0 = lane & ~(points - 1);
            const unsigned long long team_mask = points == 64 ? ~0ull : ((1ull << points) - 1ull) << lane0;
            // first bracket: from the counts of the shared round
            int first = 0;                                    // shared shifts with count <= target (a prefix)
            const int2* shared = reinterpret_cast<const int2*>(L + kTriU1);
            for (int step = kTriThreads / 2; step > 0; step >>= 1)
                if (shared[first + step - 1].x <= below_target) first += step;
            if (first == kTriThreads - 1 && shared[kTriThreads - 1].x <= below_target) first = kTriThreads;
            // the bracket, and the last minor at its ends, f 2^e, with the counts there
            double lo = fma(kTriPart, static_cast<double>(first), -kTriBound);
            double hi = fma(kTriPart, static_cast<double>(first + 1), -kTriBound);
            const int2 at_lo = shared[first > 0 ? first - 1 : 0], at_hi = shared[first < kTriThreads ? first : 0];
            bool known_lo = first > 0, known_hi = first < kTriThreads, stalled = false;
            double flo = L[kTriU0 + (known_lo ? first - 1 : 0)], fhi = L[kTriU0 + (known_hi ? first : 0)];
            int clo = at_lo.x, chi = at_hi.x, elo = at_lo.y, ehi = at_hi.y;
            // a third shift next to the bracket
            const int third = first >= 2 ? first - 2 : (first + 1 < kTriThreads ? first + 1 : first);
            double xt = fma(kTriPart, static_cast<double>(third + 1), -kTriBound), ft = L[kTriU0 + third];
            int et = shared[third].y;
            for (int round = 0; round < 24; ++round) {
                if (__ballot(hi - lo > kTriWidth) == 0ull) break;
                const double width = hi - lo, step = width * inv_parts;
                const bool line = known_lo && known_hi && chi - clo == 1 && !stalled;
                auto scale = [](int e) __attribute__((always_inline)) { return tri_pow2(e < -1000 ? -1000 : (e > 1000 ? 1000 : e)); };
                const double inv = tri_rcp(flo), rat_u = fhi * inv * scale(ehi - elo), rat_t = ft * inv * scale(et - elo);
                const double ct = xt - lo;
                double z = width * ct * (rat_u - rat_t) * tri_rcp(fma(ct * rat_t, rat_u - 1.0, width * rat_u * (1.0 - rat_t)));
                if (!(z > 0.0 && z < width)) z = width * tri_rcp(1.0 - rat_u);     // the zero of the line (rat_u < 0)
                const double est = lo + z;
                const int away = sub < half ? sub : points - 1 - sub;      // 0: farthest from the estimate
                const double dist = width * tri_pow2(-3 - fall * away);
                const double x = line ? fmin(fmax(est + (sub < half ? -dist : dist), lo), hi) : fma(step, static_cast<double>(sub + 1), lo);
                double p1;
                int cnt, ex;
                tri_minors(td, te, x, p1, cnt, ex);
                // the team's points are ascending: those with count <= target are a prefix
                const int nb = __popcll(__ballot(cnt <= below_target) & team_mask), exc = ex * 256 + cnt;
                const int pl = nb > 0 ? nb - 1 : 0, pu = nb < points ? nb : points - 1;
                auto pick = [&](int p, double& xo, double& fo, int& eco) __attribute__((always_inline)) {
                    xo = __shfl(x, lane0 + p, 64);
                    fo = __shfl(p1, lane0 + p, 64);
                    eco = __shfl(exc, lane0 + p, 64);
                };
                double xl, fl, xu, fu, xa, fa, xb, fb;
                int el, eu, ea, eb;
                pick(pl, xl, fl, el);
                pick(pu, xu, fu, eu);
                // the third shift: the nearer one of those next to the new bracket
                pick(nb >= 2 ? nb - 2 : nb + 1, xa, fa, ea);
                pick(nb + 1 < points ? nb + 1 : nb - 2, xb, fb, eb);
                if (nb > 0) { lo = xl; flo = fl; elo = el >> 8; clo = el & 255; known_lo = true; }
                if (nb < points) { hi = xu; fhi = fu; ehi = eu >> 8; chi = eu & 255; known_hi = true; }
                const bool below = lo - xa <= xb - hi && xa < lo;        // (at the ends of the range both are the same shift)
                xt = below ? xa : xb;
                ft = below ? fa : fb;
                et = (below ? ea : eb) >> 8;
                stalled = line && hi - lo > 0.125 * width;
            }
            if (sub == 0 && tid >> team_log2 == j) L[kTriLam + j] = 0.5 * (lo + hi);
        }
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
        // multiply-adds per row (5 k cycles; 8.6 k with T read from LDS and every pivot compared), and everything after it is
        // spread over all threads (eight per vector; 8 k).  The inverse iteration below, one lane per vector through two solves
        // with a reciprocal per row, took 48 us.  It is kept for eigenvalues closer than that, whose vectors come out of the twisted form
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
                double td2[8], te2[8];
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const double2 t = *reinterpret_cast<const double2*>(src + 2 * (16 * b + mi));
                    td2[b] = t.x;
                    te2[b] = -t.y;
                }
                double p0 = 0.0, p1 = 1.0;
                auto eight = [&](int b, auto hi_tag) __attribute__((always_inline)) {
                    constexpr bool HI = decltype(hi_tag)::value;
                    double p[8];
                    tri_eight<HI, true>(p, p0, p1, -lam, td2[b], te2[b], kTriPivMin);
#pragma unroll
                    for (int u = 0; u < 8; ++u) dst[32 * (16 * b + (HI ? 8 : 0) + u)] = p[u];
                    p0 = p[6];
                    p1 = p[7];
                    tri_rescale(p0, p1);                      // (the stored minors keep the old scale: redone below)
                };
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    eight(b, std::false_type{});
                    eight(b, std::true_type{});
                }
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
        // (An offset the compiler does not know: hundreds of constant addresses of S, past the reach of an LDS instruction's
        // offset, would be formed in front of the rare paths below and spilled, 3.5 k cycles of it.)
        int s_off = kTriS;
        asm("" : "+v"(s_off));
        double* S = L + s_off;
        bool ok = true;
        for (int pass = 0; pass < 3; ++pass) {
            // every wavefront takes 32 rows of the 16 x 16 tiles (0, 0), (0, 1), (1, 1), wavefront t adds up tile t; only the rb
            // real columns count (the padding columns are never used).  (A tile per wavefront over all rows: twice as long.)
            double dev = 0.0;
            const int tiles = rb > 16 ? 3 : 1;
            double* part = L + kTriU0;                        // [4 wavefronts][3 tiles][4][64]
            {
                double4v acc[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) acc[t] = double4v{0.0, 0.0, 0.0, 0.0};
                const double* xs = L + kTriX + 32 * (32 * wave + mk) + mi;
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const double x0 = xs[32 * 4 * m], x1 = xs[32 * 4 * m + 16];
                    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x0, acc[0], 0, 0, 0);
                    if (tiles > 1) {                          // uniform
                        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x1, acc[1], 0, 0, 0);
                        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x1, acc[2], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    if (t < tiles) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) part[((3 * wave + t) * 4 + q) * 64 + lane] = acc[t][q];
                    }
            }
            __syncthreads();
            if (wave < tiles) {                               // uniform
                const int ti = wave >> 1, tj = wave > 0 ? 1 : 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i2 = 16 * ti + mk + 4 * q, j2 = 16 * tj + mi;
                    const double* pq = part + (4 * wave + q) * 64 + lane;
                    const double g2 = (pq[0] + pq[768]) + (pq[1536] + pq[2304]);
                    S[i2 * 33 + j2] = g2;
                    if (ti != tj) S[j2 * 33 + i2] = g2;
                    if (i2 < rb && j2 < rb) {
                        const double d2 = fabs(g2 - (i2 == j2 ? 1.0 : 0.0));
                        dev = d2 == d2 ? fmax(dev, d2) : 1e300;
                    }
                }
            }
            // (a power of the deviation is all that matters: one bit per wavefront and threshold)
            {
                const int mine = (__ballot(!(dev < 1e300)) ? 1 : 0) | (__ballot(!(dev <= 1e-5)) ? 2 : 0) |
                                 (__ballot(!(dev <= kTriAccept)) ? 4 : 0) | (__ballot(!(dev <= 1e-10)) ? 8 : 0);
                int* flags = reinterpret_cast<int*>(misc + 36);
                if (lane == 0) flags[wave] = mine;
            }
            __syncthreads();
            const int dev_flags = reinterpret_cast<const int*>(misc + 36)[0] | reinterpret_cast<const int*>(misc + 36)[1] |
                                  reinterpret_cast<const int*>(misc + 36)[2] | reinterpret_cast<const int*>(misc + 36)[3];
            if (dev_flags & 1) ok = false;
            if (!(dev_flags & 8) || !ok) break;
            if (pass == 2) {
                ok = !(dev_flags & 4);
                break;
            }
            if (!(dev_flags & 2)) {
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

        // the operands of step 5 are on their way during steps 3 and 4
        double2 va[4][2], ma[4][2], vb[8][2], mb[8][2];
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (b <= 7 - wave) {                          // uniform
                    vb[b][q] = vmine[(b * 4 + q) * 64 + lane];
                    mb[b][q] = vmine[(b * 4 + 2 + q) * 64 + lane];
                }
                if (b < 4 && b <= wave) {
                    va[b & 3][q] = vmine[((8 - wave + b) * 4 + q) * 64 + lane];
                    ma[b & 3][q] = vmine[((8 - wave + b) * 4 + 2 + q) * 64 + lane];
                }
            }

        // ---- 4. Rayleigh quotients and residuals: thread (j, sg) takes rows 16 sg .. 16 sg + 15 of vector j
        {
            constexpr int RS = kTriN / 8;
            const int j = tid & 31, sg = tid >> 5, r0 = RS * sg;
            double* P = S;                                    // (the Gram matrix has served)
            double xv[RS + 2], yv[RS], num = 0.0, den = 0.0;
#pragma unroll
            for (int i = 0; i < RS; ++i) xv[i + 1] = L[kTriX + 32 * (r0 + i) + j];
            xv[0] = sg > 0 ? L[kTriX + 32 * (r0 - 1) + j] : 0.0;
            xv[RS + 1] = sg < 7 ? L[kTriX + 32 * (r0 + RS) + j] : 0.0;
            double eprev = sg > 0 ? L[kTriEe + r0 - 1] : 0.0;
            __syncthreads();                                  // everyone is past the Gram matrix
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                const double e = L[kTriEe + r0 + i];          // (0 in the last row)
                yv[i] = fma(L[kTriDd + r0 + i], xv[i + 1], fma(eprev, xv[i], e * xv[i + 2]));
                eprev = e;
                num = fma(xv[i + 1], yv[i], num);
                den = fma(xv[i + 1], xv[i + 1], den);
            }
            P[tid] = num;
            P[256 + tid] = den;
            __syncthreads();
            num = den = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                num += P[32 * q + j];
                den += P[256 + 32 * q + j];
            }
            const double rq = den > 0.0 ? num / den : 0.0;
            double res = 0.0;
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                const double t = fma(-rq, xv[i + 1], yv[i]);
                res = fma(t, t, res);
            }
            P[512 + tid] = res;
            if (sg == 0) L[kTriLam + 64 + j] = rq;
            __syncthreads();
            res = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) res += P[512 + 32 * q + j];
            const double w = j < rb ? sqrt(res) : 0.0;
            // every wavefront sees all 32 vectors
            if (__ballot(!(w <= kTriAccept)) != 0ull || SQUAT_TRI_REFUSED(aexp)) ok = false;
        }
        if (!ok) return false;                                // uniform: every thread saw the same flags

        // ---- 5. back-transformation, X <- (I - V T V') X block by block from the last, on the matrix cores; NC column tiles of
        // 16 vectors.  A wavefront's part of V'X over its own rows goes to LDS, every wavefront adds up the parts (in the same
        // order) and applies the product to its rows.  One barrier per block: 144 products of 64 cycles and eight exchanges
        // per wavefront for 32 vectors.  (One reflector after the other, with a dot product over 16 lanes each, took 55 k
        // cycles for 16 vectors and 90 k for 32, and the reflectors a trip through global memory; this takes 15 k and 32 k
        // with the output.)
        auto back = [&](auto nc_tag) __attribute__((always_inline)) {
            constexpr int NC = decltype(nc_tag)::value;
            const int tb = 7 - wave;
            double4v xa[NC], xb[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    xa[c][q] = L[kTriX + 32 * (16 * wave + mk + 4 * q) + 16 * c + mi];
                    xb[c][q] = L[kTriX + 32 * (16 * tb + mk + 4 * q) + 16 * c + mi];
                }
            __syncthreads();
            double* Z = L + kTriX;                            // [2][4 wavefronts][NC][4][64]
#pragma unroll
            for (int b = 7; b >= 0; --b) {
                const bool on_b = b <= tb, on_a = b < 4 && b <= wave;        // uniform; on_a implies on_b
                constexpr int kWaves = kTriThreads / 64;
                const int parts = b >= 4 ? 8 - b : kWaves;    // wavefronts 0 .. parts - 1 have a part
                double* zw = Z + (b & 1) * (kWaves * NC * 256);
                if (on_b) {
                    double4v z[NC];
#pragma unroll
                    for (int c = 0; c < NC; ++c) z[c] = double4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int c = 0; c < NC; ++c) z[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q & 1 ? vb[b][q / 2].y : vb[b][q / 2].x, xb[c][q], z[c], 0, 0, 0);
                    if (on_a) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int c = 0; c < NC; ++c) z[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q & 1 ? va[b & 3][q / 2].y : va[b & 3][q / 2].x, xa[c][q], z[c], 0, 0, 0);
                    }
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int q = 0; q < 4; ++q) zw[((wave * NC + c) * 4 + q) * 64 + lane] = z[c][q];
                }
                tri_lds_barrier();
                if (on_b) {
                    double zs[NC][4];
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int q = 0; q < 4; ++q) zs[c][q] = zw[(c * 4 + q) * 64 + lane];
#pragma unroll
                    for (int w = 1; w < kWaves; ++w)
                        if (w < parts) {
#pragma unroll
                            for (int c = 0; c < NC; ++c)
#pragma unroll
                                for (int q = 0; q < 4; ++q) zs[c][q] += zw[((w * NC + c) * 4 + q) * 64 + lane];
                        }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int c = 0; c < NC; ++c) {
                            xb[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q & 1 ? mb[b][q / 2].y : mb[b][q / 2].x, zs[c][q], xb[c], 0, 0, 0);
                            if (on_a) xa[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q & 1 ? ma[b & 3][q / 2].y : ma[b & 3][q / 2].x, zs[c][q], xa[c], 0, 0, 0);
                        }
                }
            }
            // to LDS, vector by vector (behind the exchange buffers)
            constexpr int OLd = kTriN + 1;
            double* O = L + kTriX + 2 * 4 * 2 * 256;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    O[(16 * c + mi) * OLd + 16 * wave + mk + 4 * q] = xa[c][q];
                    O[(16 * c + mi) * OLd + 16 * tb + mk + 4 * q] = xb[c][q];
                }
            __syncthreads();

            // ---- output: team of 16 lanes per vector; rank by eigenvalue, sign so that the largest component is positive, rows
            // sqrt(lambda) v
            const int bs = tid & 15;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int vj = (tid >> 4) + 16 * c;
                if (vj >= rb) continue;                       // uniform per team of 16 lanes
                const double lam = L[kTriLam + 64 + vj];
                int before = 0;
#pragma unroll
                for (int o = bs; o < 32; o += 16) {
                    const double lo = L[kTriLam + 64 + o];
                    before += o < rb && ((lo > lam) || (lo == lam && o < vj));
                }
                double x[8], best = -1.0, bestv = 0.0;
                int besti = kTriN;
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    x[m] = O[vj * OLd + bs + 16 * m];
                    const double av = fabs(x[m]);
                    if (av > best) { best = av; bestv = x[m]; besti = bs + 16 * m; }
                }
#pragma unroll
                for (int off = 8; off > 0; off >>= 1) {
                    before += __shfl_xor(before, off, 64);
                    const double ob = __shfl_xor(best, off, 64);
                    const double ov = __shfl_xor(bestv, off, 64);
                    const int oi = __shfl_xor(besti, off, 64);
                    if (ob > best || (ob == best && oi < besti)) { best = ob; bestv = ov; besti = oi; }
                }
                const double lam_true = fmax(lam, 0.0) * tmax * up;
                const double sc = (bestv < 0.0 ? -1.0 : 1.0) * sqrt(lam_true);
                float* dst = qhat + (joff + before) * kTriN;
#pragma unroll
                for (int m = 0; m < 8; ++m) dst[bs + 16 * m] = static_cast<float>(x[m] * sc);
                if (eig && bs == 0) eig[joff + before] = static_cast<float>(lam_true);
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
