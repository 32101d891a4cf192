// squat_prepare: the per-head update matrix U of Lemma 2 / Lemma 3 of the paper,
//     U[t g :, (t-1) g : t g] = B_t H_t,    t = 1 .. d/g - 1.
// Eliminating the free tail of Lemma 2's problem gives B_t H_t = -P[tg:,tg:]^{-1} P[tg:,blk]
// with P = I + lambda Qhat^T Qhat, and the Woodbury identity (the paper's O(r d^2) footnote)
// reduces this to an r x r problem:
//     W_t = -Qr^T (I/lambda + Qr Qr^T)^{-1} Qb,     Qb = Qhat[:, blk], Qr = Qhat[:, tg:].
// r <= 64 and finite lambda: block elimination in fp64 on the matrix cores, a workgroup or more per panel
// (prepare_elim_kernel).  All else, and the heads that kernel flags: one workgroup per (head, t) or per head works
// in fp64, forms S = I/lambda + Qr Qr^T, diagonalises it with the one-sided Jacobi routine (rows a_i = mu_i v_i), and applies
// S^+ = sum_i a_i a_i^T / mu_i^3.  lambda = +inf drops the I/lambda term and discards the
// (numerically) zero mu_i, which yields -pinv(Qr) Qb.  By default the result is stored as fp32 numbers that
// are exactly representable in fp16; squat_prepare_ex can store the plain fp32 rounding instead.
#include <math.h>

#include "squat_internal.h"
#include "squat_jacobi.h"

using namespace squat;

// Scratch of squat_prepare_noalloc: lives in the code object, one copy per device that loads the library,
// for the life of the process.  In host code this name only stands for the symbol; the device address is
// looked up once per device (scratch_address below) and the kernels get that pointer.
constexpr size_t kStaticScratchBytes = size_t(4) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kPrepThreads = 1024;

struct PrepParams {
    const float* qhat;    // [heads][r][d]
    float* update;        // [heads][d][d]
    double* ws;           // per workgroup: y [rp][g] then z [rp][d]
    int r, rp, g, nsteps; // rp = r rounded up to even
    int nprob;            // heads * nsteps
    double inv_lambda;    // 0 for lambda = +inf
    int hard;
    int full;             // 1: store the fp32 rounding of the fp64 result; 0: round it to the fp16 grid first
};

// The stored form of an entry of U.  On the fp16 grid (relative 2^-12) the quantize kernels contract with two
// fp16 matrix passes instead of three.
__device__ __forceinline__ float stored_entry(double v, int full) {
    const float f = static_cast<float>(v);
    return full ? f : static_cast<float>(static_cast<_Float16>(f));
}

__global__ void __launch_bounds__(256) zero_fill(float* p, int64_t n4) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n4) reinterpret_cast<f32x4*>(p)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// A head's flag: a byte per panel from the elimination kernel, 1 when the eigen route has seen it (whoever reads it meanwhile
// sees a number other than zero either way).
__device__ __forceinline__ int flagged_head(int* need) {
    const int f = *need;
    if (f != 0 && threadIdx.x == 0) *need = 1;
    return f;
}

// Large r (> 32; up to 64 with a finite lambda only for the heads the elimination kernel flags): one 1024-thread
// workgroup per (head, t) panel; intermediate products go through the global workspace.
template <int TS>
__global__ void __launch_bounds__(kPrepThreads) prepare_kernel(const PrepParams p, int* need) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    if (need && flagged_head(need + blockIdx.x / p.nsteps) == 0) return;       // done by the elimination kernel
    constexpr int THREADS = kPrepThreads;
    const int r = p.r, rp = p.rp, g = p.g;
    double* S = reinterpret_cast<double*>(smem);     // rp x rp
    double* mu = S + rp * rp;                         // rp
    int* flag = reinterpret_cast<int*>(mu + rp);
    const int head = blockIdx.x / p.nsteps;
    const int t = blockIdx.x % p.nsteps + 1;          // 1 .. d/g - 1
    const int c0 = t * g;                             // first remaining channel
    const int nrest = kD - c0;
    const float* Q = p.qhat + static_cast<int64_t>(head) * r * kD;
    double* y = p.ws + static_cast<int64_t>(blockIdx.x) * rp * (g + kD);
    double* z = y + rp * g;
    const int tid = threadIdx.x;

    // S = I/lambda + Qr Qr^T  (padded row/column rp-1 is zero when r is odd)
    for (int idx = tid; idx < rp * rp; idx += THREADS) {
        const int i = idx / rp, k = idx % rp;
        double s = 0.0;
        if (i < r && k < r) {
            for (int c = c0; c < kD; ++c) s += static_cast<double>(Q[i * kD + c]) * static_cast<double>(Q[k * kD + c]);
            if (i == k) s += p.inv_lambda;
        }
        S[idx] = s;
    }
    __syncthreads();
    jacobi_rows<THREADS, TS, (kD + TS - 1) / TS, false>(S, rp, rp, mu, flag, 60, 1e-13);
    __syncthreads();

    if (tid < rp) {
        double s = 0.0;
        for (int c = 0; c < rp; ++c) s += S[tid * rp + c] * S[tid * rp + c];
        mu[tid] = sqrt(s);
    }
    __syncthreads();
    double mumax = 0.0;
    for (int i = 0; i < rp; ++i) mumax = fmax(mumax, mu[i]);
    // pseudo-inverse cut: with a finite lambda every true mu_i >= 1/lambda, so only the
    // padding row falls below it
    const double cut = p.hard ? mumax * 1e-12 : 0.5 * p.inv_lambda;

    // y_i[j] = a_i . Qb[:, j] / mu_i^3 ;  z_i[c] = sum_k Qr[k, c] a_i[k]
    for (int idx = tid; idx < rp * g; idx += THREADS) {
        const int i = idx / g, j = idx % g;
        double s = 0.0;
        const double m = mu[i];
        if (m > cut && m > 0.0) {
            for (int k = 0; k < r; ++k) s += S[i * rp + k] * static_cast<double>(Q[k * kD + (c0 - g) + j]);
            s /= (m * m * m);
        }
        y[idx] = s;
    }
    for (int idx = tid; idx < rp * nrest; idx += THREADS) {
        const int i = idx / nrest, c = idx % nrest;
        double s = 0.0;
        for (int k = 0; k < r; ++k) s += S[i * rp + k] * static_cast<double>(Q[k * kD + c0 + c]);
        z[i * kD + c] = s;
    }
    __threadfence_block();
    __syncthreads();
    // W[c][j] = - sum_i z_i[c] y_i[j]
    float* U = p.update + static_cast<int64_t>(head) * kD * kD;
    for (int idx = tid; idx < nrest * g; idx += THREADS) {
        const int c = idx / g, j = idx % g;
        double s = 0.0;
        for (int i = 0; i < rp; ++i) s += z[i * kD + c] * y[i * g + j];
        U[(c0 + c) * kD + (c0 - g) + j] = stored_entry(-s, p.full);
    }
}

// r <= 32 (the paper's usual range): one workgroup per head, one WAVEFRONT per panel t.  The r x r
// Jacobi then needs no workgroup barrier (it is bound by synchronisation latency, not arithmetic), the
// head's Qhat is staged once in LDS as fp32, and all intermediates stay in LDS:
//   X = S^+ Qb = sum_i a_i (a_i . Qb) / mu_i^3   (rp x g),      W = -Qr^T X.
__global__ void __launch_bounds__(192) prepare_wave_kernel(const PrepParams p, int* need) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    if (need && flagged_head(need + blockIdx.x) == 0) return;                  // done by the elimination kernel
    const int r = p.r, rp = p.rp, g = p.g;
    constexpr int QLD = kD + 1;       // odd row stride: column reads across rows hit distinct LDS banks
    const int ld = rp + 2;            // padded row: teams of 4 lanes read different rows at the same column
    const int head = blockIdx.x;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float* Qf = reinterpret_cast<float*>(smem);                          // [rp][128]
    const size_t per = (static_cast<size_t>(rp) * ld + rp + 2 + 2 * static_cast<size_t>(rp) * g) * sizeof(double);
    double* S = reinterpret_cast<double*>(smem + ((static_cast<size_t>(rp) * QLD * sizeof(float) + 15) & ~size_t(15)) + wave * per);
    double* mu = S + rp * ld;
    int* flag = reinterpret_cast<int*>(mu + rp);
    double* y = mu + rp + 2;                                             // [rp][g]
    double* X = y + rp * g;                                              // [rp][g]
    const float* Q = p.qhat + static_cast<int64_t>(head) * r * kD;
    for (int idx = threadIdx.x; idx < rp * kD; idx += blockDim.x)
        Qf[(idx >> 7) * QLD + (idx & 127)] = idx < r * kD ? Q[idx] : 0.0f;
    __syncthreads();

    const int t = wave + 1;
    const int c0 = t * g, nrest = kD - c0;
    for (int idx = lane; idx < rp * rp; idx += 64) {
        const int i = idx / rp, k = idx % rp;
        double s = (i == k && i < r) ? p.inv_lambda : 0.0;
        for (int c = c0; c < kD; ++c) s = fma(static_cast<double>(Qf[i * QLD + c]), static_cast<double>(Qf[k * QLD + c]), s);
        S[i * ld + k] = s;
    }
    team_sync<64>();
    jacobi_rows<64, 4, 8, false>(S, rp, ld, mu, flag, 60, 1e-13);
    team_sync<64>();
    for (int i = lane; i < rp; i += 64) {
        double s = 0.0;
        for (int c = 0; c < rp; ++c) s = fma(S[i * ld + c], S[i * ld + c], s);
        mu[i] = sqrt(s);
    }
    team_sync<64>();
    double mumax = 0.0;
    for (int i = 0; i < rp; ++i) mumax = fmax(mumax, mu[i]);
    const double cut = p.hard ? mumax * 1e-12 : 0.5 * p.inv_lambda;
    for (int idx = lane; idx < rp * g; idx += 64) {
        const int i = idx / g, j = idx % g;
        double s = 0.0;
        const double m = mu[i];
        if (m > cut && m > 0.0) {
            for (int k = 0; k < rp; ++k) s = fma(S[i * ld + k], static_cast<double>(Qf[k * QLD + (c0 - g) + j]), s);
            s /= (m * m * m);
        }
        y[idx] = s;
    }
    team_sync<64>();
    for (int idx = lane; idx < rp * g; idx += 64) {
        const int k = idx / g, j = idx % g;
        double s = 0.0;
        for (int i = 0; i < rp; ++i) s = fma(S[i * ld + k], y[i * g + j], s);
        X[idx] = s;
    }
    team_sync<64>();
    float* U = p.update + static_cast<int64_t>(head) * kD * kD;
    for (int idx = lane; idx < nrest * g; idx += 64) {
        const int c = idx / g, j = idx % g;
        double s = 0.0;
        for (int k = 0; k < rp; ++k) s = fma(static_cast<double>(Qf[k * QLD + c0 + c]), X[k * g + j], s);
        U[(c0 + c) * kD + (c0 - g) + j] = stored_entry(-s, p.full);
    }
}

// r <= 64 and finite lambda: S = I/lambda + Qr Qr^T is positive definite with smallest eigenvalue
// >= 1/lambda, so X = S^-1 Qb comes from Gauss-Jordan elimination of [S | Qb] without pivoting (the pivots are those of
// the Cholesky factorisation) instead of an eigen-decomposition.  One workgroup of four wavefronts per panel, or several that
// share the panel's columns; everything lives in the result layout of v_mfma_f64_16x16x4_f64 (lane (j = lane & 15, m = lane >> 4),
// register q: row m + 4 q, column j of a 16 x 16 tile), NT row tiles, the column tiles dealt out to the wavefronts:
//   - S: products of the rows of Qr on the matrix cores (fp32 entries of Qhat widened on the way);
//   - four pivots a step: their columns go through LDS to every wavefront (one barrier, two buffers), every lane factors
//     the 4 x 4 pivot block, the pivot rows are in the same wavefront for every column, and the update is one product per
//     live 16 x 16 tile;
//   - W = -Qr^T X: the solution's registers are the B operands as they are, through LDS to all four wavefronts.
// Bound by the chain of its steps (LDS exchange, four reciprocals, two dependent products): 32 heads, r = 40, g = 64, one column
// tile per wavefront, 2.6 k cycles for loading, 4.9 k for S, 14.8 k for ten steps, 2.5 k for W.  us per
// launch, fallback launch included, against all panels of a head in one workgroup (results of the products in the
// accumulation registers, rows of Qhat 129 floats apart, four bytes a load): 32 heads, g = 32: r = 16 11.5 -> 8.7, 32 19.9 -> 12.9, 40 27.8 -> 14.9, 64 40.0 -> 21.1; g = 64: r = 16 10.2 -> 8.2, 40 19.5 -> 13.5, 64 26.7 -> 19.5;
// 256 heads: g = 32, r = 16 13.7 -> 12.8, 64 43.2 -> 40.4, g = 64, r = 40 22.8 -> 19.8.
// A panel whose pivots span more than 1e9 (lambda times the largest eigenvalue of Qr Qr^T that large)
// sets the head's flag: the eigen-route kernel, launched afterwards, redoes exactly the flagged heads.
typedef double double4v __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));       // 16 bytes at any float's address

constexpr int kElimThreads = 256;           // four wavefronts
constexpr int kElimQLd = kD + 4;            // rows 4 banks apart: the 16 rows x 4 channels of an operand of S lie in 64 banks

constexpr size_t elim_lds_bytes(int nt, int per) {
    // Qhat as fp32; two blocks of four columns in flight, later the solution's tiles (50 KB at r = 64, g = 32: three workgroups
    // on a compute unit, as many as a head has panels)
    return static_cast<size_t>(16 * nt) * kElimQLd * sizeof(float) + static_cast<size_t>(per * 256 > 128 ? per * 256 : 128) * nt * sizeof(double);
}

// One workgroup per (head, panel t - 1, group of `per` column tiles of Qb).  need: four bytes per head, one per panel.
template <int NT>
__global__ void __launch_bounds__(kElimThreads) prepare_elim_kernel(const PrepParams p, const int per, unsigned char* need) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int RP = 16 * NT;
    const int r = p.r, g = p.g;
    const int head = blockIdx.x, panel = blockIdx.y, tid = threadIdx.x;
    const int lane = tid & 63, mi = lane & 15, mk = lane >> 4;
    const int wt = __builtin_amdgcn_readfirstlane(tid >> 6);                             // this wavefront's column tiles: wt, wt + 4
    const int c0 = (panel + 1) * g, nrest = kD - c0;
    const int j0 = c0 - g + 16 * per * blockIdx.z;                                       // first column of Qb here
    const int ctiles = NT + per;
    float* Qf = reinterpret_cast<float*>(smem);                                          // [RP][132]
    double* cols = reinterpret_cast<double*>(smem + RP * kElimQLd * sizeof(float));
    double* Xs = cols;                                                                   // [per][4 NT][64], after the elimination
    const float* Q = p.qhat + static_cast<int64_t>(head) * r * kD;
    float* U = p.update + static_cast<int64_t>(head) * kD * kD;
    {
        // all of a thread's loads before the first is used
        f32x4 v[2 * NT];
#pragma unroll
        for (int i = 0; i < 2 * NT; ++i) {
            const int idx = 4 * (tid + kElimThreads * i);
            v[i] = *reinterpret_cast<const f32x4_any*>(Q + (idx < r * kD ? idx : 0));       // (rows from r on: zeros below)
        }
#pragma unroll
        for (int i = 0; i < 2 * NT; ++i) {
            const int idx = 4 * (tid + kElimThreads * i);
            *reinterpret_cast<f32x4*>(Qf + (idx >> 7) * kElimQLd + (idx & 127)) = idx < r * kD ? v[i] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // Everything of this head's matrix outside the panels is zero: row i from the start of its own block of g
    // columns on (the panels, written at the end or by the eigen route, are the columns before it).  The head's workgroups share it.
    {
        const int unit = blockIdx.y + gridDim.y * blockIdx.z, units = gridDim.y * gridDim.z;
        for (int idx = tid + kElimThreads * unit; idx < kD * (kD / 4); idx += kElimThreads * units) {
            const int row = idx / (kD / 4), col = 4 * (idx % (kD / 4));
            if (col >= row / g * g) *reinterpret_cast<f32x4*>(U + row * kD + col) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");                      // (the stores above are not waited for)

    // ---- [S | Qb]
    double a[2][NT][4];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int ct = wt + 4 * s;
#pragma unroll
        for (int ti = 0; ti < NT; ++ti)
#pragma unroll
            for (int q = 0; q < 4; ++q) a[s][ti][q] = 0.0;
        if (s == 0 && ct < NT) {                          // uniform; (NT <= 4: the tiles of S are all in slot 0)
            double4v acc[NT];
#pragma unroll
            for (int ti = 0; ti < NT; ++ti) acc[ti] = double4v{0.0, 0.0, 0.0, 0.0};
            const float* qc = Qf + (16 * ct + mi) * kElimQLd + c0 + mk;
            const float* qr = Qf + mi * kElimQLd + c0 + mk;
#pragma unroll 8
            for (int c = 0; c < nrest; c += 4) {
                const double bq = static_cast<double>(qc[c]);
#pragma unroll
                for (int ti = 0; ti < NT; ++ti)
                    acc[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(qr[16 * ti * kElimQLd + c]), bq, acc[ti], 0, 0, 0);
            }
#pragma unroll
            for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = 16 * ti + mk + 4 * q;
                    // rows / columns >= r: the identity
                    a[0][ti][q] = acc[ti][q] + (row == 16 * ct + mi ? (row < r ? p.inv_lambda : 1.0) : 0.0);
                }
        } else if (ct < ctiles) {
#pragma unroll
            for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    a[s][ti][q] = static_cast<double>(Qf[(16 * ti + mk + 4 * q) * kElimQLd + j0 + 16 * (ct - NT) + mi]);
        }
    }

    // ---- elimination, four pivots at a time: rows 16 kt + 4 kq .. + 3 are register kq of the row tile kt, i.e. the four pivot
    // rows R of a column tile are a B operand as they are.  [..] <- P^-1 R for the pivot block P, and A - C (P^-1 R) for the rest
    double pmin = 1e300, pmax = 0.0;
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) {
        const bool live0 = wt >= kt && wt < ctiles, live1 = wt + 4 < ctiles;             // uniform (tiles of S before kt are done)
#pragma unroll
        for (int kq = 0; kq < 4; ++kq) {
            const int k0 = 16 * kt + 4 * kq;
            if (k0 >= r) continue;                        // uniform: the rows from r on are the identity already
            double* col = cols + (kq & 1) * 4 * RP;       // [4 columns][row 16 t + m + 4 q at 16 t + 4 m + q]
            if (wt == kt && (mi >> 2) == kq) {
                double* dst = col + (mi & 3) * RP + 4 * mk;
#pragma unroll
                for (int ti = 0; ti < NT; ++ti) {
                    *reinterpret_cast<double2*>(dst + 16 * ti) = double2{a[0][ti][0], a[0][ti][1]};
                    *reinterpret_cast<double2*>(dst + 16 * ti + 2) = double2{a[0][ti][2], a[0][ti][3]};
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            // the pivot block (its lower triangle: row k0 + i, column k0 + j)
            const double* pb = col + 16 * kt + kq;
            double p[4][4], cm[NT];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = j; i < 4; ++i) p[i][j] = pb[j * RP + 4 * i];
#pragma unroll
            for (int ti = 0; ti < NT; ++ti) cm[ti] = -col[mk * RP + 16 * ti + 4 * (mi & 3) + (mi >> 2)];
            // P = L D L', every lane; then column mk of P^-1
            double d[4], l[4][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // 1 / pivot from the hardware approximation (good to 5e-8) and the series in its error up to the cube
                const double piv = p[j][j];
                double y = __builtin_amdgcn_rcp(piv);
                const double e = fma(-piv, y, 1.0);
                y = fma(y, fma(e, e, e), y);
                d[j] = y;
                if (k0 + j < r) {                         // uniform
                    pmin = fmin(pmin, piv);
                    pmax = fmax(pmax, piv);
                }
#pragma unroll
                for (int i = j + 1; i < 4; ++i) l[i][j] = p[i][j] * y;
#pragma unroll
                for (int j2 = j + 1; j2 < 4; ++j2)
#pragma unroll
                    for (int i = j2; i < 4; ++i) p[i][j2] = fma(-l[i][j], p[j2][j], p[i][j2]);
            }
            double x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[i] = mk == i ? 1.0 : 0.0;
#pragma unroll
                for (int j = 0; j < i; ++j) x[i] = fma(-l[i][j], x[j], x[i]);
            }
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                x[i] *= d[i];
#pragma unroll
                for (int j = i + 1; j < 4; ++j) x[i] = fma(-l[j][i], x[j], x[i]);
            }
            const double inv_op = mi == 0 ? x[0] : (mi == 1 ? x[1] : (mi == 2 ? x[2] : (mi == 3 ? x[3] : 0.0)));
            const double4v zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (!(s == 0 ? live0 : live1)) continue;  // uniform
                const double4v rs = __builtin_amdgcn_mfma_f64_16x16x4f64(inv_op, a[s][kt][kq], zero, 0, 0, 0);
#pragma unroll
                for (int ti = 0; ti < NT; ++ti) {
                    double4v t = {a[s][ti][0], a[s][ti][1], a[s][ti][2], a[s][ti][3]};
                    t = __builtin_amdgcn_mfma_f64_16x16x4f64(cm[ti], rs[0], t, 0, 0, 0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) a[s][ti][q] = t[q];
                }
                a[s][kt][kq] = rs[0];
            }
        }
    }
    const int bad = __builtin_amdgcn_readfirstlane(pmin > 1e-9 * pmax ? 0 : 1);           // (every lane saw the same pivots)
    if (blockIdx.z == 0 && tid < 4 && (tid == panel || (panel == 0 && tid >= static_cast<int>(gridDim.y))))
        need[4 * static_cast<int64_t>(head) + tid] = tid == panel ? bad : 0;
    if (bad) return;                                       // uniform: leave this head to the eigen route

    // ---- W_t[c][j] = -sum_k Q[k][c0 + c] X[k][j]: the solution's tiles through LDS, (tile, 16 rows c) dealt out to the wavefronts
    asm volatile("s_barrier" ::: "memory");                // everyone has read the last columns
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int ct = wt + 4 * s;
        if (ct < NT || ct >= ctiles) continue;             // uniform
#pragma unroll
        for (int ti = 0; ti < NT; ++ti)
#pragma unroll
            for (int q = 0; q < 4; ++q) Xs[((ct - NT) * 4 * NT + 4 * ti + q) * 64 + lane] = a[s][ti][q];
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int rows = nrest / 16;
    for (int item = wt; item < per * rows; item += 4) {    // uniform
        const int jt = item / rows, c = 16 * (item % rows);
        const double* xs = Xs + jt * 4 * NT * 64 + lane;
        double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 4 * NT; ++k)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(Qf[(4 * k + mk) * kElimQLd + c0 + c + mi]), xs[64 * k], acc, 0, 0, 0);
        float* dst = U + j0 + 16 * jt + mi;
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[(c0 + c + mk + 4 * q) * kD] = stored_entry(-acc[q], p.full);
    }
}

int team_size(int rp) {
    int ts = 64;
    while (ts > 1 && (rp / 2) * ts > kPrepThreads) ts >>= 1;
    return ts;
}

}  // namespace

extern "C" size_t squat_prepare_workspace(int n_heads, int d, int r, int g) {
    if (d != kD || n_heads < 1 || r < 0 || r > d || (g != 32 && g != 64 && g != 128)) return 0;
    const int nsteps = d / g - 1;
    const int rp = (r + 1) & ~1;
    const size_t per = static_cast<size_t>(rp) * (g + kD) * sizeof(double);
    const size_t total = ((static_cast<size_t>(n_heads) * nsteps * per + 255) & ~size_t(255)) +
                         ((static_cast<size_t>(n_heads) * sizeof(int) + 255) & ~size_t(255));   // + one flag per head
    return total < 256 ? 256 : total;
}

namespace {

// Bytes of the two scratch pieces a call uses: `yz` (intermediate products of the r > 32 kernel) and
// `flags` (one int per head, written by the elimination kernel and read by the eigen-route kernel that follows
// it).  Both are fully written before they are read, so neither needs clearing.
struct PrepScratch {
    size_t yz_bytes, flag_bytes;
};
PrepScratch prep_scratch(int n_heads, int r, int g, bool hard) {
    const int nsteps = kD / g - 1;
    const int rp = (r + 1) & ~1;
    PrepScratch out{0, 0};
    if (rp > 32)
        out.yz_bytes = (static_cast<size_t>(n_heads) * nsteps * rp * (g + kD) * sizeof(double) + 255) & ~size_t(255);
    if (!hard && rp <= 64)
        out.flag_bytes = (static_cast<size_t>(n_heads) * sizeof(int) + 255) & ~size_t(255);
    return out;
}

int prepare_impl(const float* qhat, int n_heads, int r, float lambda, int g, unsigned flags_arg, float* update,
                 double* yz, int* flags, hipStream_t s) {
    const int nsteps = kD / g - 1;
    const bool trivial = (r == 0 || lambda == 0.0f || nsteps == 0);
    // The elimination kernel clears its heads' matrices itself; every other route starts from a cleared tensor.
    const bool elim_route = !trivial && r <= 64 && !isinf(lambda);
    int rc = SQUAT_OK;
    if (!elim_route) {
        const int64_t n4 = static_cast<int64_t>(n_heads) * kD * kD / 4;
        hipLaunchKernelGGL(zero_fill, dim3(static_cast<unsigned>((n4 + 255) / 256)), dim3(256), 0, s, update, n4);
        rc = check_launch();
    }
    if (rc || trivial) return rc;

    PrepParams p;
    p.qhat = qhat;
    p.update = update;
    p.ws = yz;
    p.r = r;
    p.rp = (r + 1) & ~1;
    p.g = g;
    p.nsteps = nsteps;
    p.hard = isinf(lambda) ? 1 : 0;
    p.full = (flags_arg & SQUAT_PREPARE_FULL_PRECISION) ? 1 : 0;
    p.inv_lambda = p.hard ? 0.0 : 1.0 / static_cast<double>(lambda);
    p.nprob = n_heads * nsteps;
    int* need = nullptr;
    if (elim_route) {
        const int nt = (r + 15) / 16;
        // A workgroup per panel.  Its column tiles are the nt of S and those of Qb; the latter are split over several
        // workgroups, each of which eliminates S for itself, until a wavefront has one tile, as far as the launch then
        // stays within one workgroup per CU (256).
        int per = g / 16;
        while (per > 1 && nt + per > 4 && static_cast<int64_t>(n_heads) * nsteps * (g / 16) / (per / 2) <= 256) per /= 2;
        const dim3 grid(n_heads, nsteps, g / 16 / per), block(kElimThreads);
        const size_t lds = elim_lds_bytes(nt, per);        // 66 KB at most
        unsigned char* bytes = reinterpret_cast<unsigned char*>(flags);
        static std::atomic<uint64_t> elim_done[4];
        const void* kernels[4] = {reinterpret_cast<const void*>(prepare_elim_kernel<1>), reinterpret_cast<const void*>(prepare_elim_kernel<2>),
                                  reinterpret_cast<const void*>(prepare_elim_kernel<3>), reinterpret_cast<const void*>(prepare_elim_kernel<4>)};
        if ((rc = set_max_lds_once(elim_done[nt - 1], kernels[nt - 1], static_cast<int>(elim_lds_bytes(nt, 4))))) return rc;
        switch (nt) {
            case 1: hipLaunchKernelGGL(prepare_elim_kernel<1>, grid, block, lds, s, p, per, bytes); break;
            case 2: hipLaunchKernelGGL(prepare_elim_kernel<2>, grid, block, lds, s, p, per, bytes); break;
            case 3: hipLaunchKernelGGL(prepare_elim_kernel<3>, grid, block, lds, s, p, per, bytes); break;
            default: hipLaunchKernelGGL(prepare_elim_kernel<4>, grid, block, lds, s, p, per, bytes); break;
        }
        rc = check_launch();
        if (rc) return rc;
        need = flags;                                     // the eigen route below redoes the flagged heads only
    }
    if (p.rp <= 32) {
        // one workgroup per head, one wavefront per panel
        const size_t lds = ((static_cast<size_t>(p.rp) * (kD + 1) * sizeof(float) + 15) & ~size_t(15)) +
                           nsteps * (static_cast<size_t>(p.rp) * (p.rp + 2) + p.rp + 2 + 2 * static_cast<size_t>(p.rp) * g) * sizeof(double);
        static std::atomic<uint64_t> wave_done{0};
        if ((rc = set_max_lds_once(wave_done, reinterpret_cast<const void*>(prepare_wave_kernel), 140 * 1024))) return rc;
        hipLaunchKernelGGL(prepare_wave_kernel, dim3(n_heads), dim3(64 * nsteps), lds, s, p, need);
        return check_launch();
    }
    const size_t lds = (static_cast<size_t>(p.rp) * p.rp + p.rp) * sizeof(double) + 16;
    const dim3 grid(static_cast<unsigned>(p.nprob));
    const int ts = team_size(p.rp);
#define SQUAT_PREP_LAUNCH(TS)                                                                              \
    do {                                                                                                   \
        static std::atomic<uint64_t> done{0};                                                              \
        if ((rc = set_max_lds_once(done, reinterpret_cast<const void*>(prepare_kernel<TS>), 140 * 1024)))  \
            return rc;                                                                                     \
        hipLaunchKernelGGL(prepare_kernel<TS>, grid, dim3(kPrepThreads), lds, s, p, need);                 \
    } while (0)
    if (ts == 64) SQUAT_PREP_LAUNCH(64);
    else if (ts == 32) SQUAT_PREP_LAUNCH(32);
    else SQUAT_PREP_LAUNCH(16);
#undef SQUAT_PREP_LAUNCH
    return check_launch();
}

int prepare_check(const float* qhat, int n_heads, int d, int r, float lambda, int g, const float* update) {
    if (d != kD) return SQUAT_E_BADSHAPE;
    if (n_heads < 0 || r < 0 || r > d) return SQUAT_E_BADSHAPE;
    if (g != 32 && g != 64 && g != 128) return SQUAT_E_BADSHAPE;
    if (!(lambda >= 0.0f)) return SQUAT_E_BADVALUE;       // also rejects NaN
    if (n_heads == 0) return SQUAT_OK;
    if (!update || (r > 0 && !qhat)) return SQUAT_E_NULLPTR;
    if (!aligned(update, 16)) return SQUAT_E_ALIGN;
    return SQUAT_OK;
}

}  // namespace

extern "C" int squat_prepare(const float* qhat, int n_heads, int d, int r, float lambda, int g, float* update,
                             void* ws, size_t ws_bytes, squat_stream stream) {
    return squat_prepare_ex(qhat, n_heads, d, r, lambda, g, 0u, update, ws, ws_bytes, stream);
}

extern "C" int squat_prepare_ex(const float* qhat, int n_heads, int d, int r, float lambda, int g, unsigned flags_arg,
                                float* update, void* ws, size_t ws_bytes, squat_stream stream) {
    if (flags_arg & ~unsigned(SQUAT_PREPARE_FULL_PRECISION)) return SQUAT_E_BADVALUE;
    if (int rc = prepare_check(qhat, n_heads, d, r, lambda, g, update)) return rc;
    if (n_heads == 0) return SQUAT_OK;
    const int nsteps = d / g - 1;
    const bool trivial = (r == 0 || lambda == 0.0f || nsteps == 0);
    int* flags = nullptr;
    if (!trivial) {
        if (!ws || ws_bytes < squat_prepare_workspace(n_heads, d, r, g)) return SQUAT_E_WORKSPACE;
        if (!aligned(ws, 256)) return SQUAT_E_ALIGN;
        // the flags follow the (r-independent) room for the intermediate products
        const int rp = (r + 1) & ~1;
        flags = reinterpret_cast<int*>(static_cast<unsigned char*>(ws) +
                                       ((static_cast<size_t>(n_heads) * nsteps * rp * (g + kD) * sizeof(double) + 255) & ~size_t(255)));
    }
    return prepare_impl(qhat, n_heads, r, lambda, g, flags_arg, update, static_cast<double*>(ws), flags,
                        static_cast<hipStream_t>(stream));
}

namespace {

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device (each device holds its own copy at its own address).
int scratch_address(void** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SQUAT_E_HIP;
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return SQUAT_E_HIP;
        }
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // threads that race store the same address
    }
    *out = ptr;
    return SQUAT_OK;
}

}  // namespace

extern "C" int squat_prepare_noalloc(const float* qhat, int n_heads, int d, int r, float lambda, int g,
                                     float* update, squat_stream stream) {
    if (int rc = prepare_check(qhat, n_heads, d, r, lambda, g, update)) return rc;
    if (n_heads == 0) return SQUAT_OK;
    const bool trivial = (r == 0 || lambda == 0.0f || d / g - 1 == 0);
    double* yz = nullptr;
    int* flags = nullptr;
    if (!trivial) {
        const PrepScratch need = prep_scratch(n_heads, r, g, isinf(lambda));
        if (need.yz_bytes + need.flag_bytes > kStaticScratchBytes) return SQUAT_E_WORKSPACE;
        void* base = nullptr;
        if (int rc = scratch_address(&base)) return rc;
        // the intermediate products first (if any), the flags behind them
        yz = static_cast<double*>(base);
        flags = reinterpret_cast<int*>(static_cast<unsigned char*>(base) + need.yz_bytes);
    }
    return prepare_impl(qhat, n_heads, r, lambda, g, 0u, update, yz, flags, static_cast<hipStream_t>(stream));
}
