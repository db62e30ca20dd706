// Block-diagonal preconditioner of Sec. 3.1 (Eq. precond, Eq. block_diag_const_res).
//
// Build (once per state), per body p with m = 3 n_p:
//   pc_assemble  M_pp (m x m, row-major) from the same pair code as the mat-vec
//   pc_sweep     (no body above 256 rows) M_pp^-1 by the symmetric block sweep,
//                the matrix held in registers as 16 x 16 matrix-core tiles, one
//                workgroup per body; M_pp is kept.  Larger bodies:
//   pc_potrf     M_pp = L L^T in place, blocked by 32 columns: the panel is
//                factored in LDS, the trailing lower triangle updated in 64 x 64
//                tiles on the FP64 matrix cores; the inverses of the 32 x 32
//                diagonal blocks of L are kept for the next step
//   pc_trtri     X = L^-1 by block forward substitution on the identity, one
//                workgroup per (body, 32 columns), the block column held in LDS;
//                every block step is a small GEMM on the matrix cores because
//                the diagonal blocks are applied through their stored inverses;
//                X^T is kept in the strictly upper triangle
//   pc_lauum     M_pp^-1 = X^T X on the matrix cores, one workgroup per (body,
//                64 x 64 tile)
//   (bodies with more than 480 rows: pc_chol / pc_inverse, the unblocked
//   right-looking versions, with X = L^-1 kept transposed in the upper triangle)
//   pc_body      Z_p = M_pp^-1 K_p (m x 6), R_p = K_p^T Z_p, N~_p = R_p^+
//                (cyclic Jacobi eigen-decomposition, eigenvalues below
//                1e-12 * max dropped: the minimum-norm velocity of bodies with
//                a resistance-free motion)
// per assembly a (bodies joined by constraints):
//   pc_asm       S_a = C_a N~_a C_a^T, G~_a = S_a^-1 (by the sweep up to 256 rows,
//                else by Cholesky), or S_a^+ when a pivot falls below 1e-12 * max
//                diagonal (C_a without full row rank)
// Apply (every GMRES iteration), for residual r = (r_lam, r_U, r_phi):
//   pc_apply1    t_p = M_pp^-1 r_lam,p;  U^_p = -N~_p (r_U,p + Z_p^T r_lam,p)
//   pc_apply2    phi_a = G~_a (r_phi,a - C_a U^_a)
//   pc_apply3    U_p = U^_p + N~_p (C^T phi)_p;  lam_p = t_p + Z_p U_p
// (one launch, pc_apply_asm, when every assembly is small)
// which is the exact solution of the body-diagonal saddle problem: row 1 gives
// lam = M~^-1 (r_lam + K U), row 2 gives N~^-1 U = -r_U - K^T M~^-1 r_lam + C^T phi,
// row 3 gives (C N~ C^T) phi = r_phi - C U^.
#include "rpy_device.h"
#include "sweep_index.h"

namespace arb {

constexpr int kMaxBodyBlobs = 512;
constexpr int kMaxM = 3 * kMaxBodyBlobs;
constexpr int kMaxAsmRows = 2048;

// cyclic Jacobi eigen-decomposition of symmetric S (n x n, destroyed) with
// eigenvectors accumulated in V; writes the pseudo-inverse (cutoff relative to
// the largest |eigenvalue|) to out.  Returns the number of dropped eigenvalues.
// Single thread.
__device__ __forceinline__ int sym_pinv_serial(double *S, double *V, int n, double *out,
                                                double cutoff) {
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) V[i * n + j] = (i == j) ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 60; ++sweep) {
        double off = 0.0, dia = 0.0;
        for (int i = 0; i < n; ++i) {
            dia += S[i * n + i] * S[i * n + i];
            for (int j = i + 1; j < n; ++j) off += S[i * n + j] * S[i * n + j];
        }
        if (!(off > 1e-32 * dia)) break;
        for (int p = 0; p < n - 1; ++p) {
            for (int q = p + 1; q < n; ++q) {
                const double apq = S[p * n + q];
                if (apq == 0.0) continue;
                const double tau = (S[q * n + q] - S[p * n + p]) / (2.0 * apq);
                const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                const double c = 1.0 / sqrt(1.0 + t * t);
                const double s = t * c;
                for (int k = 0; k < n; ++k) {  // S <- S J
                    const double akp = S[k * n + p], akq = S[k * n + q];
                    S[k * n + p] = c * akp - s * akq;
                    S[k * n + q] = s * akp + c * akq;
                }
                for (int k = 0; k < n; ++k) {  // S <- J^T S
                    const double apk = S[p * n + k], aqk = S[q * n + k];
                    S[p * n + k] = c * apk - s * aqk;
                    S[q * n + k] = s * apk + c * aqk;
                }
                for (int k = 0; k < n; ++k) {  // V <- V J
                    const double vkp = V[k * n + p], vkq = V[k * n + q];
                    V[k * n + p] = c * vkp - s * vkq;
                    V[k * n + q] = s * vkp + c * vkq;
                }
            }
        }
    }
    double wmax = 0.0;
    for (int i = 0; i < n; ++i) wmax = fmax(wmax, fabs(S[i * n + i]));
    const double lim = cutoff * wmax;
    int dropped = 0;
    for (int i = 0; i < n; ++i) {
        const double w = S[i * n + i];
        const double inv = fabs(w) > lim ? 1.0 / w : 0.0;
        dropped += fabs(w) > lim ? 0 : 1;
        S[i * n + i] = inv;  // keep 1/w on the diagonal
    }
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) {
            double s = 0.0;
            for (int k = 0; k < n; ++k) s += V[i * n + k] * S[k * n + k] * V[j * n + k];
            out[i * n + j] = s;
        }
    return dropped;
}

__global__ __launch_bounds__(256) void pc_assemble_kernel(const int *__restrict__ order,
                                                          const int *__restrict__ blob_off,
                                                          const int64_t *__restrict__ mat_off,
                                                          const double *__restrict__ pos, CoefD c,
                                                          double scale, int wall, double a,
                                                          double *__restrict__ mats,
                                                          int *__restrict__ status) {
    const int p = order ? order[blockIdx.x] : blockIdx.x;
    const int b0 = blob_off[p], n = blob_off[p + 1] - b0, m = 3 * n;
    double *A = mats + mat_off[p];
    for (int idx = blockIdx.y * 256 + threadIdx.x; idx < n * n; idx += 256 * gridDim.y) {
        const int i = idx / n, j = idx - (idx / n) * n;
        const double *xi = pos + 3 * (size_t)(b0 + i);
        const double *xj = pos + 3 * (size_t)(b0 + j);
        if (wall && i == j && !(xi[2] > a)) atomicOr(&status[2], 1);
        double B[9];
        rpy_block_f64(xi[0] - xj[0], xi[1] - xj[1], xi[2] - xj[2], xi[2], xj[2], wall != 0, c, B);
        for (int r = 0; r < 3; ++r)
            for (int s = 0; s < 3; ++s) A[(size_t)(3 * i + r) * m + 3 * j + s] = scale * B[3 * r + s];
    }
}

// In-place Cholesky M = L L^T.  Lower triangle: L; upper triangle: L^T (kept
// for coalesced access by pc_inverse); Ldiag receives diag(L).
__global__ __launch_bounds__(256) void pc_chol_kernel(const int *__restrict__ blob_off,
                                                      const int64_t *__restrict__ mat_off,
                                                      double *__restrict__ mats,
                                                      double *__restrict__ ldiag,
                                                      int *__restrict__ status) {
    __shared__ double col[kMaxM];
    __shared__ int fail;
    const int p = blockIdx.x;
    const int m = 3 * (blob_off[p + 1] - blob_off[p]);
    double *A = mats + mat_off[p];
    if (threadIdx.x == 0) fail = 0;
    for (int k = 0; k < m; ++k) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const double d = A[(size_t)k * m + k];
            if (!(d > 0.0)) {
                fail = 1;
            } else {
                const double s = sqrt(d);
                A[(size_t)k * m + k] = s;
                col[k] = s;
            }
        }
        __syncthreads();
        if (fail) break;
        const double inv = 1.0 / col[k];
        for (int i = k + 1 + threadIdx.x; i < m; i += blockDim.x) {
            const double v = A[(size_t)i * m + k] * inv;
            A[(size_t)i * m + k] = v;
            A[(size_t)k * m + i] = v;
            col[i] = v;
        }
        __syncthreads();
        const int w = m - k - 1;
        for (int idx = threadIdx.x; idx < w * w; idx += blockDim.x) {
            const int ii = k + 1 + idx / w, jj = k + 1 + (idx - (idx / w) * w);
            A[(size_t)ii * m + jj] -= col[ii] * col[jj];
        }
    }
    __syncthreads();
    if (fail) {
        if (threadIdx.x == 0) atomicMax(&status[0], p + 1);
        return;
    }
    const int b0 = 3 * blob_off[p];
    for (int k = threadIdx.x; k < m; k += blockDim.x) ldiag[b0 + k] = col[k];
}

// X = L^-1 by right-looking forward substitution on the identity, X stored
// as X^T in the upper triangle (the diagonal of X replaces that of L, whose
// diagonal is saved in ldiag); then Minv = X^T X.
__global__ __launch_bounds__(256) void pc_inverse_kernel(const int *__restrict__ blob_off,
                                                         const int64_t *__restrict__ mat_off,
                                                         double *__restrict__ mats,
                                                         const double *__restrict__ ldiag,
                                                         double *__restrict__ minv,
                                                         const int *__restrict__ status) {
    __shared__ double colL[kMaxM];
    __shared__ double rowX[kMaxM];
    const int p = blockIdx.x;
    if (status[0] != 0) return;
    const int m = 3 * (blob_off[p + 1] - blob_off[p]);
    const double *Ld = ldiag + 3 * blob_off[p];
    double *A = mats + mat_off[p];
    double *Mi = minv + mat_off[p];
    // upper triangle incl. diagonal <- identity (X^T)
    for (int idx = threadIdx.x; idx < m * m; idx += blockDim.x) {
        const int j = idx / m, i = idx - (idx / m) * m;  // element (j, i) = X[i][j]
        if (i >= j) A[(size_t)j * m + i] = (i == j) ? 1.0 : 0.0;
    }
    for (int k = 0; k < m; ++k) {
        __syncthreads();
        const double inv = 1.0 / Ld[k];
        // row k of X: X[k][j], j <= k, lives at A[j*m + k]
        for (int j = threadIdx.x; j <= k; j += blockDim.x) {
            const double v = A[(size_t)j * m + k] * inv;
            A[(size_t)j * m + k] = v;
            rowX[j] = v;
        }
        for (int i = k + 1 + threadIdx.x; i < m; i += blockDim.x) colL[i] = A[(size_t)i * m + k];
        __syncthreads();
        const int w = m - k - 1;
        const int tot = w * (k + 1);
        for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
            const int j = idx / w, i = k + 1 + (idx - (idx / w) * w);
            A[(size_t)j * m + i] -= colL[i] * rowX[j];
        }
    }
    __syncthreads();
    // Minv[i][j] = sum_{k >= max(i,j)} X[k][i] X[k][j] = sum_k A[i*m+k] A[j*m+k]
    for (int idx = threadIdx.x; idx < m * m; idx += blockDim.x) {
        const int i = idx / m, j = idx - (idx / m) * m;
        if (j < i) continue;
        const double *ri = A + (size_t)i * m;
        const double *rj = A + (size_t)j * m;
        double s = 0.0;
        for (int k = j; k < m; ++k) s += ri[k] * rj[k];
        Mi[(size_t)i * m + j] = s;
        Mi[(size_t)j * m + i] = s;
    }
}

constexpr int kNB = 32;          // block size of the blocked factorisation
constexpr int kLd = kNB + 1;     // padded LDS row stride (doubles)
constexpr int kFastMaxM = 480;   // largest body handled by the blocked kernels

// FP64 matrix core, one wavefront: D (16 x 16) += A (16 x 4) B (4 x 16).  Lane l
// supplies a = A[l % 16][l / 16] and b = B[l / 16][l % 16] and holds
// D[4 e + l / 16][l % 16] in element e of the accumulator.
typedef double mfma_acc __attribute__((ext_vector_type(4)));
__device__ __forceinline__ mfma_acc mfma_f64_16x16x4(double a, double b, mfma_acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// A batch of symmetric positive definite matrices for the blocked kernels:
// matrix p has m_p = scale * (off[p+1] - off[p]) rows (scale 3 for the blob
// mobilities, off = blob offsets; scale 1 for the assemblies' S_a, off = row
// offsets), row-major at mats + mat_off[p]; its diagonal-block inverses at
// dinv_offset.  A matrix whose pivot falls to rel_tol * (its largest diagonal
// entry) or below fails: with fail != nullptr it is flagged there (and skipped
// by the later kernels), else status[0] receives p + 1 (an error).
struct MatBatch {
    const int *off;
    int scale;
    const int64_t *mat_off;
    double *mats;
    double *ldiag;  // diag(L) per row (may be null)
    double *dinv;
    double *out;    // the inverses (same offsets as mats)
    int *status;
    int *fail;
    double rel_tol;
    // matrix of a workgroup, largest first (may be null; the sweep's).  Workgroups go
    // round XCDs and shader engines in a fixed order, which gave every other engine all
    // the large matrices when sizes alternate (512 bacteria: 537 us, sorted 416)
    const int *order;
};
__device__ __forceinline__ int mat_rows(const MatBatch &B, int p) {
    return B.scale * (B.off[p + 1] - B.off[p]);
}
__device__ __forceinline__ bool mat_skip(const MatBatch &B, int p) {
    return B.status[0] != 0 || (B.fail && B.fail[p]);
}
// offset (doubles) of matrix p's diagonal-block inverses: 1024 per 32-row block
__device__ __forceinline__ int64_t dinv_offset(const MatBatch &B, int p) {
    return 32 * B.scale * (int64_t)B.off[p] + 1024 * (int64_t)p;
}


// Blocked right-looking Cholesky of each matrix of the batch, in place (lower
// triangle; the upper triangle is not touched), one workgroup per matrix,
// 32-column panels.  Per panel:
//   1. the 32 x 32 diagonal block is factored in LDS (outer-product form: one
//      barrier per pivot, the columns scaled once at the end), and its inverse
//      L_kk^-1 formed by the same row operations on the identity (kept in LDS and
//      stored for the triangular-inverse kernel);
//   2. the rows below become L_bel = A_bel L_kk^-T on the matrix cores (wavefront
//      w takes the 16-row tiles w, w + 4, ...; both column tiles of a row tile in
//      one wavefront, so a row is read completely before it is overwritten), stored
//      in the matrix and, column-major, in a panel scratch: the first 32 m doubles
//      of the matrix's slot in B.out, which only the later kernels write;
//   3. the trailing lower triangle takes A -= L_bel L_bel^T on the matrix cores in
//      64 x 64 tiles (wavefront w: the 32 x 32 quarter (w / 2, w % 2)), operands
//      read from the scratch (16 consecutive rows per load); a tile's entries are
//      read before its products run.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void pc_potrf_kernel(
    MatBatch B) {
    __shared__ double Dk[kNB * kLd];  // diagonal block, then L_kk
    __shared__ double Wi[kNB * kLd];  // L_kk^-1, zero padded
    __shared__ double isq[kNB];
    __shared__ int fail;
    __shared__ double piv_tol;
    const int p = blockIdx.x, tid = threadIdx.x;
    if (mat_skip(B, p)) return;
    const int m = mat_rows(B, p);
    double *A = B.mats + B.mat_off[p];
    double *Lp = B.out + B.mat_off[p];  // panel scratch, Lp[t * m + i]
    double *Dg = B.dinv + dinv_offset(B, p);
    const int w = tid >> 6, l = tid & 63;
    if (tid == 0) {
        fail = 0;
        double dmax = 0.0;
        if (B.rel_tol > 0.0)
            for (int k = 0; k < m; ++k) dmax = fmax(dmax, A[(size_t)k * m + k]);
        piv_tol = B.rel_tol * dmax;
    }
    for (int k0 = 0; k0 < m; k0 += kNB) {
        const int nb = min(kNB, m - k0), nt = m - k0 - nb;  // nt rows below the block
        __syncthreads();
        // 1. the diagonal block: thread tid holds entries (i, c) = (tid / 32 + 8 q, tid % 32).
        // The row operations of the elimination (row i -= l_ij row j, l_ij = D_ij / D_jj)
        // are applied to the identity in Wi as well, which turns it into the unit lower
        // triangular inverse factor; scaled by the pivots' 1/sqrt it is L_kk^-1
        const int c = tid & 31;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = (tid >> 5) + 8 * q;
            Dk[i * kLd + c] = (i < nb && c <= i) ? A[(size_t)(k0 + i) * m + k0 + c] : 0.0;
            Wi[i * kLd + c] = (i < nb && c == i) ? 1.0 : 0.0;
        }
        __syncthreads();
        bool bad = false;
        for (int j = 0; j < nb; ++j) {
            const double d = Dk[j * kLd + j];
            if (!(d > piv_tol)) {  // the same value for every thread: a uniform exit
                bad = true;
                break;
            }
            const double inv = 1.0 / d;
            // the pivot-row factor of this thread's column, then its four entries
            // (loads in bounds and unconditional; stores only below the pivot)
            const bool right = c > j;
            double *X = right ? Dk : Wi;
            const double pj = (right ? Dk[c * kLd + j] : Wi[j * kLd + c]) * inv;
            double lij[4], xv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = (tid >> 5) + 8 * q;
                lij[q] = Dk[i * kLd + j];
                xv[q] = X[i * kLd + c];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = (tid >> 5) + 8 * q;
                if (i > j && i < nb && (!right || c <= i)) X[i * kLd + c] = xv[q] - lij[q] * pj;
            }
            __syncthreads();
        }
        if (bad) {
            if (tid == 0) fail = 1;
            break;
        }
        // L_ic = D_ic / sqrt(D_cc), (L^-1)_ic = E_ic / sqrt(D_ii) with the final pivots D
        if (tid < nb) isq[tid] = 1.0 / sqrt(Dk[tid * kLd + tid]);
        __syncthreads();
        double lv[4], xv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = (tid >> 5) + 8 * q;
            const bool in = i < nb && c <= i;
            lv[q] = in ? Dk[i * kLd + c] * isq[c] : 0.0;
            xv[q] = in ? Wi[i * kLd + c] * isq[i] : 0.0;
        }
        __syncthreads();
        double *Db = Dg + (k0 / kNB) * (kNB * kNB);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = (tid >> 5) + 8 * q;
            Dk[i * kLd + c] = lv[q];
            Wi[i * kLd + c] = xv[q];
            Db[i * kNB + c] = xv[q];
            if (i < nb && c <= i) A[(size_t)(k0 + i) * m + k0 + c] = lv[q];
            if (B.ldiag && i < nb && c == i) B.ldiag[B.scale * (int64_t)B.off[p] + k0 + i] = lv[q];
        }
        if (nt <= 0) break;  // the last panel (nb = 32 whenever rows remain below)
        __syncthreads();
        // 2. L_bel = A_bel L_kk^-T: tile (row tile rt, column tile ct), lane l supplies
        // a = A_bel[16 rt + l % 16][4 s + l / 16] and b = Wi[16 ct + l % 16][4 s + l / 16]
        const int nrt = (nt + 15) >> 4;
        double *Abel = A + (size_t)(k0 + kNB) * m + k0;
        for (int rt = w; rt < nrt; rt += 4) {
            const int ra = min(16 * rt + (l & 15), nt - 1);
            double av[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) av[s] = Abel[(size_t)ra * m + 4 * s + (l >> 4)];
            mfma_acc acc0 = {}, acc1 = {};
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int kk = 4 * s + (l >> 4);
                acc0 = mfma_f64_16x16x4(av[s], Wi[(l & 15) * kLd + kk], acc0);
                acc1 = mfma_f64_16x16x4(av[s], Wi[(16 + (l & 15)) * kLd + kk], acc1);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 16 * rt + 4 * e + (l >> 4);
                if (i < nt) {
                    const int cc = l & 15;
                    Abel[(size_t)i * m + cc] = acc0[e];
                    Abel[(size_t)i * m + 16 + cc] = acc1[e];
                    Lp[(size_t)cc * m + i] = acc0[e];
                    Lp[(size_t)(16 + cc) * m + i] = acc1[e];
                }
            }
        }
        __syncthreads();
        // 3. trailing update of the lower triangle, A_ij -= sum_t L_it L_jt
        const int t0 = k0 + kNB;
        const int ntile = (nt + 63) / 64;
        const int wr = w >> 1, wc = w & 1;
        const int ntiles = ntile * (ntile + 1) / 2;
        // tile -> (bi, bj), bj <= bi, row by row of the lower triangle of tiles
        auto tile_ij = [](int tile, int &bi, int &bj) {
            bi = 0;
            while ((bi + 1) * (bi + 2) / 2 <= tile) ++bi;
            bj = tile - bi * (bi + 1) / 2;
        };
        // this lane's 16 entries of a tile's 32 x 32 quarter (clamped into the matrix)
        auto load_quarter = [&](int i0, int j0, double (&v)[2][2][4]) {
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                for (int tj = 0; tj < 2; ++tj)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = min(i0 + 16 * ti + 4 * e + (l >> 4), nt - 1);
                        const int j = min(j0 + 16 * tj + (l & 15), nt - 1);
                        v[ti][tj][e] = A[(size_t)(t0 + i) * m + t0 + j];
                    }
        };
        for (int tile = 0; tile < ntiles; ++tile) {
            int bi, bj;
            tile_ij(tile, bi, bj);
            const int i0 = 64 * bi + 32 * wr, j0 = 64 * bj + 32 * wc;
            double cur[2][2][4];
            load_quarter(i0, j0, cur);
            const int ra0 = min(i0 + (l & 15), nt - 1), ra1 = min(i0 + 16 + (l & 15), nt - 1);
            const int rb0 = min(j0 + (l & 15), nt - 1), rb1 = min(j0 + 16 + (l & 15), nt - 1);
            mfma_acc acc[2][2] = {};
#pragma unroll 2
            for (int s = 0; s < 8; ++s) {
                const double *col = Lp + (size_t)(4 * s + (l >> 4)) * m;
                const double a0 = col[ra0], a1 = col[ra1], b0 = col[rb0], b1 = col[rb1];
                acc[0][0] = mfma_f64_16x16x4(a0, b0, acc[0][0]);
                acc[0][1] = mfma_f64_16x16x4(a0, b1, acc[0][1]);
                acc[1][0] = mfma_f64_16x16x4(a1, b0, acc[1][0]);
                acc[1][1] = mfma_f64_16x16x4(a1, b1, acc[1][1]);
            }
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                for (int tj = 0; tj < 2; ++tj)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = i0 + 16 * ti + 4 * e + (l >> 4);
                        const int j = j0 + 16 * tj + (l & 15);
                        if (i < nt && j <= i)
                            A[(size_t)(t0 + i) * m + t0 + j] = cur[ti][tj][e] - acc[ti][tj][e];
                    }
        }
    }
    __syncthreads();
    if (fail && tid == 0) {
        if (B.fail)
            B.fail[p] = 1;
        else
            atomicMax(&B.status[0], p + 1);
    }
}

// load (4 per thread) the 32 x 32 block of L at (R0, C0), zero padded beyond m
__device__ __forceinline__ void load_block(double v[4], const double *A, int m, int R0, int C0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int idx = threadIdx.x + 256 * e, t = idx / kNB, u = idx % kNB;
        v[e] = (R0 + t < m && C0 + u < m) ? A[(size_t)(R0 + t) * m + C0 + u] : 0.0;
    }
}
__device__ __forceinline__ void store_block(double (*Ls)[kLd], const double v[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int idx = threadIdx.x + 256 * e;
        Ls[idx / kNB][idx % kNB] = v[e];
    }
}

// X = L^-1, block column [32 cb, 32 cb + 32): forward block substitution on the
// identity, X_i = Dinv_i (E_i - sum_{cb <= k < i} L_ik X_k); the next block of
// L is read into registers while the current one is used.  The strictly lower
// part of X is stored transposed in the strictly upper triangle of M_pp's
// storage (the diagonal of X is 1 / diag(L)).  Dynamic LDS: the block column,
// ceil(max_m / 32) * 32 x kLd doubles.
__global__ __launch_bounds__(256) void pc_trtri_kernel(MatBatch B) {
    extern __shared__ double X[];
    __shared__ double Ls[kNB][kLd];
    const int p = blockIdx.y, cb = blockIdx.x;
    if (mat_skip(B, p)) return;
    const int m = mat_rows(B, p);
    const int nbk = (m + kNB - 1) / kNB;
    if (cb >= nbk) return;
    double *A = B.mats + B.mat_off[p];
    const double *Dg = B.dinv + dinv_offset(B, p);
    // wavefront w holds the 16 x 16 tile (w / 2, w % 2) of each 32 x 32 block step
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int wr = 16 * (w >> 1), wc = 16 * (w & 1);
    const int lr = l & 15, lk = l >> 4;  // operand row and k offset of this lane
    const int c0 = kNB * cb;
    for (int i = cb; i < nbk; ++i) {
        double dreg[4], nxt[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) dreg[e] = Dg[(size_t)i * kNB * kNB + tid + 256 * e];
        if (cb < i) load_block(nxt, A, m, kNB * i, kNB * cb);
        mfma_acc acc;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = (kNB * i + wr + 4 * e + lk == c0 + wc + lr) ? 1.0 : 0.0;
        for (int k = cb; k < i; ++k) {
            __syncthreads();
            store_block(Ls, nxt);
            __syncthreads();
            if (k + 1 < i) load_block(nxt, A, m, kNB * i, kNB * (k + 1));
            const double *Xk = X + (size_t)kNB * k * kLd + wc + lr;
#pragma unroll
            for (int kk = 0; kk < kNB; kk += 4)
                acc = mfma_f64_16x16x4(-Ls[wr + lr][kk + lk], Xk[(kk + lk) * kLd], acc);
        }
        double *Xi = X + (size_t)kNB * i * kLd;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) Xi[(wr + 4 * e + lk) * kLd + wc + lr] = acc[e];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int idx = tid + 256 * e;
            Ls[idx / kNB][idx % kNB] = dreg[e];
        }
        __syncthreads();
        mfma_acc y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < kNB; kk += 4)
            y = mfma_f64_16x16x4(Ls[wr + lr][kk + lk], Xi[(kk + lk) * kLd + wc + lr], y);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) Xi[(wr + 4 * e + lk) * kLd + wc + lr] = y[e];
    }
    __syncthreads();
    // X[i][c0 + c] for i > c0 + c  ->  A[(c0 + c) m + i]  (consecutive i: coalesced)
    const int rows = m - c0;
    for (int idx = tid; idx < rows * kNB; idx += 256) {
        const int c = idx / rows, i = c0 + idx % rows;
        const int j = c0 + c;
        if (j < m && i > j) A[(size_t)j * m + i] = X[(size_t)i * kLd + c];
    }
}

// M_pp^-1 = X^T X = U U^T with U = X^T upper triangular (strictly upper part in
// M_pp's storage; the diagonal, 1 / diag(L), read from the diagonal-block
// inverses).  One workgroup per (body, 64 x 64 tile (I, J), I <= J); the sum
// over k >= J runs in chunks of 32 staged in LDS, the next chunk read into
// registers meanwhile.  Writes both (I, J) and (J, I).
__global__ __launch_bounds__(256) void pc_lauum_kernel(MatBatch B) {
    __shared__ double Ua[64][kLd], Ub[64][kLd];
    const int p = blockIdx.y;
    if (mat_skip(B, p)) return;
    const int m = mat_rows(B, p);
    const int nt = (m + 63) / 64;
    const int tile = blockIdx.x;
    if (tile >= nt * (nt + 1) / 2) return;
    int bj = 0;
    while ((bj + 1) * (bj + 2) / 2 <= tile) ++bj;
    const int bi = tile - bj * (bj + 1) / 2;  // bi <= bj
    const int I0 = 64 * bi, J0 = 64 * bj;
    const double *A = B.mats + B.mat_off[p];
    const double *Dg = B.dinv + dinv_offset(B, p);
    double *Mi = B.out + B.mat_off[p];
    const int tid = threadIdx.x;
    const int kl = tid & 31, r0 = tid >> 5;  // a thread stages column kl of rows r0 + 8e
    // wavefront w computes the 32 x 32 quarter (w / 2, w % 2) as 2 x 2 matrix-core tiles
    const int w = tid >> 6, l = tid & 63, wr = 32 * (w >> 1), wc = 32 * (w & 1);
    const int lr = l & 15, lk = l >> 4;
    // U[row][kk]: 0 below the diagonal, 1/L_kk on it, X[kk][row] above
    auto u_at = [&](int row, int kk) -> double {
        if (row >= m || kk >= m || kk < row) return 0.0;
        if (kk == row) return Dg[(size_t)(row >> 5) * kNB * kNB + (row & 31) * (kNB + 1)];
        return A[(size_t)row * m + kk];
    };
    double na[8], nb8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        na[e] = u_at(I0 + r0 + 8 * e, J0 + kl);
        nb8[e] = u_at(J0 + r0 + 8 * e, J0 + kl);
    }
    mfma_acc acc[2][2] = {};
    for (int k0 = J0; k0 < m; k0 += kNB) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            Ua[r0 + 8 * e][kl] = na[e];
            Ub[r0 + 8 * e][kl] = nb8[e];
        }
        __syncthreads();
        if (k0 + kNB < m) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                na[e] = u_at(I0 + r0 + 8 * e, k0 + kNB + kl);
                nb8[e] = u_at(J0 + r0 + 8 * e, k0 + kNB + kl);
            }
        }
#pragma unroll
        for (int kk = 0; kk < kNB; kk += 4) {
            const double a0 = Ua[wr + lr][kk + lk], a1 = Ua[wr + 16 + lr][kk + lk];
            const double b0 = Ub[wc + lr][kk + lk], b1 = Ub[wc + 16 + lr][kk + lk];
            acc[0][0] = mfma_f64_16x16x4(a0, b0, acc[0][0]);
            acc[0][1] = mfma_f64_16x16x4(a0, b1, acc[0][1]);
            acc[1][0] = mfma_f64_16x16x4(a1, b0, acc[1][0]);
            acc[1][1] = mfma_f64_16x16x4(a1, b1, acc[1][1]);
        }
    }
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = I0 + wr + 16 * ti + 4 * e + lk;
                const int j = J0 + wc + 16 * tj + lr;
                if (i < m && j < m) {
                    Mi[(size_t)i * m + j] = acc[ti][tj][e];
                    Mi[(size_t)j * m + i] = acc[ti][tj][e];
                }
            }
}

// restore L's diagonal (for inspection) once the inverse no longer needs X
__global__ void pc_restore_diag_kernel(const int *__restrict__ blob_off,
                                       const int64_t *__restrict__ mat_off,
                                       double *__restrict__ mats,
                                       const double *__restrict__ ldiag) {
    const int p = blockIdx.x;
    const int m = 3 * (blob_off[p + 1] - blob_off[p]);
    double *A = mats + mat_off[p];
    for (int k = threadIdx.x; k < m; k += blockDim.x)
        A[(size_t)k * m + k] = ldiag[3 * blob_off[p] + k];
}

// rows of K_p: blob i, component a: u part e_a, w part row a of -(d_i^x)
__device__ __forceinline__ double K_entry(const double *d, int a, int c) {
    if (c < 3) return a == c ? 1.0 : 0.0;
    const int b = c - 3;
    // -(d^x)[a][b] with d^x = [[0,-d2,d1],[d2,0,-d0],[-d1,d0,0]]
    if (a == b) return 0.0;
    if (a == 0) return b == 1 ? d[2] : -d[1];
    if (a == 1) return b == 0 ? -d[2] : d[0];
    return b == 0 ? d[1] : -d[0];
}

// X = L^-1 of a symmetric positive definite 6 x 6 R = L L^T (R^-1 = X^T X); false when a
// pivot falls to 1e-8 of the largest diagonal entry or below (then the caller takes the
// pseudo-inverse, which is the inverse whenever this succeeds).
// Lane c < 6 gets column c of L^-1 (zeros above the diagonal); the factor itself is
// computed by every lane, in registers.
__device__ __forceinline__ bool chol_inv6(const double *R, int c, double *X) {
    double dmax = 0.0;
#pragma unroll
    for (int i = 0; i < 6; ++i) dmax = fmax(dmax, R[i * 6 + i]);
    const double tol = 1e-8 * dmax;
    double L[6][6];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double d = R[j * 6 + j];
#pragma unroll
        for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
        ok &= d > tol;
        L[j][j] = sqrt(d);
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            double v = R[i * 6 + j];
#pragma unroll
            for (int k = 0; k < j; ++k) v -= L[i][k] * L[j][k];
            L[i][j] = v / L[j][j];
        }
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        double v = i == c ? 1.0 : 0.0;
#pragma unroll
        for (int k = 0; k < i; ++k) v -= L[i][k] * X[k];
        X[i] = v / L[i][i];
    }
    return ok;
}

// Per body: Z = M^-1 K (m x 6) and N~ = (K^T M^-1 K)^-1 (Sec. 3.1).  Thread r
// takes row r of Z (M^-1 is symmetric, so the row is read as column r:
// consecutive threads read consecutive addresses) and adds K_r^T Z_r to its
// partial R = K^T Z (the 21 entries of the upper triangle); the partials are
// summed over the wavefronts, then N~ = R^-1 by Cholesky, in registers and a lane per
// column; when R is singular (a rod of collinear blobs) R is stored and flagged for
// pc_body_pinv_kernel.  A few bodies wait on their loads, many are bound by M^-1 (512
// bacteria: 301 MB): with five blobs' loads in flight a row, and the factor in registers
// instead of one thread's LDS, 33 -> 21 us for 16 bacteria, 101 -> 85 for 512 (3.6 TB/s).
// Four threads a row: 181 us, too few workgroups fit a compute unit.
__global__ __launch_bounds__(256) void pc_body_kernel(const int *__restrict__ order,
                                                      const int *__restrict__ blob_off,
                                                      const int64_t *__restrict__ mat_off,
                                                      const int64_t *__restrict__ z_off,
                                                      const double *__restrict__ minv,
                                                      const double *__restrict__ dvec,
                                                      double *__restrict__ Zbuf,
                                                      double *__restrict__ Nt,
                                                      int *__restrict__ body_pinv,
                                                      int *__restrict__ status) {
    __shared__ double red[4][21];
    __shared__ double S6[36], V6[36];  // R, L^-1
    __shared__ int singular;
    const int p = order ? order[blockIdx.x] : blockIdx.x;
    if (status[0] != 0) return;
    const int b0 = blob_off[p], n = blob_off[p + 1] - b0, m = 3 * n;
    const double *Mi = minv + mat_off[p];
    double *Z = Zbuf + z_off[p];
    const double *d = dvec + 3 * (size_t)b0;
    double racc[21];
#pragma unroll
    for (int e = 0; e < 21; ++e) racc[e] = 0.0;
    for (int r = threadIdx.x; r < m; r += blockDim.x) {
        double z[6] = {0, 0, 0, 0, 0, 0};
        const double *col = Mi + r;
#pragma unroll 5
        for (int i = 0; i < n; ++i) {
            const double m0 = col[(size_t)(3 * i) * m], m1 = col[(size_t)(3 * i + 1) * m],
                         m2 = col[(size_t)(3 * i + 2) * m];
            const double *di = d + 3 * i;
            z[0] += m0;
            z[1] += m1;
            z[2] += m2;
            // sum_a M[r][3i+a] * (-(d^x))[a][b]
            z[3] += -m1 * di[2] + m2 * di[1];
            z[4] += m0 * di[2] - m2 * di[0];
            z[5] += -m0 * di[1] + m1 * di[0];
        }
        for (int c = 0; c < 6; ++c) Z[(size_t)r * 6 + c] = z[c];
        // row r = 3 i + a of K: e_a, then -(d_i^x) row a
        const double *dr = d + 3 * (r / 3);
        const int a = r % 3;
        double kr[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) kr[c] = K_entry(dr, a, c);
        int e = 0;
#pragma unroll
        for (int c1 = 0; c1 < 6; ++c1)
#pragma unroll
            for (int c2 = c1; c2 < 6; ++c2) racc[e++] += kr[c1] * z[c2];
    }
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int e = 0; e < 21; ++e) {
        double v = racc[e];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) red[w][e] = v;
    }
    __syncthreads();
    if (threadIdx.x < 36) {
        const int i = threadIdx.x / 6, j = threadIdx.x % 6, c1 = min(i, j), c2 = max(i, j);
        const int e = c1 * 6 - c1 * (c1 - 1) / 2 + c2 - c1;
        double v = 0.0;
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) v += red[k][e];
        S6[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        double X[6];
        const bool ok = chol_inv6(S6, threadIdx.x, X);
        for (int i = 0; i < 6; ++i) V6[i * 6 + threadIdx.x] = X[i];
        if (threadIdx.x == 0) singular = !ok;
    }
    __syncthreads();
    if (threadIdx.x < 36) {
        const int i = threadIdx.x / 6, j = threadIdx.x % 6;
        double v = 0.0;
        for (int k = max(i, j); k < 6; ++k) v += V6[k * 6 + i] * V6[k * 6 + j];
        // singular: R for pc_body_pinv_kernel
        Nt[36 * (size_t)p + threadIdx.x] = singular ? S6[threadIdx.x] : v;
    }
    if (threadIdx.x == 0) body_pinv[p] = singular;
}

// N~_p = R_p^+ (symmetric pseudo-inverse, eigenvalues below 1e-12 of the largest
// dropped) for the bodies whose R_p failed the Cholesky test, one thread each
__global__ __launch_bounds__(64) void pc_body_pinv_kernel(int M, const int *__restrict__ body_pinv,
                                                          double *__restrict__ Nt,
                                                          int *__restrict__ status) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= M || !body_pinv[p] || status[0] != 0) return;
    double S[36], V[36];
    double *out = Nt + 36 * (size_t)p;
    for (int k = 0; k < 36; ++k) S[k] = out[k];
    if (sym_pinv_serial(S, V, 6, out, 1e-12)) atomicAdd(&status[3], 1);
}

// S = C_a N~_a C_a^T (na x na, row-major) for the assembly's rows r0 .. r0+na-1,
// all threads of the block
__device__ void asm_form_S(int r0, int na, const int *__restrict__ asm_rows,
                           const int *__restrict__ row_p, const int *__restrict__ row_q,
                           const double *__restrict__ crow, const double *__restrict__ Nt,
                           double *__restrict__ S) {
    for (int idx = threadIdx.x; idx < na * na; idx += blockDim.x) {
        const int k = idx / na, l = idx - (idx / na) * na;
        const int rk = asm_rows[r0 + k], rl = asm_rows[r0 + l];
        double sum = 0.0;
#pragma unroll 1
        for (int sk = 0; sk < 2; ++sk) {
            const int bk = sk ? row_q[rk] : row_p[rk];
            if (bk < 0) continue;
            const double *ck = crow + 12 * (size_t)rk + 6 * sk;
#pragma unroll 1
            for (int sl = 0; sl < 2; ++sl) {
                const int bl = sl ? row_q[rl] : row_p[rl];
                if (bl != bk) continue;
                const double *cl = crow + 12 * (size_t)rl + 6 * sl;
                const double *Nb = Nt + 36 * (size_t)bk;
                for (int u = 0; u < 6; ++u) {
                    double t = 0.0;
                    for (int v = 0; v < 6; ++v) t += Nb[u * 6 + v] * cl[v];
                    sum += ck[u] * t;
                }
            }
        }
        S[(size_t)k * na + l] = sum;
    }
}

// The rows of one assembly staged in LDS: cl[12 k + 6 side + u] the row's
// coefficients on the body of that side, bl[2 k + side] the body (-1: none).
__device__ void asm_stage_rows(int r0, int na, const int *__restrict__ asm_rows,
                               const int *__restrict__ row_p, const int *__restrict__ row_q,
                               const double *__restrict__ crow, double *cl, int *bl) {
    for (int idx = threadIdx.x; idx < 12 * na; idx += blockDim.x) {
        const int k = idx / 12, u = idx - 12 * k;
        cl[idx] = crow[12 * (size_t)asm_rows[r0 + k] + u];
    }
    for (int k = threadIdx.x; k < na; k += blockDim.x) {
        const int rk = asm_rows[r0 + k];
        bl[2 * k] = row_p[rk];
        bl[2 * k + 1] = row_q[rk];
    }
}

// the lower triangle of the assemblies' S_a for the blocked kernels (assemblies of
// at most kFastMaxM rows; the factorisation reads no other entries): N~_b c for both
// sides of each row, then an entry per thread, the sum over the side pairs on the same
// body (a thread per column took 56 us for 64 diatom colonies, this 25).  Dynamic LDS:
// the staged rows and N~_b c, 24 doubles and 2 ints per row of the largest assembly.
constexpr int kAsmForm = 1024;
__global__ __launch_bounds__(kAsmForm) void pc_asm_form_kernel(
    const int *__restrict__ asm_row_ptr, const int *__restrict__ asm_rows,
    const int64_t *__restrict__ asm_mat_off, const int *__restrict__ row_p,
    const int *__restrict__ row_q, const double *__restrict__ crow, const double *__restrict__ Nt,
    double *__restrict__ Sbuf, int *__restrict__ fail, const int *__restrict__ status,
    int max_rows) {
    extern __shared__ double sm[];
    double *cl = sm, *tl = cl + 12 * (size_t)max_rows;  // N~_b c for both sides of each row
    int *bl = reinterpret_cast<int *>(tl + 12 * (size_t)max_rows);
    const int a = blockIdx.x, tid = threadIdx.x;
    const int r0 = asm_row_ptr[a], na = asm_row_ptr[a + 1] - r0;
    if (tid == 0) fail[a] = 0;
    if (na == 0 || status[0] != 0) return;
    asm_stage_rows(r0, na, asm_rows, row_p, row_q, crow, cl, bl);
    __syncthreads();
    for (int idx = tid; idx < 12 * na; idx += kAsmForm) {
        const int l = idx / 12, sd = (idx / 6) & 1, u = idx % 6;
        const int b = bl[2 * l + sd];
        double v = 0.0;
        if (b >= 0)
            for (int w = 0; w < 6; ++w) v += Nt[36 * (size_t)b + u * 6 + w] * cl[12 * l + 6 * sd + w];
        tl[idx] = v;
    }
    __syncthreads();
    double *S = Sbuf + asm_mat_off[a];
    for (int k = tid / kWave; k < na; k += kAsmForm / kWave)
        for (int l = tid % kWave; l <= k; l += kWave) {
            double sum = 0.0;
            for (int sk = 0; sk < 2; ++sk) {
                const int bk = bl[2 * k + sk];
                if (bk < 0) continue;
                for (int sl = 0; sl < 2; ++sl)
                    if (bl[2 * l + sl] == bk)
                        for (int u = 0; u < 6; ++u)
                            sum += cl[12 * k + 6 * sk + u] * tl[12 * l + 6 * sl + u];
            }
            S[(size_t)k * na + l] = sum;
        }
}

// assemblies whose S_a failed the Cholesky pivot test: S_a formed again and its
// symmetric pseudo-inverse (eigenvalues below 1e-12 * max dropped), Sec. 3.1;
// X is scratch of na^2 doubles after S in the same assembly slot of Xbuf
__global__ __launch_bounds__(256) void pc_asm_pinv_kernel(
    const int *__restrict__ asm_row_ptr, const int *__restrict__ asm_rows,
    const int64_t *__restrict__ asm_mat_off, const int *__restrict__ row_p,
    const int *__restrict__ row_q, const double *__restrict__ crow, const double *__restrict__ Nt,
    double *__restrict__ Xbuf, double *__restrict__ Gbuf, const int *__restrict__ fail,
    int *__restrict__ status) {
    const int a = blockIdx.x;
    if (!fail[a] || status[0] != 0) return;
    const int r0 = asm_row_ptr[a], na = asm_row_ptr[a + 1] - r0;
    double *S = Xbuf + 2 * asm_mat_off[a];
    asm_form_S(r0, na, asm_rows, row_p, row_q, crow, Nt, S);
    __syncthreads();
    if (threadIdx.x == 0) {
        sym_pinv_serial(S, S + (size_t)na * na, na, Gbuf + asm_mat_off[a], 1e-12);
        atomicAdd(&status[1], 1);
    }
}

// Assemblies of at most kAsmSmall rows, one workgroup of 256 threads each,
// everything in LDS (dynamic: S and E, n (n + 1) doubles each, the staged rows and
// N~_b c per row, for n rows of the largest assembly):
//   S = C_a N~ C_a^T (lower triangle, an entry per thread);
//   elimination in outer-product form (row i -= l_ij row j, l_ij = S_ij / S_jj,
//   one barrier per pivot; pivot test relative to the largest diagonal entry),
//   the same row operations applied to the identity in E, which becomes the unit
//   lower triangular factor E with E S E^T = D (the final pivots);
//   G~ = S^-1 = E^T D^-1 E, each entry by one thread.
// A failed pivot flags the assembly for the pseudo-inverse kernel.  A barrier and a
// division per pivot: 14 us at 12 rows, where forming S and the block sweep take 13 and a
// launch more; at 27 rows 26.5 us against 16, at 63 91 against 26.
constexpr int kAsmSmall = 16;
constexpr int kAsmThreads = 256;
constexpr int kAsmSlots = kAsmSmall * kAsmSmall / kAsmThreads;  // rows per thread
constexpr int kAsmStep = kAsmThreads / kAsmSmall;
__global__ __launch_bounds__(kAsmThreads) void pc_asm_small_kernel(
    const int *__restrict__ asm_row_ptr, const int *__restrict__ asm_rows,
    const int64_t *__restrict__ asm_mat_off, const int *__restrict__ row_p,
    const int *__restrict__ row_q, const double *__restrict__ crow, const double *__restrict__ Nt,
    double *__restrict__ Gbuf, int *__restrict__ fail, const int *__restrict__ status,
    int max_rows) {
    extern __shared__ double sm[];
    const int ld = max_rows + 1;
    double *S = sm, *E = S + (size_t)max_rows * ld, *cl = E + (size_t)max_rows * ld;
    double *tl = cl + 12 * (size_t)max_rows;  // N~_b c for both sides of each row
    int *bl = reinterpret_cast<int *>(tl + 12 * (size_t)max_rows);
    __shared__ double tol;
    __shared__ double invd[kAsmSmall];
    const int a = blockIdx.x, tid = threadIdx.x;
    const int r0 = asm_row_ptr[a], na = asm_row_ptr[a + 1] - r0;
    if (tid == 0) fail[a] = 0;
    if (na == 0 || status[0] != 0) return;
    asm_stage_rows(r0, na, asm_rows, row_p, row_q, crow, cl, bl);
    for (int idx = tid; idx < kAsmSmall * kAsmSmall; idx += kAsmThreads) {
        const int i = idx / kAsmSmall, c = idx % kAsmSmall;
        if (i < na && c <= i) E[i * ld + c] = i == c ? 1.0 : 0.0;
    }
    __syncthreads();
    // t = N~_b c per row and side (a thread per entry), then every entry of the
    // lower triangle of S = C N~ C^T at once
    for (int idx = tid; idx < 12 * na; idx += kAsmThreads) {
        const int l = idx / 12, sd = (idx / 6) & 1, u = idx % 6;
        const int b = bl[2 * l + sd];
        double v = 0.0;
        if (b >= 0)
            for (int w = 0; w < 6; ++w) v += Nt[36 * (size_t)b + u * 6 + w] * cl[12 * l + 6 * sd + w];
        tl[idx] = v;
    }
    __syncthreads();
    for (int idx = tid; idx < kAsmSmall * kAsmSmall; idx += kAsmThreads) {
        const int k = idx / kAsmSmall, l = idx % kAsmSmall;
        if (k >= na || l > k) continue;
        double sum = 0.0;
        for (int sk = 0; sk < 2; ++sk) {
            const int bk = bl[2 * k + sk];
            if (bk < 0) continue;
            for (int sl = 0; sl < 2; ++sl)
                if (bl[2 * l + sl] == bk)
                    for (int u = 0; u < 6; ++u)
                        sum += cl[12 * k + 6 * sk + u] * tl[12 * l + 6 * sl + u];
        }
        S[k * ld + l] = sum;
    }
    __syncthreads();
    if (tid == 0) {
        double dmax = 0.0;
        for (int k = 0; k < na; ++k) dmax = fmax(dmax, S[k * ld + k]);
        tol = 1e-12 * dmax;
    }
    __syncthreads();
    // thread tid owns column c = tid % 16 of rows i = tid / 16 + 16 q (q < kAsmSlots):
    // the column-c entries of row j are read once per pivot, the rows' entries all
    // issued before they are updated
    const int c = tid % kAsmSmall, i0 = tid / kAsmSmall;
    for (int j = 0; j < na; ++j) {
        const double d = S[j * ld + j];
        if (!(d > tol)) {  // the same value for every thread: a uniform exit
            if (tid == 0) fail[a] = 1;
            return;
        }
        const double inv = 1.0 / d;
        if (c < na) {
            const bool right = c > j;  // S entry (right of the pivot column), else E entry
            const double pj = (right ? S[c * ld + j] : E[j * ld + c]) * inv;
            double *X = right ? S : E;
            // every load in bounds (rows clamped to the matrix) and issued before
            // the updates, which only the slots below the pivot row store
            double sij[kAsmSlots], xv[kAsmSlots];
#pragma unroll
            for (int q = 0; q < kAsmSlots; ++q) {
                const int i = min(i0 + kAsmStep * q, na - 1);
                sij[q] = S[i * ld + j];
                xv[q] = X[i * ld + c];
            }
#pragma unroll
            for (int q = 0; q < kAsmSlots; ++q) {
                const int i = i0 + kAsmStep * q;
                if (i > j && i < na && c <= i) X[i * ld + c] = xv[q] - sij[q] * pj;
            }
        }
        __syncthreads();
    }
    if (tid < na) invd[tid] = 1.0 / S[tid * ld + tid];
    __syncthreads();
    // G~_ij = sum_k E_ki E_kj / D_k over k >= max(i, j): thread tid takes column
    // j = tid % 16 of rows i = tid / 16 + 16 q, one pass over k
    double *G = Gbuf + asm_mat_off[a];
    const int j = c;
    double acc[kAsmSlots];
#pragma unroll
    for (int q = 0; q < kAsmSlots; ++q) acc[q] = 0.0;
    if (j < na)
        for (int k = j; k < na; ++k) {
            const double ekj = E[k * ld + j] * invd[k];
#pragma unroll
            for (int q = 0; q < kAsmSlots; ++q) {
                const int i = i0 + kAsmStep * q;
                const double eki = E[k * ld + min(i, k)];  // in bounds; used for i <= k
                acc[q] += i <= k ? eki * ekj : 0.0;
            }
        }
#pragma unroll
    for (int q = 0; q < kAsmSlots; ++q) {
        const int i = i0 + kAsmStep * q;
        if (i < na && j < na) G[(size_t)i * na + j] = acc[q];
    }
}

// assemblies beyond kFastMaxM rows: unblocked Cholesky and inverse in global memory
__global__ __launch_bounds__(256) void pc_asm_kernel(
    const int *__restrict__ asm_row_ptr, const int *__restrict__ asm_rows,
    const int64_t *__restrict__ asm_mat_off, const int *__restrict__ row_p,
    const int *__restrict__ row_q, const double *__restrict__ crow, const double *__restrict__ Nt,
    double *__restrict__ Sbuf, double *__restrict__ Gbuf, int *__restrict__ status) {
    __shared__ double col[kMaxAsmRows];
    __shared__ int fail;
    __shared__ double dmax;
    const int a = blockIdx.x;
    const int r0 = asm_row_ptr[a], na = asm_row_ptr[a + 1] - r0;
    if (na == 0) return;
    if (status[0] != 0) return;
    double *S = Sbuf + 2 * asm_mat_off[a];
    double *X = S + (size_t)na * na;
    double *G = Gbuf + asm_mat_off[a];
    for (int pass = 0; pass < 2; ++pass) {
        // S = C_a N~ C_a^T
        asm_form_S(r0, na, asm_rows, row_p, row_q, crow, Nt, S);
        __syncthreads();
        if (pass == 1) {
            // rank-deficient: symmetric pseudo-inverse (Sec. 3.1)
            if (threadIdx.x == 0) {
                sym_pinv_serial(S, X, na, G, 1e-12);
                atomicAdd(&status[1], 1);
            }
            return;
        }
        if (threadIdx.x == 0) {
            double mx = 0.0;
            for (int k = 0; k < na; ++k) mx = fmax(mx, S[(size_t)k * na + k]);
            dmax = mx;
            fail = 0;
        }
        // Cholesky in place (lower = L, upper = L^T), pivot test relative to max diagonal
        for (int k = 0; k < na; ++k) {
            __syncthreads();
            if (threadIdx.x == 0) {
                const double dd = S[(size_t)k * na + k];
                if (!(dd > 1e-12 * dmax)) {
                    fail = 1;
                } else {
                    const double s = sqrt(dd);
                    S[(size_t)k * na + k] = s;
                    col[k] = s;
                }
            }
            __syncthreads();
            if (fail) break;
            const double inv = 1.0 / col[k];
            for (int i = k + 1 + threadIdx.x; i < na; i += blockDim.x) {
                const double v = S[(size_t)i * na + k] * inv;
                S[(size_t)i * na + k] = v;
                S[(size_t)k * na + i] = v;
                col[i] = v;
            }
            __syncthreads();
            const int w = na - k - 1;
            for (int idx = threadIdx.x; idx < w * w; idx += blockDim.x) {
                const int ii = k + 1 + idx / w, jj = k + 1 + (idx - (idx / w) * w);
                S[(size_t)ii * na + jj] -= col[ii] * col[jj];
            }
        }
        __syncthreads();
        if (fail) continue;  // recompute S, then pseudo-inverse
        // X = L^-1 (row-major lower), column by column of the identity
        for (int idx = threadIdx.x; idx < na * na; idx += blockDim.x) {
            const int i = idx / na, j = idx - (idx / na) * na;
            X[idx] = (i == j) ? 1.0 : 0.0;
        }
        for (int k = 0; k < na; ++k) {
            __syncthreads();
            const double inv = 1.0 / S[(size_t)k * na + k];
            for (int j = threadIdx.x; j <= k; j += blockDim.x) X[(size_t)k * na + j] *= inv;
            __syncthreads();
            const int w = na - k - 1;
            for (int idx = threadIdx.x; idx < w * (k + 1); idx += blockDim.x) {
                const int i = k + 1 + idx / (k + 1), j = idx - (idx / (k + 1)) * (k + 1);
                X[(size_t)i * na + j] -= S[(size_t)i * na + k] * X[(size_t)k * na + j];
            }
        }
        __syncthreads();
        for (int idx = threadIdx.x; idx < na * na; idx += blockDim.x) {
            const int i = idx / na, j = idx - (idx / na) * na;
            double s = 0.0;
            for (int k = (i > j ? i : j); k < na; ++k)
                s += X[(size_t)k * na + i] * X[(size_t)k * na + j];
            G[idx] = s;
        }
        return;
    }
}

__device__ __forceinline__ double block_sum(double v, double *red) {
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < (int)(blockDim.x / kWave); ++k) s += red[k];
    return s;
}

// Row i of M_pp^-1 x, the part k = [k0, k1) of its sum.  The apply kernels give a row
// several threads, each a part, so that a workgroup keeps enough loads in flight: with
// one thread per row it waited on its m loads (51 us for the 1,591 plates of 64 diatom
// colonies, 43 us with parts).
__device__ __forceinline__ double row_part(const double *__restrict__ Mi, int m, int i, int k0,
                                           int k1, const double *x) {
    double s = 0.0;
#pragma unroll 8
    for (int k = k0; k < k1; ++k) s += Mi[(size_t)k * m + i] * x[k];
    return s;
}

constexpr int kApply = 1024;  // most threads of the apply kernels

__global__ __launch_bounds__(kApply) void pc_apply1_kernel(
    int N, const int *__restrict__ order, const int *__restrict__ blob_off, const int64_t *__restrict__ mat_off,
    const int64_t *__restrict__ z_off, const double *__restrict__ minv,
    const double *__restrict__ Zbuf, const double *__restrict__ Nt, const double *__restrict__ r,
    double *__restrict__ z, double *__restrict__ uhat) {
    __shared__ double x[kMaxM];
    __shared__ double part[kApply];
    __shared__ double w6[6];
    const int p = order ? order[blockIdx.x] : blockIdx.x, tid = threadIdx.x, T = blockDim.x;
    const int b0 = blob_off[p], m = 3 * (blob_off[p + 1] - b0);
    const double *Mi = minv + mat_off[p];
    const double *Z = Zbuf + z_off[p];
    const double *rl = r + 3 * (size_t)b0;
    for (int i = tid; i < m; i += T) x[i] = rl[i];
    __syncthreads();
    // t = Minv r_lam (Minv symmetric: column access is coalesced)
    const int ks = T / m;  // parts per row (0: more rows than threads)
    if (ks < 2) {
        for (int i = tid; i < m; i += T)
            z[3 * (size_t)b0 + i] = row_part(Mi, m, i, 0, m, x);
    } else {
        const int g = tid / m, i = tid - g * m;
        if (g < ks) part[tid] = row_part(Mi, m, i, m * g / ks, m * (g + 1) / ks, x);
    }
    // Z^T r_lam + r_U, a wavefront per component
    const int lane = tid % kWave, w = tid / kWave;
    for (int c = w; c < 6; c += T / kWave) {
        double s = 0.0;
        for (int i = lane; i < m; i += kWave) s += Z[(size_t)i * 6 + c] * x[i];
        for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) w6[c] = s + r[3 * (size_t)N + 6 * (size_t)p + c];
    }
    __syncthreads();
    if (ks >= 2 && tid < m) {
        double s = part[tid];
        for (int g = 1; g < ks; ++g) s += part[g * m + tid];
        z[3 * (size_t)b0 + tid] = s;
    }
    if (tid < 6) {
        const double *Nb = Nt + 36 * (size_t)p;
        double s = 0.0;
        for (int c = 0; c < 6; ++c) s += Nb[tid * 6 + c] * w6[c];
        uhat[6 * (size_t)p + tid] = -s;
    }
}

// The whole apply of small assemblies in one launch, in place of the three kernels
// around it, which stay for assemblies beyond the limits (precond_fuse: what LDS holds
// and one thread per row covers).  An assembly is taken by gridDim.y workgroups: each
// repeats the short chain Z^T r, U^, phi, U (a few kB of Z, N~, C, G~) and does its
// share of the rows of M_pp^-1 r + Z U, whose blocks are the traffic (590 kB for a 42-
// and an 80-blob body).  About 10 us of dependent loads and barriers up to 256
// workgroups, then bound by the blocks' bandwidth.  With alpha, r / alpha is applied and
// stored to v: GMRES scales its new basis vector here.  Against three kernels and the
// scaling (launches without their gaps): 16 bacteria 27.0 -> 10.7 us, 100 37.9 -> 18.6
// (59 MB, 3.2 TB/s), 1,000 free 42-blob shells 38.5 -> 26.2.  A chain of 20 bodies with 57 constraint rows: 22.6 us when each step
// searched bodies and rows one after the other, 14.8 with bisection and a mask of a body's
// rows (three kernels and the scaling 14.1 + 2.3 and two launches more).
constexpr int kFuseBlocks = 256;  // workgroups an apply is split into (100 bacteria with
                                  // 500: 26.7 us, with 1,000: 40.5: the chain is repeated)
constexpr int kFuseRows = 1024, kFuseBodies = 32, kFuseCons = 64;
// from kFuseMany assemblies on, two workgroups to a compute unit, only those of at most
// kFuseShort rows, a workgroup of 256 threads each: 1,024 threads and the LDS of the
// largest for every one of them run in turns (2,000 free bodies of 42 blobs and a chain of
// 8: 78 us, the three kernels 59; 8,000 of 6 blobs and the chain: 143, 37; 1,024 bacteria:
// 149, 129; all short, 4,000 bodies of 6 blobs: 27, 23 and the scaling's launch; 1,000
// shells of 42: 28, 36)
constexpr int kFuseMany = 512, kFuseShort = 256;

__host__ __device__ inline size_t fuse_doubles(const PcFuse &f, int threads) {
    return (size_t)f.rows + threads + 18 * f.bodies + (size_t)f.cons * (14 + f.cons);
}

__global__ __launch_bounds__(kApply) void pc_apply_asm_kernel(
    int N, int M, PrecondDev P, const double *__restrict__ r, const double *__restrict__ alpha,
    double *__restrict__ v, double *__restrict__ z) {
    extern __shared__ double lds[];
    __shared__ int s_p[kFuseBodies], s_row[kFuseBodies + 1], s_b[kFuseBodies];
    __shared__ int s_rows[kFuseCons], s_side[kFuseCons][2];  // rows; their bodies, local
    __shared__ uint64_t s_mask[kFuseBodies][2];              // rows of a body by side
    const int T = blockDim.x;
    double *x = lds, *part = x + P.fuse.rows, *y = part + T, *ph = y + P.fuse.cons;
    double(*ru)[6] = reinterpret_cast<double(*)[6]>(ph + P.fuse.cons);
    double(*w6)[6] = ru + P.fuse.bodies, (*uh)[6] = w6 + P.fuse.bodies;
    double(*cr)[12] = reinterpret_cast<double(*)[12]>(uh + P.fuse.bodies);
    double *G = cr[P.fuse.cons];
    const int a = blockIdx.x, tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
    const bool first = blockIdx.y == 0;  // writes z_U, z_phi and their part of v
    const int bp = P.asm_body_ptr[a], nb = P.asm_body_ptr[a + 1] - bp;
    const int r0 = P.asm_row_ptr[a], na = P.asm_row_ptr[a + 1] - r0;
    const size_t off_u = 3 * (size_t)N, off_phi = off_u + 6 * (size_t)M;
    const double al = alpha ? alpha[0] : 1.0;
    auto load = [&](size_t i, bool mine) {
        double t = r[i];
        if (alpha) {
            t /= al;
            if (mine) v[i] = t;
        }
        return t;
    };
    if (w == 0) {  // the bodies' rows, numbered through
        int m = 0;
        if (lane < nb) {
            const int p = P.asm_bodies[bp + lane];
            s_p[lane] = p;
            s_b[lane] = 3 * P.blob_off[p];
            m = 3 * P.blob_off[p + 1] - s_b[lane];
        }
        for (int off = 1; off < kFuseBodies; off <<= 1) {
            const int u = __shfl_up(m, off);
            if (lane >= off) m += u;
        }
        if (lane < nb) s_row[lane + 1] = m;
        if (lane == 0) s_row[0] = 0;
    }
    if (tid < na) s_rows[tid] = P.asm_rows[r0 + tid];
    for (int e = tid; e < na * na; e += T) G[e] = P.G[P.asm_mat_off[a] + e];
    __syncthreads();
    const int mt = s_row[nb];
    const int i0 = mt * blockIdx.y / gridDim.y, nr = mt * (blockIdx.y + 1) / gridDim.y - i0;
    // last i < n with a[i] <= v (a ascending, a[0] <= v)
    auto last_at_most = [](const int *a, int n, int v) {
        int i = 0;
#pragma unroll
        for (int step = kFuseBodies / 2; step > 0; step /= 2)
            if (i + step < n && a[i + step] <= v) i += step;
        return i;
    };
    auto body_of = [&](int row) { return last_at_most(s_row, nb, row); };
    for (int i = tid; i < mt; i += T) {
        const int b = body_of(i);
        x[i] = load((size_t)s_b[b] + (i - s_row[b]), i >= i0 && i < i0 + nr);
    }
    // a thread per (body, component) and per constraint row.  All that the chain below
    // reads is loaded here: its steps then wait on barriers only, not on memory
    const int eb = tid / 6, ec = tid - 6 * eb;
    double Nb[6];
    if (eb < nb) {
        ru[eb][ec] = load(off_u + 6 * (size_t)s_p[eb] + ec, first);
        for (int c = 0; c < 6; ++c) Nb[c] = P.Nt[36 * (size_t)s_p[eb] + 6 * ec + c];
    }
    if (tid < na) y[tid] = load(off_phi + s_rows[tid], first);
    for (int e = tid; e < 12 * na; e += T)
        cr[e / 12][e % 12] = P.crow[12 * (size_t)s_rows[e / 12] + e % 12];
    for (int e = tid; e < 2 * na; e += T) {
        const int p = (e & 1) ? P.row_q[s_rows[e / 2]] : P.row_p[s_rows[e / 2]];
        s_side[e / 2][e & 1] = p >= 0 ? last_at_most(s_p, nb, p) : -1;
    }
    __syncthreads();
    // parts of t = M_pp^-1 r_lam
    // at most 16, whose sums one thread adds up at the end (8, 16, 32 or 64: within 3 % from
    // 16 to 1,024 bacteria and for chains; 8 and fewer lose up to 14 % where bodies are small)
    const int ks = nr ? min(T / nr, 16) : 0, g = nr ? tid / nr : 0, row = tid - g * nr;
    int b = 0, il = 0;
    if (g < ks) {
        b = body_of(i0 + row);
        il = i0 + row - s_row[b];
        const int m = s_row[b + 1] - s_row[b];
        part[tid] = row_part(P.minv + P.mat_off[s_p[b]], m, il, m * g / ks, m * (g + 1) / ks,
                             x + s_row[b]);
    }
    // Z^T r_lam + r_U, a wavefront per (body, component)
    for (int e = w; e < 6 * nb; e += T / kWave) {
        const int q = e / 6, c = e % 6, m = s_row[q + 1] - s_row[q];
        const double *Z = P.Z + P.z_off[s_p[q]];
        double s = 0.0;
        for (int i = lane; i < m; i += kWave) s += Z[(size_t)i * 6 + c] * x[s_row[q] + i];
        for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) w6[q][c] = s + ru[q][c];
    }
    // the rows of each body, a bit per row
    for (int q = w; q < nb && na > 0; q += T / kWave)
        for (int side = 0; side < 2; ++side) {
            const uint64_t m = __ballot(lane < na && s_side[min(lane, kFuseCons - 1)][side] == q);
            if (lane == 0) s_mask[q][side] = m;
        }
    __syncthreads();
    if (eb < nb) {  // U^
        double s = 0.0;
        for (int c = 0; c < 6; ++c) s += Nb[c] * w6[eb][c];
        uh[eb][ec] = -s;
    }
    __syncthreads();
    if (tid < na) {
        const int q = s_side[tid][1];
        const double *Up = uh[s_side[tid][0]];
        double s = 0.0;
        for (int u = 0; u < 6; ++u) s += cr[tid][u] * Up[u];
        if (q >= 0)
            for (int u = 0; u < 6; ++u) s += cr[tid][6 + u] * uh[q][u];
        y[tid] -= s;
    }
    __syncthreads();
    if (tid < na) {
        double s = 0.0;
#pragma unroll 8
        for (int l = 0; l < na; ++l) s += G[tid * na + l] * y[l];
        ph[tid] = s;
        if (first) z[off_phi + s_rows[tid]] = s;
    }
    __syncthreads();
    if (eb < nb) {  // f = C^T phi per body
        double s = 0.0;
        const uint64_t q = na > 0 ? s_mask[eb][1] : 0;
        for (uint64_t m = na > 0 ? s_mask[eb][0] | q : 0; m; m &= m - 1) {
            const int t = __builtin_ctzll(m);
            s += ph[t] * cr[t][6 * (int)(q >> t & 1) + ec];
        }
        w6[eb][ec] = s;
    }
    __syncthreads();
    if (eb < nb) {  // U = U^ + N~ f
        double s = uh[eb][ec];
        for (int c = 0; c < 6; ++c) s += Nb[c] * w6[eb][c];
        ru[eb][ec] = s;
        if (first) z[off_u + 6 * (size_t)s_p[eb] + ec] = s;
    }
    __syncthreads();
    if (tid < nr) {
        double s = part[tid];
        for (int q = 1; q < ks; ++q) s += part[q * nr + tid];
        const double *Z = P.Z + P.z_off[s_p[b]] + (size_t)il * 6;
        double d = 0.0;
        for (int c = 0; c < 6; ++c) d += Z[c] * ru[b][c];
        z[(size_t)s_b[b] + il] = s + d;
    }
}

PcFuse precond_fuse(int A, const int *body_ptr, const int *bodies, const int *row_ptr,
                    const int *blob_off) {
    PcFuse f;
    for (int a = 0; a < A; ++a) {
        int64_t rows = 0;
        for (int e = body_ptr[a]; e < body_ptr[a + 1]; ++e)
            rows += 3 * (int64_t)(blob_off[bodies[e] + 1] - blob_off[bodies[e]]);
        const int nb = body_ptr[a + 1] - body_ptr[a], na = row_ptr[a + 1] - row_ptr[a];
        if (nb > kFuseBodies || na > kFuseCons || rows > kFuseRows) return PcFuse();
        f.rows = std::max(f.rows, (int)rows);
        f.bodies = std::max(f.bodies, nb);
        f.cons = std::max(f.cons, na);
    }
    return A >= kFuseMany && f.rows > kFuseShort ? PcFuse() : f;
}

__global__ __launch_bounds__(256) void pc_apply2_kernel(
    int N, int M, const int *__restrict__ asm_row_ptr, const int *__restrict__ asm_rows,
    const int64_t *__restrict__ asm_mat_off, const int *__restrict__ row_p,
    const int *__restrict__ row_q, const double *__restrict__ crow, const double *__restrict__ Gbuf,
    const double *__restrict__ r, const double *__restrict__ uhat, double *__restrict__ z) {
    __shared__ double y[kMaxAsmRows];
    const int a = blockIdx.x;
    const int r0 = asm_row_ptr[a], na = asm_row_ptr[a + 1] - r0;
    if (na == 0) return;
    const double *G = Gbuf + asm_mat_off[a];
    const size_t off_phi = 3 * (size_t)N + 6 * (size_t)M;
    for (int k = threadIdx.x; k < na; k += blockDim.x) {
        const int rk = asm_rows[r0 + k];
        const double *c = crow + 12 * (size_t)rk;
        const double *Up = uhat + 6 * (size_t)row_p[rk];
        double s = 0.0;
        for (int u = 0; u < 6; ++u) s += c[u] * Up[u];
        const int q = row_q[rk];
        if (q >= 0) {
            const double *Uq = uhat + 6 * (size_t)q;
            for (int u = 0; u < 6; ++u) s += c[6 + u] * Uq[u];
        }
        y[k] = r[off_phi + rk] - s;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < na; k += blockDim.x) {
        double s = 0.0;
        for (int l = 0; l < na; ++l) s += G[(size_t)k * na + l] * y[l];
        z[off_phi + asm_rows[r0 + k]] = s;
    }
}

__global__ __launch_bounds__(256) void pc_apply3_kernel(
    int N, int M, const int *__restrict__ blob_off, const int64_t *__restrict__ z_off,
    const double *__restrict__ Zbuf, const double *__restrict__ Nt,
    const int *__restrict__ brow_ptr, const int *__restrict__ brow_ent,
    const double *__restrict__ crow, const double *__restrict__ uhat, double *__restrict__ z,
    int has_rows) {
    __shared__ double U[6];
    __shared__ double f[6];
    const int p = blockIdx.x;
    const size_t off_phi = 3 * (size_t)N + 6 * (size_t)M;
    if (threadIdx.x < 6) {
        double s = 0.0;
        if (has_rows) {
            for (int e = brow_ptr[p]; e < brow_ptr[p + 1]; ++e) {
                const int ent = brow_ent[e];
                const int row = ent >> 1, side = ent & 1;
                s += z[off_phi + row] * crow[12 * (size_t)row + 6 * side + threadIdx.x];
            }
        }
        f[threadIdx.x] = s;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const double *Nb = Nt + 36 * (size_t)p;
        double s = uhat[6 * (size_t)p + threadIdx.x];
        for (int c = 0; c < 6; ++c) s += Nb[threadIdx.x * 6 + c] * f[c];
        U[threadIdx.x] = s;
        z[3 * (size_t)N + 6 * (size_t)p + threadIdx.x] = s;
    }
    __syncthreads();
    const int b0 = blob_off[p], m = 3 * (blob_off[p + 1] - b0);
    const double *Z = Zbuf + z_off[p];
    for (int i = threadIdx.x; i < m; i += blockDim.x) {
        double s = 0.0;
        for (int c = 0; c < 6; ++c) s += Z[(size_t)i * 6 + c] * U[c];
        z[3 * (size_t)b0 + i] += s;
    }
}


// Per-type variants (learned body mobility and body-frame blocks): each body's
// block starts from the unbounded blob mobility of its type in the body frame
// (factored once), rotated by R_p: A_p = (I x R) Minv_type (I x R^T),
// Z_f = A_p K_p = (I x R) Z_type Q^T with Q = diag(R, R), N~_f = Q N~_type Q^T.
// Body-frame variant: N~_p = N~_f, an exact block solve of the unbounded blocks.
// Learned variant: the network gives the wall body mobility N~_w, and the blob
// block is modified by a rank-6 term so that the block solve stays exact for
// a consistent pair (M~, N~_w):
//   M~^-1 = A_p + Z_f D Z_f^T,  D = N~_f N~_w^-1 N~_f - N~_f,
// which gives K^T M~^-1 K = N~_w^-1 and K^T M~^-1 = N~_w^-1 N~_f Z_f^T.  Per body
// E1 = D and E2 = D N~_f^-1 are formed at build time; the apply then reads
//   U^ = -N~_w r_U - N~_f s,  s = Z_f^T r_lam,
//   lam = A_p r_lam + Z_f (U + E1 s + E2 U),
// with U = U^ + N~_w C^T phi as in the exact variant.
__global__ __launch_bounds__(256) void pc_apply1_learned_kernel(
    int N, const int *__restrict__ blob_off, const int *__restrict__ type,
    const int64_t *__restrict__ tmat_off, const int64_t *__restrict__ tz_off,
    const double *__restrict__ tminv, const double *__restrict__ tZ, const double *__restrict__ R9,
    const double *__restrict__ Nt, const double *__restrict__ lcorr, const double *__restrict__ r,
    double *__restrict__ z, double *__restrict__ uhat, double *__restrict__ stmp) {
    __shared__ double x[kMaxM];
    __shared__ double tb[kMaxM];
    __shared__ double red[8];
    __shared__ double w6[6];
    __shared__ double R[9];
    const int p = blockIdx.x;
    const int b0 = blob_off[p], n = blob_off[p + 1] - b0, m = 3 * n;
    const int ty = type[p];
    const double *Mi = tminv + tmat_off[ty];
    const double *Z = tZ + tz_off[ty];
    if (threadIdx.x < 9) R[threadIdx.x] = R9[9 * (size_t)p + threadIdx.x];
    __syncthreads();
    const double *rl = r + 3 * (size_t)b0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {  // x_b = R^T r_lam (per blob)
        const double a0 = rl[3 * i], a1 = rl[3 * i + 1], a2 = rl[3 * i + 2];
        for (int c = 0; c < 3; ++c) x[3 * i + c] = R[c] * a0 + R[3 + c] * a1 + R[6 + c] * a2;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += blockDim.x) {
        double s = 0.0;
        for (int k = 0; k < m; ++k) s += Mi[(size_t)k * m + i] * x[k];
        tb[i] = s;
    }
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int i = threadIdx.x; i < m; i += blockDim.x)
        for (int c = 0; c < 6; ++c) acc[c] += Z[(size_t)i * 6 + c] * x[i];
    double zb[6];
    for (int c = 0; c < 6; ++c) zb[c] = block_sum(acc[c], red);  // syncs: tb complete
    for (int i = threadIdx.x; i < n; i += blockDim.x) {  // t_p = R t_b
        const double a0 = tb[3 * i], a1 = tb[3 * i + 1], a2 = tb[3 * i + 2];
        for (int c = 0; c < 3; ++c)
            z[3 * (size_t)b0 + 3 * i + c] = R[3 * c] * a0 + R[3 * c + 1] * a1 + R[3 * c + 2] * a2;
    }
    __shared__ double s6[6];
    if (threadIdx.x < 6) {
        // s = Z_f^T r_lam = Q (Z_type^T x_b)
        const int h = threadIdx.x / 3, c = threadIdx.x % 3;
        const double v = R[3 * c] * zb[3 * h] + R[3 * c + 1] * zb[3 * h + 1] + R[3 * c + 2] * zb[3 * h + 2];
        const double ru = r[3 * (size_t)N + 6 * (size_t)p + threadIdx.x];
        s6[threadIdx.x] = v;
        w6[threadIdx.x] = lcorr ? ru : v + ru;
        if (lcorr) stmp[6 * (size_t)p + threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const double *Nb = Nt + 36 * (size_t)p;
        double acc = 0.0;
        for (int c = 0; c < 6; ++c) acc += Nb[threadIdx.x * 6 + c] * w6[c];
        if (lcorr) {  // - N~_f s
            const double *Nf = lcorr + 108 * (size_t)p;
            for (int c = 0; c < 6; ++c) acc += Nf[threadIdx.x * 6 + c] * s6[c];
        }
        uhat[6 * (size_t)p + threadIdx.x] = -acc;
    }
}

__global__ __launch_bounds__(256) void pc_apply3_learned_kernel(
    int N, int M, const int *__restrict__ blob_off, const int *__restrict__ type,
    const int64_t *__restrict__ tz_off, const double *__restrict__ tZ, const double *__restrict__ R9,
    const double *__restrict__ Nt, const double *__restrict__ lcorr,
    const double *__restrict__ stmp, const int *__restrict__ brow_ptr,
    const int *__restrict__ brow_ent, const double *__restrict__ crow,
    const double *__restrict__ uhat, double *__restrict__ z, int has_rows) {
    __shared__ double U[6], V[6], Ub[6], f[6], R[9];
    const int p = blockIdx.x;
    const size_t off_phi = 3 * (size_t)N + 6 * (size_t)M;
    if (threadIdx.x < 9) R[threadIdx.x] = R9[9 * (size_t)p + threadIdx.x];
    if (threadIdx.x < 6) {
        double s = 0.0;
        if (has_rows) {
            for (int e = brow_ptr[p]; e < brow_ptr[p + 1]; ++e) {
                const int ent = brow_ent[e];
                const int row = ent >> 1, side = ent & 1;
                s += z[off_phi + row] * crow[12 * (size_t)row + 6 * side + threadIdx.x];
            }
        }
        f[threadIdx.x] = s;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const double *Nb = Nt + 36 * (size_t)p;
        double s = uhat[6 * (size_t)p + threadIdx.x];
        for (int c = 0; c < 6; ++c) s += Nb[threadIdx.x * 6 + c] * f[c];
        U[threadIdx.x] = s;
        z[3 * (size_t)N + 6 * (size_t)p + threadIdx.x] = s;
    }
    __syncthreads();
    if (threadIdx.x < 6) {  // V = U (+ E1 s + E2 U with the learned correction)
        double v = U[threadIdx.x];
        if (lcorr) {
            const double *E1 = lcorr + 108 * (size_t)p + 36, *E2 = E1 + 36;
            const double *sp = stmp + 6 * (size_t)p;
            for (int c = 0; c < 6; ++c) v += E1[threadIdx.x * 6 + c] * sp[c] + E2[threadIdx.x * 6 + c] * U[c];
        }
        V[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x < 6) {  // Q^T V
        const int h = threadIdx.x / 3, c = threadIdx.x % 3;
        Ub[threadIdx.x] = R[c] * V[3 * h] + R[3 + c] * V[3 * h + 1] + R[6 + c] * V[3 * h + 2];
    }
    __syncthreads();
    const int b0 = blob_off[p], n = blob_off[p + 1] - b0;
    const double *Z = tZ + tz_off[type[p]];
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        double v[3];
        for (int c = 0; c < 3; ++c) {
            double s = 0.0;
            for (int k = 0; k < 6; ++k) s += Z[(size_t)(3 * i + c) * 6 + k] * Ub[k];
            v[c] = s;
        }
        for (int c = 0; c < 3; ++c)
            z[3 * (size_t)b0 + 3 * i + c] += R[3 * c] * v[0] + R[3 * c + 1] * v[1] + R[3 * c + 2] * v[2];
    }
}

// N~_p = Q N~_type Q^T, Q = diag(R_p, R_p): the free-space body mobility of
// the body's type rotated into its orientation (no wall)
__global__ void pc_rotate_nt_kernel(int M, const int *__restrict__ type,
                                    const double *__restrict__ tNt, const double *__restrict__ R9,
                                    double *__restrict__ Nt) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= M) return;
    const double *R = R9 + 9 * (size_t)p;
    const double *A = tNt + 36 * (size_t)type[p];
    double T[36];
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) {  // (Q A)_ij
            const int bi = i / 3, ri = i % 3;
            double s = 0.0;
            for (int k = 0; k < 3; ++k) s += R[3 * ri + k] * A[(3 * bi + k) * 6 + j];
            T[i * 6 + j] = s;
        }
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) {  // (Q A) Q^T
            const int bj = j / 3, rj = j % 3;
            double s = 0.0;
            for (int k = 0; k < 3; ++k) s += T[i * 6 + 3 * bj + k] * R[3 * rj + k];
            Nt[36 * (size_t)p + i * 6 + j] = s;
        }
}

// 6 x 6 SPD inverse by Cholesky; false if a pivot is not positive
__device__ bool spd6_inverse(const double *A, double *X) {
    double L[36] = {};
    for (int j = 0; j < 6; ++j) {
        double d = A[j * 6 + j];
        for (int k = 0; k < j; ++k) d -= L[j * 6 + k] * L[j * 6 + k];
        if (!(d > 0.0)) return false;
        L[j * 6 + j] = sqrt(d);
        for (int i = j + 1; i < 6; ++i) {
            double v = 0.5 * (A[i * 6 + j] + A[j * 6 + i]);
            for (int k = 0; k < j; ++k) v -= L[i * 6 + k] * L[j * 6 + k];
            L[i * 6 + j] = v / L[j * 6 + j];
        }
    }
    for (int c = 0; c < 6; ++c) {  // X e_c = L^-T L^-1 e_c
        double y[6];
        for (int i = 0; i < 6; ++i) {
            double v = i == c ? 1.0 : 0.0;
            for (int k = 0; k < i; ++k) v -= L[i * 6 + k] * y[k];
            y[i] = v / L[i * 6 + i];
        }
        for (int i = 5; i >= 0; --i) {
            double v = y[i];
            for (int k = i + 1; k < 6; ++k) v -= L[k * 6 + i] * y[k];
            y[i] = v / L[i * 6 + i];
        }
        for (int i = 0; i < 6; ++i) X[i * 6 + c] = y[i];
    }
    return true;
}

// per body: N~_f (rotated type mobility), E1 = N~_f N~_w^-1 N~_f - N~_f,
// E2 = E1 N~_f^-1 (108 doubles); flags bodies whose N~_w or N~_f is not SPD
__global__ void pc_learned_corr_kernel(int M, const int *__restrict__ type,
                                       const double *__restrict__ tNt,
                                       const double *__restrict__ R9,
                                       const double *__restrict__ Nw, double *__restrict__ out,
                                       int *__restrict__ bad) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= M) return;
    const double *R = R9 + 9 * (size_t)p;
    const double *A = tNt + 36 * (size_t)type[p];
    double T[36], Nf[36], Wi[36], Fi[36];
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) {
            const int bi = i / 3, ri = i % 3;
            double s = 0.0;
            for (int k = 0; k < 3; ++k) s += R[3 * ri + k] * A[(3 * bi + k) * 6 + j];
            T[i * 6 + j] = s;
        }
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) {
            const int bj = j / 3, rj = j % 3;
            double s = 0.0;
            for (int k = 0; k < 3; ++k) s += T[i * 6 + 3 * bj + k] * R[3 * rj + k];
            Nf[i * 6 + j] = s;
        }
    const bool ok = spd6_inverse(Nw + 36 * (size_t)p, Wi) && spd6_inverse(Nf, Fi);
    if (!ok) atomicOr(bad, 1);
    double *o = out + 108 * (size_t)p;
    for (int k = 0; k < 36; ++k) o[k] = Nf[k];
    double WN[36], E1[36];
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) {
            double s = 0.0;
            for (int k = 0; k < 6; ++k) s += Wi[i * 6 + k] * Nf[k * 6 + j];
            WN[i * 6 + j] = s;
        }
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) {
            double s = -Nf[i * 6 + j];
            for (int k = 0; k < 6; ++k) s += Nf[i * 6 + k] * WN[k * 6 + j];
            E1[i * 6 + j] = ok ? s : 0.0;
        }
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) {
            double s = 0.0;
            for (int k = 0; k < 6; ++k) s += E1[i * 6 + k] * Fi[k * 6 + j];
            o[36 + i * 6 + j] = E1[i * 6 + j];
            o[72 + i * 6 + j] = ok ? s : 0.0;
        }
}

void learned_correction(hipStream_t s, int M, const int *type, const double *tNt,
                        const double *R9, const double *Nw, double *out, int *bad) {
    if (M > 0)
        pc_learned_corr_kernel<<<(M + 255) / 256, 256, 0, s>>>(M, type, tNt, R9, Nw, out, bad);
}

void rotate_body_mobility(hipStream_t s, int M, const int *type, const double *tNt,
                          const double *R9, double *Nt) {
    if (M > 0) pc_rotate_nt_kernel<<<(M + 255) / 256, 256, 0, s>>>(M, type, tNt, R9, Nt);
}

void precond_assemble(hipStream_t s, const PrecondDev &P, const double *pos, double a, double eta,
                      bool wall) {
    if (P.M <= 0) return;
    const CoefD c = make_coef<CoefD, double>(a);
    // a few bodies: several workgroups each
    const int parts = std::min(16, std::max(1, 1024 / P.M));
    pc_assemble_kernel<<<dim3(P.M, parts), 256, 0, s>>>(P.order, P.blob_off, P.mat_off, pos, c,
                                                        1.0 / (8 * kPi * eta), wall ? 1 : 0, a,
                                                        P.mats, P.status);
}

// SPD inverse of each matrix of the batch by the symmetric block sweep (block
// Gauss-Jordan elimination without pivoting, which positive definite matrices
// allow; the pivot blocks are the Schur complements of the Cholesky
// factorisation), out of place, for matrices of at most kSwRows rows.  One
// workgroup per matrix holds its lower triangle in registers as 16 x 16 tiles in the
// matrix-core accumulator layout: tile t = (ti, tj), tj <= ti, counted row by row,
// belongs to wavefront t % WAVES (slot t / WAVES).  Rows beyond m are padded with the
// identity.  Sweeping block k with P = A_kk^-1 takes, with the values before the step,
//   A_ij -= A_ik P A_kj (i, j != k),   A_ik <- A_ik P,   A_kk <- -P,
// which keeps the matrix symmetric; after the last block it holds -A^-1.  Per step:
// W_r = C_r P (C_r = A_rk) is formed on the matrix cores, block row r by wavefront
// r % WAVES; then every wavefront updates its tiles there, A_ij -= W_i C_j^T.  The
// next step's serial part runs under that update: the wavefront that holds A_k+1,k+1
// updates it first and inverts it in registers (sweep_invert16), and the tiles of
// block column k+1 go to the other C buffer as they are updated, so a step has two
// barriers.  The flop count equals that of factor, triangular inverse and product
// (m^3 in all), with the matrix read once and its inverse (both triangles) written
// once.  Dynamic LDS: two C, W, and two each of P, P^T and A_kk, 16 nb or 16 rows of
// kSwLd doubles.
// Bound by the matrix cores and by memory in turn: one 240-row matrix takes 118 us (51 at
// the FP64 peak of one compute unit; 159 with the inverse between barriers and a branch
// per tile), of which the updates are 12,000 of 15,400 cycles a step, two wavefronts to a
// SIMD.  16 wavefronts spill (114 us, 534 for 512 bacteria against 541 then).  512 bacteria
// (a 126- and a 240-row matrix each): 688 -> 399 us, most of it from the order
// (MatBatch::order).
constexpr int kSwRows = 256;
// matrices of at most kSwSmall tile rows (144 rows) take an instance with fewer
// registers, two or more workgroups per compute unit
constexpr int kSwSmall = kSweepSmall / 16;

size_t sweep_lds_bytes(int max_m) {
    const int nb = (max_m + 15) / 16;
    return sweep_lds(nb).end * sizeof(double);
}

// lane Q of each row of 16 lanes, to the whole row
template <int Q>
__device__ __forceinline__ double row_bcast(double x) {
    return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + Q, 0xf, 0xf, true);
}

// row G of 16 lanes, to all four rows
template <int G>
__device__ __forceinline__ unsigned all_rows(unsigned x) {
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const unsigned y = h[G >> 1];
    const auto r = __builtin_amdgcn_permlane16_swap(y, y, false, false);
    return r[G & 1];
}

// D_Q,c in every row of lanes, and its entry Q
template <int Q>
__device__ __forceinline__ void sweep_pivot_row(const double *d, double &row, double &piv) {
    row = __hiloint2double(all_rows<Q & 3>(__double2hiint(d[Q >> 2])),
                           all_rows<Q & 3>(__double2loint(d[Q >> 2])));
    piv = row_bcast<Q>(row);
}

// one pivot of sweep_invert16; row, piv, ip = 1 / piv of this pivot, then of the next,
// whose row is updated first: its reciprocal's chain runs under the other rows' updates
template <int Q>
__device__ __forceinline__ void sweep_pivot(double *d, int lr, int lc, double tol, bool &bad,
                                            double &mypiv, double &row, double &piv, double &ip) {
    // a failed pivot is recorded, the (meaningless) steps still run
    bad |= !(piv > tol);
    mypiv = lr == 0 && lc == Q ? piv : mypiv;
    // pivot row scaled, pivot column scaled and negated, the rest eliminated: the pivot
    // column takes the elimination's form with 0 in place of the entry
    const double rq = lc == Q ? ip : row * ip;
    auto eliminate = [&](int e) {
        const double el = fma(-row_bcast<Q>(d[e]), rq, lc == Q ? 0.0 : d[e]);
        d[e] = e == (Q >> 2) && lr == (Q & 3) ? rq : el;
    };
    constexpr int kNext = Q < 15 ? Q + 1 : Q, e0 = kNext >> 2;
    eliminate(e0);
    if (Q < 15) sweep_pivot_row<kNext>(d, row, piv);
    __builtin_amdgcn_sched_barrier(0);
    // 1 / piv: the hardware estimate and two Newton steps
    ip = __builtin_amdgcn_rcp(piv);
    eliminate((e0 + 1) & 3);
    double t = fma(-piv, ip, 1.0);
    ip = fma(t, ip, ip);
    eliminate((e0 + 2) & 3);
    t = fma(-piv, ip, 1.0);
    ip = fma(t, ip, ip);
    eliminate((e0 + 3) & 3);
    __builtin_amdgcn_sched_barrier(0);
}

// D <- D^-1 by Gauss-Jordan steps in one wavefront, lane l holding D[4 e + l / 16][l % 16]:
// lane moves only (through LDS, which every pivot wrote and read again, a block took
// about 5 us).  Lane q < 16 gets pivot q; false if a pivot was not above tol.
template <int... Q>
__device__ __forceinline__ bool sweep_invert16(double *d, int lr, int lc, double tol,
                                               double &mypiv, std::integer_sequence<int, Q...>) {
    bool bad = false;
    double row, piv;
    sweep_pivot_row<0>(d, row, piv);
    double ip = __builtin_amdgcn_rcp(piv);
    ip = fma(fma(-piv, ip, 1.0), ip, ip);
    ip = fma(fma(-piv, ip, 1.0), ip, ip);
    (sweep_pivot<Q>(d, lr, lc, tol, bad, mypiv, row, piv, ip), ...);
    return !bad;
}

// NBMAX: the most tile rows this instance holds (matrices of more are skipped)
template <int NBMAX, int WAVES>
__global__ __launch_bounds__(64 * WAVES, NBMAX <= kSwSmall ? 4 : 2) void pc_sweep_kernel(MatBatch B) {
    constexpr int kSwSlots = (NBMAX * (NBMAX + 1) / 2 + WAVES - 1) / WAVES;
    // slots without a branch between them
    constexpr int kRun = 3;
    extern __shared__ double sw_lds[];
    __shared__ int fail;
    __shared__ double piv_tol;
    __shared__ double red[WAVES];
    const int p = B.order ? B.order[blockIdx.x] : blockIdx.x;
    if (mat_skip(B, p)) return;
    const int m = mat_rows(B, p);
    const int nb = (m + 15) >> 4, T = nb * (nb + 1) / 2;
    if (nb == 0 || nb > NBMAX) return;
    const SweepLds S = sweep_lds(nb);
    const int buf = S.buf, oW = S.W, oP = S.P, oT = S.T, oD = S.D;
    const double *A = B.mats + B.mat_off[p];
    double *Out = B.out + B.mat_off[p];
    const int tid = threadIdx.x, l = tid & 63, lr = l >> 4, lc = l & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this wavefront's tiles t0 .. t0 + nt - 1, row by row; row | column << 8 in scalar
    // registers.  Wavefront 0 inverts the diagonal blocks and takes what the others leave
    const int per = min(kSwSlots, (T + WAVES - 2) / (WAVES - 1));
    const int t0 = min(T, (w > 0 ? w - 1 : WAVES - 1) * per), nt = min(per, T - t0);
    int tij[kSwSlots];
    int li = kSwNone, lj = kSwNone;  // lane s: the tile of slot s
    {
        int i = 0, j = t0;
        for (; j > i; ++i) j -= i + 1;
#pragma unroll
        for (int s = 0; s < kSwSlots; ++s) {
            tij[s] = __builtin_amdgcn_readfirstlane(i | j << 8);
            if (l == s && s < nt) {
                li = i;
                lj = j;
            }
            if (++j > i) {
                j = 0;
                ++i;
            }
        }
    }
    // load the lower triangle (the upper part of diagonal tiles by symmetry), from offsets
    // clamped into the matrix, a run of slots at a time (a branch, an address and a wait
    // per entry took 17 us of 160)
    mfma_acc acc[kSwSlots];
    double dloc = 0.0;
    unsigned o_diag[4];  // entry (4 e + lr, lc) of a diagonal tile, taken from below
#pragma unroll
    for (int e = 0; e < 4; ++e) o_diag[e] = max(4 * e + lr, lc) * m + min(4 * e + lr, lc);
    const unsigned o_tile = lr * m + lc;
#pragma unroll
    for (int s0 = 0; s0 < kSwSlots; s0 += kRun) {
        if (s0 >= nt) continue;
#pragma unroll
        for (int s = s0; s < kSwSlots && s < s0 + kRun; ++s) {
            const int i = min(tij[s] & 255, nb - 1), j = min(tij[s] >> 8, nb - 1);
            const unsigned at = 16 * (i * m + j), last = m * m - 1 - at;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[s][e] = A[at + min(i == j ? o_diag[e] : o_tile + 4 * e * m, last)];
        }
#pragma unroll
        for (int s = s0; s < kSwSlots && s < s0 + kRun; ++s) {
            const int i = tij[s] & 255, j = tij[s] >> 8;
            if (i >= nb - 1)  // the last tile row: the identity beyond m
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (16 * i + 4 * e + lr >= m || 16 * j + lc >= m)
                        acc[s][e] = i == j && 4 * e + lr == lc ? 1.0 : 0.0;
            if (i == j && i < nb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * e + lr == lc && 16 * i + lc < m) dloc = fmax(dloc, acc[s][e]);
        }
    }
    if (B.rel_tol > 0.0) {
        for (int o = 32; o > 0; o >>= 1) dloc = fmax(dloc, __shfl_xor(dloc, o));
        if (l == 0) red[w] = dloc;
    }
    if (tid == 0) fail = 0;
    __syncthreads();
    if (tid == 0) {
        double dmax = 0.0;
        if (B.rel_tol > 0.0)
            for (int q = 0; q < WAVES; ++q) dmax = fmax(dmax, red[q]);
        piv_tol = B.rel_tol * dmax;
    }
    // lane offsets into rows and columns of a 16 x 16 LDS block.  They pass through an
    // empty asm every step: hoisted out of the loop, two addresses a tile would spill
    int o_row = lc * kSwLd + lr, o_col = lr * kSwLd + lc;
    // tiles after step k - 1: those of block column k to its buffer, A_k+1,k+1 to where
    // wavefront 0 takes it up
    auto publish = [&](int k) __attribute__((always_inline)) {
        const bool diag = li == lj && li == k + 1;
        // as rows of the buffer (i, k), or transposed (k, j)
        const bool col = lj == k || diag;
        const uint64_t sel = __ballot(diag || (li == k) != (lj == k));
        const int base = diag ? oD + 16 * (li & 1) * kSwLd
                              : (k & 1) * buf + 16 * (col ? li : lj) * kSwLd;
        const uint64_t cols = __ballot(col);
        const int o_diff = o_col - o_row;
#pragma unroll
        for (int s = 0; s < kSwSlots; ++s) {
            const int at = __builtin_amdgcn_readlane(base, s);
            const bool c = cols >> s & 1;
            double *q = sw_lds + at + o_row + (c ? o_diff : 0);
            const int st = c ? 4 * kSwLd : 4;
            if (sel >> s & 1) {
                q[0] = acc[s][0];
                q[st] = acc[s][1];
                q[2 * st] = acc[s][2];
                q[3 * st] = acc[s][3];
            }
        }
    };
    // wavefront 0: A_kk, its update by the step before (none before the first), P
    auto invert = [&](int k) __attribute__((always_inline)) {
        const double *D = sw_lds + oD + 16 * (k & 1) * kSwLd + o_col;
        mfma_acc x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = D[4 * e * kSwLd];
        if (k > 0) {
            const double *W = sw_lds + oW + 16 * k * kSwLd + o_row;
            const double *C = sw_lds + ((k - 1) & 1) * buf + 16 * k * kSwLd + o_row;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) x = mfma_f64_16x16x4(W[4 * kk], C[4 * kk], x);
        }
        double d[4] = {x[0], x[1], x[2], x[3]};
        double mypiv = 1.0;  // lane q < 16: pivot q
        const bool ok = sweep_invert16(d, lr, lc, piv_tol, mypiv,
                                       std::make_integer_sequence<int, 16>());
        double *P = sw_lds + oP + 16 * (k & 1) * kSwLd + o_col;
        double *PT = sw_lds + oT + 16 * (k & 1) * kSwLd + o_row;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            P[4 * e * kSwLd] = d[e];
            PT[4 * e] = d[e];
        }
        if (B.ldiag && l < 16 && 16 * k + l < m)
            B.ldiag[B.scale * (int64_t)B.off[p] + 16 * k + l] = sqrt(mypiv);
        if (!ok && l == 0) fail = 1;  // checked at the end: a way out of the loop costs 40
    };                                // copies of accumulators a step
    publish(0);
    publish(-1);
    __syncthreads();
    if (w == 0) invert(0);
    for (int k = 0; k < nb; ++k) {
        double *C = sw_lds + (k & 1) * buf;
        __syncthreads();
        asm volatile("" : "+v"(o_row), "+v"(o_col));
        // W_r = C_r P (stored negated), block row r by wavefront r % WAVES; block k of
        // both: -I
        for (int r = w; r < nb; r += WAVES) {
            double *W = sw_lds + oW + 16 * r * kSwLd + o_col;
            if (r == k) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double v = 4 * e + lr == lc ? -1.0 : 0.0;
                    W[4 * e * kSwLd] = v;
                    C[(16 * r + 4 * e) * kSwLd + o_col] = v;
                }
                continue;
            }
            const double *P = sw_lds + oP + 16 * (k & 1) * kSwLd + o_col;
            mfma_acc x = {};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                x = mfma_f64_16x16x4(C[16 * r * kSwLd + 4 * kk + o_row], P[4 * kk * kSwLd], x);
#pragma unroll
            for (int e = 0; e < 4; ++e) W[4 * e * kSwLd] = -x[e];
        }
        __syncthreads();
        // A_k+1,k+1 and its inverse; the tiles: A_ij -= W_i C_j^T.  Those of row and
        // column k start from 0 and have -I as one factor (exact): A_ik <- W_i I,
        // A_kj <- I W_j^T, A_kk <- -I P, so that a run of slots has no branch (a branch
        // per tile cost 1,200 cycles a tile, against 256 of its products)
        if (w == 0 && k + 1 < nb) invert(k + 1);
        const uint64_t zero = __ballot(li == k || lj == k);
        const int offA = sweep_operand_a(S, nb, li), offB = sweep_operand_b(S, nb, li, lj, k);
#pragma unroll
        for (int s0 = 0; s0 < kSwSlots; s0 += kRun) {
            if (s0 >= nt) continue;
#pragma unroll
            for (int q = 0; q < kRun; ++q) {
                const int s = s0 + q;
                if (s >= kSwSlots) continue;
                const bool z = zero >> s & 1;
                const double *qa = sw_lds + __builtin_amdgcn_readlane(offA, s) + o_row;
                const double *qb = sw_lds + __builtin_amdgcn_readlane(offB, s) + o_row;
                mfma_acc x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = z ? 0.0 : acc[s][e];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) x = mfma_f64_16x16x4(qa[4 * kk], qb[4 * kk], x);
                acc[s] = x;
            }
        }
        publish(k + 1);
    }
    if (fail) {
        if (tid == 0) {
            if (B.fail)
                B.fail[p] = 1;
            else
                atomicMax(&B.status[0], p + 1);
        }
        return;
    }
    // A^-1 = -(the tiles), both triangles; the upper one through LDS, so that both are
    // written in rows of 128 bytes
    __syncthreads();
    double *tr = sw_lds + 16 * w * kSwLd;
#pragma unroll
    for (int s = 0; s < kSwSlots; ++s) {
        if (s >= nt) continue;
        const int i = 16 * (tij[s] & 255), j = 16 * (tij[s] >> 8);
        const bool whole = i + 16 <= m;
        double *lo = Out + ((size_t)i * m + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double v = -acc[s][e];
            if (whole || (i + 4 * e + lr < m && j + lc < m)) lo[o_tile + 4 * e * m] = v;
            tr[4 * e * kSwLd + o_col] = v;
        }
        if (i == j) continue;
        asm volatile("" ::: "memory");
        double *up = Out + ((size_t)j * m + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double v = tr[4 * e + o_row];
            if (whole || i + lc < m) up[o_tile + 4 * e * m] = v;
        }
        asm volatile("" ::: "memory");
    }
}

bool precond_factor_in_place(int max_m) { return max_m > kSwRows; }

template <int NBMAX, int WAVES>
static hipError_t launch_sweep_as(hipStream_t s, const MatBatch &B, int count, int max_m) {
    const size_t lds = sweep_lds_bytes(max_m);
    const hipError_t e = hipFuncSetAttribute((const void *)pc_sweep_kernel<NBMAX, WAVES>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    pc_sweep_kernel<NBMAX, WAVES><<<count, 64 * WAVES, lds, s>>>(B);
    return hipSuccess;
}

// the sweep over a batch of count matrices of at most max_m <= kSwRows rows, n_large of
// them (the first of B.order) beyond the small instance: the small instance when every
// matrix fits it, else the large one for all of them in one launch (small matrices then
// run beside the large ones), else, when both kinds fill the chip, one launch of each:
// two small ones share a compute unit (512 bacteria: 416 us in one
// launch, 399 in two)
static hipError_t launch_sweep(hipStream_t s, MatBatch B, int count, int max_m, int n_large) {
    constexpr int kUnits = 256;  // compute units, one large matrix each
    if (max_m <= 16 * kSwSmall) return launch_sweep_as<kSwSmall, 8>(s, B, count, max_m);
    if (!B.order || n_large < kUnits || count - n_large < kUnits)
        return launch_sweep_as<kSwRows / 16, 8>(s, B, count, max_m);
    const hipError_t e = launch_sweep_as<kSwRows / 16, 8>(s, B, n_large, max_m);
    if (e != hipSuccess) return e;
    B.order += n_large;
    return launch_sweep_as<kSwSmall, 8>(s, B, count - n_large, 16 * kSwSmall);
}

hipError_t precond_factor(hipStream_t s, const PrecondDev &P, const double *dvec, int max_m) {
    if (P.M <= 0) return hipSuccess;
    if (max_m <= kSwRows) {
        const MatBatch B{P.blob_off, 3, P.mat_off, P.mats, P.ldiag, P.dinv, P.minv, P.status,
                         nullptr, 0.0, P.order};
        const hipError_t e = launch_sweep(s, B, P.M, max_m, P.n_large);
        if (e != hipSuccess) return e;
    } else if (max_m <= kFastMaxM) {
        const int nbk = (max_m + kNB - 1) / kNB;
        const size_t lds_i = (size_t)nbk * kNB * kLd * sizeof(double);
        const hipError_t e = hipFuncSetAttribute(
            (const void *)pc_trtri_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_i);
        if (e != hipSuccess) return e;
        const int nt = (max_m + 63) / 64;
        const MatBatch B{P.blob_off, 3, P.mat_off, P.mats, P.ldiag, P.dinv, P.minv, P.status,
                         nullptr, 0.0, nullptr};
        pc_potrf_kernel<<<P.M, 256, 0, s>>>(B);
        pc_trtri_kernel<<<dim3(nbk, P.M), 256, lds_i, s>>>(B);
        pc_lauum_kernel<<<dim3(nt * (nt + 1) / 2, P.M), 256, 0, s>>>(B);
    } else {
        pc_chol_kernel<<<P.M, 256, 0, s>>>(P.blob_off, P.mat_off, P.mats, P.ldiag, P.status);
        pc_inverse_kernel<<<P.M, 256, 0, s>>>(P.blob_off, P.mat_off, P.mats, P.ldiag, P.minv,
                                              P.status);
        pc_restore_diag_kernel<<<P.M, 256, 0, s>>>(P.blob_off, P.mat_off, P.mats, P.ldiag);
    }
    pc_body_kernel<<<P.M, 256, 0, s>>>(P.order, P.blob_off, P.mat_off, P.z_off, P.minv, dvec, P.Z,
                                       P.Nt, P.body_pinv, P.status);
    pc_body_pinv_kernel<<<(P.M + 63) / 64, 64, 0, s>>>(P.M, P.body_pinv, P.Nt, P.status);
    return hipGetLastError();
}

// doubles needed for the diagonal-block inverses of bodies holding n_blobs blobs
int64_t precond_dinv_size(int64_t n_blobs, int M) { return 32 * 3 * n_blobs + 1024 * (int64_t)M; }

// Single-blob bodies (Sec. 2.4 with Sec. 3.1): N~_p = diag(mt I, mr I), the
// self mobilities 1/(6 pi eta a) and 1/(8 pi eta a^3)
__global__ void single_blob_nt_kernel(int M, double mt, double mr, double *__restrict__ Nt) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= 36 * M) return;
    const int e = idx % 36, r = e / 6, c = e % 6;
    Nt[idx] = r != c ? 0.0 : (r < 3 ? mt : mr);
}

__global__ void copy_kernel(int64_t n, const double *__restrict__ x, double *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = x[i];
}

void single_blob_body_mobility(hipStream_t s, int M, double a, double eta, double *Nt) {
    if (M <= 0) return;
    single_blob_nt_kernel<<<(36 * M + 255) / 256, 256, 0, s>>>(
        M, 1.0 / (6.0 * kPi * eta * a), 1.0 / (8.0 * kPi * eta * a * a * a), Nt);
}

// z = P^-1 r for y = [U; phi]: phi = G~ (r_phi - C r_U), U = r_U + N~ C^T phi.
// These are the assembly and body stages of the multiblob apply with no blobs
// (r_U takes the place of U^); zero_off / zero_off64 are M+1 zeros.
void precond_apply_single(hipStream_t s, const PrecondDev &P, const int *zero_off,
                          const int64_t *zero_off64, const double *r, double *z) {
    if (P.M <= 0) return;
    const int64_t m6 = 6 * (int64_t)P.M;
    copy_kernel<<<(int)((m6 + 255) / 256), 256, 0, s>>>(m6, r, P.tmp);
    if (P.A > 0)
        pc_apply2_kernel<<<P.A, 256, 0, s>>>(0, P.M, P.asm_row_ptr, P.asm_rows, P.asm_mat_off,
                                             P.row_p, P.row_q, P.crow, P.G, r, P.tmp, z);
    pc_apply3_kernel<<<P.M, 256, 0, s>>>(0, P.M, zero_off, zero_off64, P.Nt, P.Nt, P.brow_ptr,
                                         P.brow_ent, P.crow, P.tmp, z, P.A > 0 ? 1 : 0);
}

// G~_a = S_a^-1 for every assembly (Sec. 3.1), with a pivot test relative to the
// largest diagonal entry; assemblies that fail it (constraints without full row
// rank) take the symmetric pseudo-inverse.  Largest assembly of at most kAsmSmall
// rows: one workgroup per assembly in LDS; up to kFastMaxM rows: the blocked
// kernels of the blob mobilities (S_a formed in P.S, factored in place, the
// inverse written to P.G); beyond: the unblocked kernel.
hipError_t precond_assembly(hipStream_t s, const PrecondDev &P) {
    if (P.A <= 0) return hipSuccess;
    const int nmax = std::max(P.asm_max_rows, 1);
    if (nmax <= kAsmSmall && P.asm_fail) {
        const size_t lds = (2 * (size_t)nmax * (nmax + 1) + 24 * (size_t)nmax) * sizeof(double) +
                           2 * (size_t)nmax * sizeof(int);
        const hipError_t e = hipFuncSetAttribute(
            (const void *)pc_asm_small_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        pc_asm_small_kernel<<<P.A, kAsmThreads, lds, s>>>(P.asm_row_ptr, P.asm_rows,
                                                          P.asm_mat_off, P.row_p, P.row_q, P.crow,
                                                          P.Nt, P.G, P.asm_fail, P.status, nmax);
        pc_asm_pinv_kernel<<<P.A, 256, 0, s>>>(P.asm_row_ptr, P.asm_rows, P.asm_mat_off, P.row_p,
                                               P.row_q, P.crow, P.Nt, P.S, P.G, P.asm_fail,
                                               P.status);
        return hipGetLastError();
    }
    if (P.asm_max_rows > kFastMaxM || !P.asm_dinv || !P.asm_fail) {
        pc_asm_kernel<<<P.A, 256, 0, s>>>(P.asm_row_ptr, P.asm_rows, P.asm_mat_off, P.row_p,
                                          P.row_q, P.crow, P.Nt, P.S, P.G, P.status);
        return hipGetLastError();
    }
    const int max_m = nmax;
    const int nbk = (max_m + kNB - 1) / kNB;
    const size_t lds_i = (size_t)nbk * kNB * kLd * sizeof(double);
    const size_t lds_r = 24 * (size_t)max_m * sizeof(double) + 2 * (size_t)max_m * sizeof(int);
    const bool sweep = max_m <= kSwRows;
    hipError_t e = hipFuncSetAttribute((const void *)pc_trtri_kernel,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_i);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void *)pc_asm_form_kernel,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_r);
    if (e != hipSuccess) return e;
    const int nt = (max_m + 63) / 64;
    pc_asm_form_kernel<<<P.A, kAsmForm, lds_r, s>>>(P.asm_row_ptr, P.asm_rows, P.asm_mat_off,
                                               P.row_p, P.row_q, P.crow, P.Nt, P.S, P.asm_fail,
                                               P.status, max_m);
    const MatBatch B{P.asm_row_ptr, 1, P.asm_mat_off, P.S, nullptr, P.asm_dinv, P.G, P.status,
                     P.asm_fail, 1e-12, nullptr};
    if (sweep) {
        e = launch_sweep(s, B, P.A, max_m, 0);
        if (e != hipSuccess) return e;
    } else {
        pc_potrf_kernel<<<P.A, 256, 0, s>>>(B);
        pc_trtri_kernel<<<dim3(nbk, P.A), 256, lds_i, s>>>(B);
        pc_lauum_kernel<<<dim3(nt * (nt + 1) / 2, P.A), 256, 0, s>>>(B);
    }
    pc_asm_pinv_kernel<<<P.A, 256, 0, s>>>(P.asm_row_ptr, P.asm_rows, P.asm_mat_off, P.row_p,
                                           P.row_q, P.crow, P.Nt, P.S, P.G, P.asm_fail, P.status);
    return hipGetLastError();
}

// threads of a body's workgroup in the first of three kernels: all of them while the
// bodies are few, then what gives a mean body's rows about 4 parts, so that more bodies are
// resident (all three kernels, with 1,024, 8, 4 and 2 parts: 8,000 bodies of 6 and 8 of 42
// blobs 72, 37, 37 and 37 us, 2,000 of 42 59, 62, 59 and 56, 1,000 of 42 and one of 300
// 120, 121, 123 and 187)
static int apply1_threads(int N, int M) {
    int T = 256;
    while (T < kApply && (M < kFuseMany || T < 4 * 3 * (N / M))) T *= 2;
    return T;
}

void precond_apply(hipStream_t s, const PrecondDev &P, int N, const double *r, double *z,
                   const double *alpha, double *v) {
    if (P.M <= 0) return;
    if (P.fuse.rows) {
        // a workgroup per compute unit while the assemblies are few, at most 16 each (a
        // workgroup's chain is the same however few rows it has: one body of 300 blobs 18,
        // 14, 13 and 11 us with 8, 16, 32 and 64, one of 8 bodies of 42 15 to 16 with
        // each).  From two per unit on, 256 threads each, so that more are resident (1,000
        // shells of 42 blobs: 26.2 us, with 1,024 threads 38.5)
        const int split = std::min(16, std::max(1, kFuseBlocks / P.A));
        const int T = P.A >= kFuseMany ? 256 : kApply;
        pc_apply_asm_kernel<<<dim3(P.A, split), T, fuse_doubles(P.fuse, T) * sizeof(double), s>>>(
            N, P.M, P, r, alpha, v, z);
        return;
    }
    if (P.learned)
        pc_apply1_learned_kernel<<<P.M, 256, 0, s>>>(N, P.blob_off, P.type, P.tmat_off, P.tz_off,
                                                     P.tminv, P.tZ, P.R9, P.Nt, P.lcorr, r, z,
                                                     P.tmp, P.stmp);
    else
        pc_apply1_kernel<<<P.M, apply1_threads(N, P.M), 0, s>>>(N, P.order, P.blob_off, P.mat_off,
                                                                P.z_off, P.minv, P.Z, P.Nt, r, z,
                                                                P.tmp);
    if (P.A > 0)
        pc_apply2_kernel<<<P.A, 256, 0, s>>>(N, P.M, P.asm_row_ptr, P.asm_rows, P.asm_mat_off,
                                             P.row_p, P.row_q, P.crow, P.G, r, P.tmp, z);
    if (P.learned)
        pc_apply3_learned_kernel<<<P.M, 256, 0, s>>>(N, P.M, P.blob_off, P.type, P.tz_off, P.tZ,
                                                     P.R9, P.Nt, P.lcorr, P.stmp, P.brow_ptr,
                                                     P.brow_ent, P.crow, P.tmp, z,
                                                     P.A > 0 ? 1 : 0);
    else
        pc_apply3_kernel<<<P.M, 256, 0, s>>>(N, P.M, P.blob_off, P.z_off, P.Z, P.Nt, P.brow_ptr,
                                             P.brow_ent, P.crow, P.tmp, z, P.A > 0 ? 1 : 0);
}

}  // namespace arb
