// Device side of the rigid-body rows of the saddle operator (Eq. linear_system): the
// body and constraint rows that a launch of the pair product's last step carries along.
#pragma once
#include "common.h"

namespace arb {

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// body p by one wavefront: out_p = sign (K^T lambda)_p + (C^T phi)_p
__device__ __forceinline__ void kt_ct_row(int p, int lane, const int *__restrict__ blob_off,
                                          const double *__restrict__ dvec,
                                          const double *__restrict__ lam, double sign,
                                          const int *__restrict__ brow_ptr,
                                          const int *__restrict__ brow_ent,
                                          const double *__restrict__ crow,
                                          const double *__restrict__ phi,
                                          double *__restrict__ out) {
    double f[6] = {0, 0, 0, 0, 0, 0};
    if (lam) {
        for (int i = blob_off[p] + lane; i < blob_off[p + 1]; i += kWave) {
            const double l0 = lam[3 * (size_t)i], l1 = lam[3 * (size_t)i + 1],
                         l2 = lam[3 * (size_t)i + 2];
            const double d0 = dvec[3 * (size_t)i], d1 = dvec[3 * (size_t)i + 1],
                         d2 = dvec[3 * (size_t)i + 2];
            f[0] += l0;
            f[1] += l1;
            f[2] += l2;
            f[3] += d1 * l2 - d2 * l1;
            f[4] += d2 * l0 - d0 * l2;
            f[5] += d0 * l1 - d1 * l0;
        }
    }
    for (int k = 0; k < 6; ++k) f[k] = sign * wave_sum(f[k]);
    if (lane == 0) {
        if (phi) {
            for (int e = brow_ptr[p]; e < brow_ptr[p + 1]; ++e) {
                const int ent = brow_ent[e];
                const int row = ent >> 1, side = ent & 1;
                const double *c = crow + 12 * (size_t)row + 6 * side;
                const double ph = phi[row];
                for (int k = 0; k < 6; ++k) f[k] += ph * c[k];
            }
        }
        for (int k = 0; k < 6; ++k) out[6 * (size_t)p + k] = f[k];
    }
}

// constraint row k: (C U)_k
__device__ __forceinline__ double c_row(int k, const int *__restrict__ row_p,
                                        const int *__restrict__ row_q,
                                        const double *__restrict__ crow,
                                        const double *__restrict__ U) {
    const double *c = crow + 12 * (size_t)k;
    const double *Up = U + 6 * (size_t)row_p[k];
    double s = 0.0;
    for (int a = 0; a < 6; ++a) s += c[a] * Up[a];
    const int q = row_q[k];
    if (q >= 0) {
        const double *Uq = U + 6 * (size_t)q;
        for (int a = 0; a < 6; ++a) s += c[6 + a] * Uq[a];
    }
    return s;
}

// Workgroup b of those that follow the blob workgroups: bodies first (a wavefront
// each), then constraint rows (a thread each).  They read lambda, U and phi only, so
// they need no order against the pair sums.  With launches of their own (5.4 and 4.1 us
// for 16 bacteria, 6.5 and 4.7 for 100) the reduction took 4.6 and 4.5 us, with them
// 6.7 and 5.7.
__device__ __forceinline__ void saddle_rows(const SaddleRows &R, int b) {
    const int T = blockDim.x, lane = threadIdx.x & (kWave - 1);
    const int bodies = T / kWave, nb = (R.M + bodies - 1) / bodies;
    if (b < nb) {
        const int p = b * bodies + threadIdx.x / kWave;
        if (p < R.M)
            kt_ct_row(p, lane, R.blob_off, R.dvec, R.lam, -1.0, R.brow_ptr, R.brow_ent, R.crow,
                      R.phi, R.out_u);
        return;
    }
    const int k = (b - nb) * T + threadIdx.x;
    if (k < R.Nc) R.out_phi[k] = c_row(k, R.row_p, R.row_q, R.crow, R.U);
}

inline int saddle_blocks(const SaddleRows &R, int T) {
    const int bodies = T / kWave;
    return (R.M + bodies - 1) / bodies + (R.Nc + T - 1) / T;
}

}  // namespace arb
