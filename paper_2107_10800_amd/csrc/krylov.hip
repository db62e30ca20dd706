// Dense FP64 kernels of the restarted GMRES (Sec. 3.1): Arnoldi with
// classical Gram-Schmidt applied twice, Givens rotations of the Hessenberg
// column, triangular solve and basis combination.  Reductions are two-stage
// with a fixed order, so results do not depend on scheduling.
#include <type_traits>

#include "common.h"

namespace arb {

static inline int nblk(int64_t n, int b) { return (int)((n + b - 1) / b); }
__device__ __forceinline__ double wave_sum64(double v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// out[i] = sum over nb workgroups of partial[i * nb + block], i < k, in block order per
// lane (4 wavefronts, one row each in turn)
__device__ __forceinline__ void reduce_rows(int k, int nb, const double *__restrict__ partial,
                                            double *out) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll 2
    for (int i = w; i < k; i += 4) {
        double s = 0.0;
#pragma unroll 4
        for (int c = lane; c < nb; c += kWave) s += partial[(int64_t)i * nb + c];
        s = wave_sum64(s);
        if (lane == 0) out[i] = s;
    }
}

__global__ __launch_bounds__(256) void reduce_rows_kernel(int nb,
                                                          const double *__restrict__ partial,
                                                          double *__restrict__ h) {
    const int i = blockIdx.x;
    reduce_rows(1, nb, partial + (int64_t)i * nb, h + i);
}

// Classical Gram-Schmidt of w against V_0..V_{k-1}, one launch per pass.  A workgroup
// keeps 256 E elements of w:
//   SUB = false: partial sums of V^T w;
//   SUB = true, NORM = false: w -= V h, then partial sums of V^T w (the second pass's
//     products while this part of V is still in the caches);
//   SUB = true, NORM = true: w -= V h, then partial sums of ||w||^2.
// h are the sums over the last pass's workgroups (pin, nb of them): every workgroup adds
// them up for itself, in the same order, which costs less than a launch or a
// device-wide fence (the last workgroup to finish adding them up: 16 us a pass on
// 38,400 unknowns, most of it the fences' cache write-back), and workgroup 0 stores them
// to hout; pin = NULL: h are in hout already.  Latency-bound at a few thousand
// unknowns, where products, reductions, updates and scalars took nine launches and
// about 30 us an Arnoldi step; HBM-bound (two readings of V) above.
template <int E, bool SUB, bool NORM>
__global__ __launch_bounds__(256) void cgs_kernel(int64_t n, int k, const double *__restrict__ V,
                                                  int64_t ldv, const double *__restrict__ pin,
                                                  double *__restrict__ hout,
                                                  double *__restrict__ w,
                                                  double *__restrict__ partial) {
    __shared__ double ws[256 * E];
    __shared__ double sh[kMaxRestart + 4];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave, nb = gridDim.x;
    const int64_t base = (int64_t)blockIdx.x * (256 * E);
    if (SUB) {
        if (pin) {
            reduce_rows(k, nb, pin, sh);
        } else {
            for (int i = tid; i < k; i += 256) sh[i] = hout[i];
        }
        __syncthreads();
        if (pin && blockIdx.x == 0)
            for (int i = tid; i < k; i += 256) hout[i] = sh[i];
    }
    double nrm = 0.0;
#pragma unroll
    for (int q = 0; q < E; ++q) {
        const int64_t t = base + q * 256 + tid;
        double v = 0.0;
        if (t < n) {
            v = w[t];
            if (SUB) {
                double s = 0.0;
#pragma unroll 8
                for (int i = 0; i < k; ++i) s += V[(int64_t)i * ldv + t] * sh[i];
                v -= s;
                w[t] = v;
            }
        }
        ws[q * 256 + tid] = v;
        nrm += v * v;
    }
    if (NORM) {
        nrm = wave_sum64(nrm);
        __syncthreads();  // sh read as h above
        if (lane == 0) sh[wv] = nrm;
        __syncthreads();
        if (tid == 0) partial[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
        return;
    }
    __syncthreads();
    // a wavefront per product: the workgroup's elements of V_i against w in LDS
#pragma unroll 4
    for (int i = wv; i < k; i += 4) {
        const double *v = V + (int64_t)i * ldv + base;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < 4 * E; ++q) {
            const int o = q * kWave + lane;
            if (base + o < n) s += v[o] * ws[o];
        }
        s = wave_sum64(s);
        if (lane == 0) partial[(int64_t)i * nb + blockIdx.x] = s;
    }
}

struct PostArgs {
    int j, m;
    const double *h1, *h2;
    double *Hbar, *cs, *sn, *g, *out, *host;
};

__device__ void arnoldi_post_dev(const PostArgs &p, double hn2, double *sh);

// the step's end: ||w||^2 from its partial sums and the Givens update; one workgroup
__global__ __launch_bounds__(256) void arnoldi_finish_kernel(int nb,
                                                             const double *__restrict__ partial,
                                                             PostArgs post) {
    __shared__ double sh[4 * (kMaxRestart + 4)];
    reduce_rows(1, nb, partial, sh);
    __syncthreads();
    const double hn2 = sh[0];
    __syncthreads();
    arnoldi_post_dev(post, hn2, sh);
}

// partial sums of ||x||^2
template <int E>
__global__ __launch_bounds__(256) void norm_kernel(int64_t n, const double *__restrict__ x,
                                                   double *__restrict__ partial) {
    __shared__ double sh[4];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < E; ++q) {
        const int64_t t = (int64_t)blockIdx.x * (256 * E) + q * 256 + tid;
        if (t < n) s += x[t] * x[t];
    }
    s = wave_sum64(s);
    if (lane == 0) sh[wv] = s;
    __syncthreads();
    if (tid == 0) partial[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// out[0] = the sum of x[0..n) (partial sums) or with SQUARE of their squares; with g: g =
// [sqrt, 0, ...] (m + 1 entries) and out[1] = sqrt; host[0] = out[0], or out[1] with g
template <bool SQUARE>
__global__ __launch_bounds__(1024) void norm_finish_kernel(int64_t n, const double *__restrict__ x,
                                                           int m, double *__restrict__ g,
                                                           double *__restrict__ out,
                                                           double *host) {
    __shared__ double sh[16];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    double s = 0.0;
#pragma unroll 4
    for (int64_t t = tid; t < n; t += 1024) s += SQUARE ? x[t] * x[t] : x[t];
    s = wave_sum64(s);
    if (lane == 0) sh[wv] = s;
    __syncthreads();
    double b2 = 0.0;
    for (int q = 0; q < 16; ++q) b2 += sh[q];
    const double b = sqrt(b2);
    if (g)
        for (int i = tid; i <= m; i += 1024) g[i] = i == 0 ? b : 0.0;
    if (tid == 0) {
        out[0] = b2;
        if (g) out[1] = b;
        host[0] = g ? b : b2;
        __threadfence_system();
    }
}

__global__ __launch_bounds__(256) void gemv_set_kernel(int64_t n, int k,
                                                       const double *__restrict__ V, int64_t ldv,
                                                       const double *__restrict__ h,
                                                       double *__restrict__ out) {
    __shared__ double hs[260];
    for (int i = threadIdx.x; i < k; i += 256) hs[i] = h[i];
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    double s = 0.0;
    for (int i = 0; i < k; ++i) s += V[(int64_t)i * ldv + t] * hs[i];
    out[t] = s;
}

__global__ void scale_copy_kernel(int64_t n, const double *__restrict__ x,
                                  const double *__restrict__ alpha, double *__restrict__ y) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < n) y[t] = x[t] / alpha[0];
}

__global__ void axpby_kernel(int64_t n, double a, const double *__restrict__ x, double b,
                             double *__restrict__ y) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < n) y[t] = a * x[t] + b * y[t];
}

// h1[0..j] = first CGS pass h, h2[0..j] = second pass, hn2 = ||w||^2.  Applies the
// previous rotations, builds rotation j, updates g, stores the rotated column in Hbar
// (column-major, ld = m+1), writes hn = ||w|| and the residual estimate |g[j+1]| to
// out[0], out[1] and to host memory (host[0], host[1]).  A whole workgroup, sh: 4
// (kMaxRestart + 4) doubles of LDS: the serial recursion runs on LDS copies.
__device__ void arnoldi_post_dev(const PostArgs &p, double hn2, double *sh) {
    double *col = sh, *cs = col + kMaxRestart + 4, *sn = cs + kMaxRestart + 4;
    const int j = p.j, tid = threadIdx.x;
    for (int i = tid; i <= j; i += blockDim.x) {
        col[i] = p.h1[i] + p.h2[i];
        if (i < j) {
            cs[i] = p.cs[i];
            sn[i] = p.sn[i];
        }
    }
    __syncthreads();
    if (tid == 0) {
        const double hn = sqrt(hn2);
        col[j + 1] = hn;
        for (int i = 0; i < j; ++i) {
            const double t = cs[i] * col[i] + sn[i] * col[i + 1];
            col[i + 1] = -sn[i] * col[i] + cs[i] * col[i + 1];
            col[i] = t;
        }
        const double rho = hypot(col[j], col[j + 1]);
        const double c = col[j] / rho, s = col[j + 1] / rho;
        p.cs[j] = c;
        p.sn[j] = s;
        col[j] = rho;
        col[j + 1] = 0.0;
        const double gj = p.g[j], g1 = -s * gj;
        p.g[j + 1] = g1;
        p.g[j] = c * gj;
        p.out[0] = hn;
        p.out[1] = fabs(g1);
        p.host[0] = hn;
        p.host[1] = fabs(g1);
        __threadfence_system();
    }
    __syncthreads();
    double *H = p.Hbar + (int64_t)j * (p.m + 1);
    for (int i = tid; i <= j + 1; i += blockDim.x) H[i] = col[i];
}

// The whole orthogonalisation of one Arnoldi step for a system of at most
// kSmallArnoldi unknowns in one workgroup: w against V_0..V_j by classical
// Gram-Schmidt twice (w held in LDS), ||w||, then the Givens update of
// arnoldi_post.  One launch instead of four; the same steps with a different
// summation order (one wave per dot product, lanes strided over the rows).
__global__ __launch_bounds__(1024) void arnoldi_small_kernel(
    int n, const double *__restrict__ V, int64_t ldv, double *__restrict__ w, PostArgs post) {
    __shared__ double ws[kSmallArnoldi];
    __shared__ double hs[2][kMaxRestart + 1];
    __shared__ double sh[4 * (kMaxRestart + 4)];
    const int j = post.j;
    __shared__ double red[1024 / kWave];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    constexpr int nwave = 1024 / kWave;
    for (int t = tid; t < n; t += 1024) ws[t] = w[t];
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
        double *h = hs[pass];
        for (int i = wave; i <= j; i += nwave) {
            const double *v = V + (int64_t)i * ldv;
            double sacc = 0.0;
            for (int t = lane; t < n; t += kWave) sacc += v[t] * ws[t];
            for (int off = kWave / 2; off > 0; off >>= 1) sacc += __shfl_xor(sacc, off);
            if (lane == 0) h[i] = sacc;
        }
        __syncthreads();
        for (int t = tid; t < n; t += 1024) {
            double acc = 0.0;
            for (int i = 0; i <= j; ++i) acc += V[(int64_t)i * ldv + t] * h[i];
            ws[t] -= acc;
        }
        __syncthreads();
    }
    double sq = 0.0;
    for (int t = tid; t < n; t += 1024) {
        sq += ws[t] * ws[t];
        w[t] = ws[t];
    }
    for (int off = kWave / 2; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if (lane == 0) red[wave] = sq;
    __syncthreads();
    double hn2 = 0.0;
    for (int k = 0; k < nwave; ++k) hn2 += red[k];
    post.h1 = hs[0];
    post.h2 = hs[1];
    arnoldi_post_dev(post, hn2, sh);
}

// back substitution of the rotated (upper-triangular) Hessenberg, k <= kMaxRestart = 256:
// s = H^-1 g by columns, a thread per row, the next column loaded before this one's
// barrier (one thread for the whole chain of loads: 17.5 us at k = 18, 24.8 at 23)
__global__ __launch_bounds__(kMaxRestart) void upper_solve_kernel(
    int k, int m, const double *__restrict__ Hbar, const double *__restrict__ g,
    double *__restrict__ sv) {
    __shared__ double y;
    const int i = threadIdx.x;
    const bool row = i < k;
    double s = row ? g[i] : 0.0;
    const double d = row ? Hbar[(int64_t)i * (m + 1) + i] : 1.0;
    double next = row ? Hbar[(int64_t)(k - 1) * (m + 1) + i] : 0.0;
    for (int c = k - 1; c >= 0; --c) {
        const double h = next;
        if (c > 0 && row) next = Hbar[(int64_t)(c - 1) * (m + 1) + i];
        if (i == c) sv[c] = y = s / d;
        __syncthreads();
        if (i < c) s -= h * y;
        __syncthreads();
    }
}

// b = [u_s; -F; B]
__global__ void rhs_kernel(int N, int M, int Nc, const double *__restrict__ us,
                           const double *__restrict__ F, const double *__restrict__ B,
                           double *__restrict__ b) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t n3 = 3 * (int64_t)N, m6 = 6 * (int64_t)M;
    if (t < n3)
        b[t] = us ? us[t] : 0.0;
    else if (t < n3 + m6)
        b[t] = -F[t - n3];
    else if (t < n3 + m6 + Nc)
        b[t] = B[t - n3 - m6];
}

// elements of a vector per thread: 1 up to 65,536 unknowns (256 workgroups), 8 at most
static int cgs_elems(int64_t n) {
    int e = 1;
    while (e < 8 && n > (int64_t)e * 256 * 512) e *= 2;
    return n <= 65536 ? 1 : e;
}
int cgs_blocks(int64_t n) { return nblk(n, 256 * cgs_elems(n)); }

template <class F> static void with_elems(int64_t n, F &&f) {
    switch (cgs_elems(n)) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
    }
}

// up to this many unknowns one workgroup forms a norm
constexpr int64_t kNormOne = 16384;

void vector_norm(hipStream_t s, int64_t n, const double *x, double *partial, int m, double *g,
                 double *out, double *host) {
    if (n <= kNormOne) {
        norm_finish_kernel<true><<<1, 1024, 0, s>>>(n, x, m, g, out, host);
        return;
    }
    with_elems(n, [&](auto e) {
        norm_kernel<decltype(e)::value><<<cgs_blocks(n), 256, 0, s>>>(n, x, partial);
    });
    norm_finish_kernel<false><<<1, 1024, 0, s>>>(cgs_blocks(n), partial, m, g, out, host);
}

// up to this many workgroups every workgroup of the next pass adds the partial sums up
// for itself; more (from 65,537 unknowns) have a launch for it, so that the readings of
// the partial sums, a square of the workgroups, stay small against those of V
constexpr int kOwnSums = 256;

void arnoldi_step(hipStream_t s, int64_t n, int j, int m, const double *V, double *w,
                  double *partial, double *h1, double *h2, double *Hbar, double *cs, double *sn,
                  double *g, double *out, double *host) {
    const PostArgs post{j, m, h1, h2, Hbar, cs, sn, g, out, host};
    if (n <= kSmallArnoldi) {
        arnoldi_small_kernel<<<1, 1024, 0, s>>>((int)n, V, n, w, post);
        return;
    }
    const int nb = cgs_blocks(n), k = j + 1;
    double *pa = partial, *pb = partial + (size_t)(m + 1) * nb;
    const bool own = nb <= kOwnSums;
    with_elems(n, [&](auto e) {
        constexpr int E = decltype(e)::value;
        cgs_kernel<E, false, false><<<nb, 256, 0, s>>>(n, k, V, n, nullptr, nullptr, w, pa);
        if (!own) reduce_rows_kernel<<<k, 256, 0, s>>>(nb, pa, h1);
        cgs_kernel<E, true, false><<<nb, 256, 0, s>>>(n, k, V, n, own ? pa : nullptr, h1, w, pb);
        if (!own) reduce_rows_kernel<<<k, 256, 0, s>>>(nb, pb, h2);
        cgs_kernel<E, true, true><<<nb, 256, 0, s>>>(n, k, V, n, own ? pb : nullptr, h2, w, pa);
    });
    arnoldi_finish_kernel<<<1, 256, 0, s>>>(nb, pa, post);
}
void gemv_set(hipStream_t s, int64_t n, int k, const double *V, int64_t ldv, const double *h,
              double *out) {
    gemv_set_kernel<<<nblk(n, 256), 256, 0, s>>>(n, k, V, ldv, h, out);
}
void scale_copy(hipStream_t s, int64_t n, const double *x, const double *alpha, double *y) {
    scale_copy_kernel<<<nblk(n, 256), 256, 0, s>>>(n, x, alpha, y);
}
void axpby(hipStream_t s, int64_t n, double a, const double *x, double b, double *y) {
    axpby_kernel<<<nblk(n, 256), 256, 0, s>>>(n, a, x, b, y);
}
void upper_solve(hipStream_t s, int k, int m, const double *Hbar, const double *g, double *sv) {
    upper_solve_kernel<<<1, (k + 63) / 64 * 64, 0, s>>>(k, m, Hbar, g, sv);
}
void rhs_assemble(hipStream_t s, int N, int M, int Nc, const double *us, const double *F,
                  const double *B, double *b) {
    const int64_t n = 3 * (int64_t)N + 6 * (int64_t)M + Nc;
    rhs_kernel<<<nblk(n, 256), 256, 0, s>>>(N, M, Nc, us, F, B, b);
}

}  // namespace arb
