// Fast blob mobility product u = M lambda for large systems (Sec. 2.3; the
// paper names fast summation, Sec. 1 and Sec. 6, as the route past dense sums).
//
// A kernel-independent multipole method (the black-box FMM of Fong and Darve,
// J. Comput. Phys. 228, 2009): the RPY tensor of two well-separated cells is
// replaced by its tensor-product Chebyshev interpolant in both arguments,
//   M(x, y) ~ sum_k sum_m S_k(x) M(t_k, s_m) S_m(y),
// with t, s the n^3 proxy points of the target and source cells.  The pair
// function is the one of the direct sums (unbounded, or with the wall image):
// above the wall nothing else changes, since the image y* of a source is never
// closer to a target than y itself, so a well-separated pair stays
// well-separated for the image term too.
//
// Tree (built on the host once per geometry, in units of length):
//   root cube: origin o = componentwise minimum of the positions, side
//   S = largest extent * (1 + 2^-20) (S = a when all blobs coincide); a blob
//   lies at level l in the cell floor(((x - o) / S) 2^l); cells of one level are
//   adjacent when their coordinates differ by at most 1 per direction.  Leaf
//   level L: fixed by the options, or the shallowest level whose mean
//   occupancy is at most the requested blobs per leaf, or by default the level
//   with the fewest pair evaluations per product (direct pairs plus M2L pairs,
//   counted level by level from level 2 while they fall); never deeper than
//   the deepest level with a cell side >= 2a (so every
//   interpolated pair has r > 2a and stays off the overlap branch of the
//   tensor).  Interaction list of a cell at level l >= 2: the non-empty cells
//   whose parent is adjacent to its parent and which are not adjacent to it.
// Per product (all on the GPU, sorted by Morton key):
//   P2M  qhat^c_m = sum_{j in c} S^c_m(y_j) lam_j at the leaves;
//   M2M  the parent's qhat from its children's proxies (exact: the parent's
//        Lagrange polynomials have degree n-1 and the children interpolate
//        them exactly);
//   M2L  v^c_k = sum_{c' in IL(c)} sum_m M(t^c_k, s^c'_m) qhat^c'_m with FP32 tensor
//        values (fmm_m2l.hip): batches of equal (level, offset, height) on the
//        matrix cores; a listed cell with fewer blobs than proxies enters with
//        its blobs, n^3 |c'| pairs instead of n^6;
//   L2L  the children's v gain the parent's interpolant at their proxies;
//   near + L2P  direct sums over the adjacent leaves (fmm_near.hip: hi/lo split
//        positions, float runs promoted to double, each pair once for both
//        directions) plus sum_k S^leaf_k(x_i) v^leaf_k, written in the original
//        blob order.
// With L <= 1 there is no interaction list: one cell, the direct sum.
// Single-blob bodies (Sec. 2.4): the generalised tensor, with the forces and
// the torques / a in two channels through P2M, M2M and L2L; M2L and the near
// field apply the 6 x 6 tensor between them.
// Two arithmetic variants share the tree and the float-rounded kernel values
// and weights: A = float (lambda, qhat and the runs of sums in float) and
// A = double (lambda, qhat and every sum in double).  The second is linear in
// lambda to double rounding, so Krylov iterations on it converge to any
// tolerance; the float variant serves the inner iterations of FP64 iterative
// refinement.
#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <functional>
#include <mutex>
#include <numeric>
#include <memory>
#include <cmath>
#include <cstdlib>
#include <exception>
#include <system_error>
#include <thread>
#include <type_traits>
#include <utility>

#include "fmm_device.h"

namespace arb {

namespace {

constexpr int kNearBlock = 64;

// Lagrange polynomial l_k(u) at the Chebyshev points (product form)
__device__ __forceinline__ float lag(const float *tab, int n, int k, float u) {
    float p = tab[kTabDen + k];
    for (int j = 0; j < n; ++j)
        if (j != k) p *= u - tab[kTabNode + j];
    return p;
}

__global__ void fmm_sort_pos_kernel(int N, const int *__restrict__ perm,
                                    const float4 *__restrict__ hi, const float4 *__restrict__ lo,
                                    float4 *__restrict__ shi, float4 *__restrict__ slo) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    const int i = perm[k];
    shi[k] = hi[i];
    slo[k] = lo[i];
}

template <class A>
__global__ void fmm_gather_lam_kernel(int N, const int *__restrict__ perm,
                                      const double *__restrict__ lam, Vec4<A> *__restrict__ slam) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    const int i = perm[k];
    slam[k] = vec4<A>((A)lam[3 * i], (A)lam[3 * i + 1], (A)lam[3 * i + 2]);
}

// qhat of the leaves (NO points per direction), one workgroup per leaf: the leaf's blobs
// are staged in LDS in chunks with their 1D Lagrange values, computed once per blob and
// direction.  A lane takes a column of proxies (kx, ky) and every G-th blob: two reads of
// 1D values and three broadcasts serve NO proxies.  (A lane per proxy read LDS four times
// per proxy and blob, which bound it: 1M blobs 176 us, now 86; 256 diatom colonies in FP64
// 127, now 61.)  The groups' sums meet in LDS in FP64, in group order.
constexpr int kP2MChunk = 64;

template <int NO>
struct P2MShape {
    static constexpr int Q = NO * NO, P = Q * NO;
    static constexpr int G = 256 / Q < 8 ? 256 / Q : 8;      // groups of blobs
    static constexpr int T = (G * Q + kWave - 1) / kWave * kWave;
};

template <class A, int NO>
__global__ __launch_bounds__(P2MShape<NO>::T) void fmm_p2m_kernel(
    Geo g, const float *__restrict__ tabg, const int4 *__restrict__ cc,
    const int2 *__restrict__ rng, int cell0, const float4 *__restrict__ shi,
    const float4 *__restrict__ slo, const Vec4<A> *__restrict__ slam, Vec4<A> *__restrict__ qhat) {
    constexpr int n = NO, Q = P2MShape<NO>::Q, P = P2MShape<NO>::P, G = P2MShape<NO>::G,
                  T = P2MShape<NO>::T;
    __shared__ float tab[kTabSize];
    __shared__ float s_l[3][kP2MChunk][kFmmMaxOrder];
    __shared__ Vec4<A> s_lam[kP2MChunk];
    __shared__ double sum[P][3];
    load_tab(tabg, tab);
    const int c = cell0 + blockIdx.x;
    const int tid = threadIdx.x, grp = tid / Q;
    const int kx = tid % Q / n, ky = tid % n;
    const int4 ci = cc[c];
    const int2 r = rng[c];
    const double side = ldexp(g.S, -ci.w);
    const F2 cd[3] = {split(centre(g.ox, side, ci.x)), split(centre(g.oy, side, ci.y)),
                      split(centre(g.oz, side, ci.z))};
    const float iw = (float)(2.0 / side);
    double q[n][3] = {};
    for (int j0 = r.x; j0 < r.y; j0 += kP2MChunk) {
        const int cnt = min(kP2MChunk, r.y - j0);
        __syncthreads();
        for (int t = tid; t < 3 * cnt; t += T) {
            const int jj = t / 3, d = t - 3 * jj;
            const float4 h = shi[j0 + jj], l = slo[j0 + jj];
            const float hx = d == 0 ? h.x : (d == 1 ? h.y : h.z);
            const float lx = d == 0 ? l.x : (d == 1 ? l.y : l.z);
            const float u = ((hx - cd[d].h) + (lx - cd[d].l)) * iw;
#pragma unroll
            for (int kk = 0; kk < n; ++kk) s_l[d][jj][kk] = lag(tab, n, kk, u);
            if (d == 0) s_lam[jj] = slam[j0 + jj];
        }
        __syncthreads();
        if (grp >= G) continue;
        A f[n][3] = {};
        for (int jj = grp; jj < cnt; jj += G) {
            const float wxy = s_l[0][jj][kx] * s_l[1][jj][ky];
            const Vec4<A> L = s_lam[jj];
#pragma unroll
            for (int kz = 0; kz < n; ++kz) {
                const A w = (A)(wxy * s_l[2][jj][kz]);
                f[kz][0] = fma(w, L.x, f[kz][0]);
                f[kz][1] = fma(w, L.y, f[kz][1]);
                f[kz][2] = fma(w, L.z, f[kz][2]);
            }
        }
#pragma unroll
        for (int kz = 0; kz < n; ++kz)
#pragma unroll
            for (int d = 0; d < 3; ++d) q[kz][d] += f[kz][d];
    }
    for (int s = 0; s < G; ++s) {
        if (s == grp)
#pragma unroll
            for (int kz = 0; kz < n; ++kz)
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    double &at = sum[tid % Q * n + kz][d];
                    at = s == 0 ? q[kz][d] : at + q[kz][d];
                }
        __syncthreads();
    }
    for (int k = tid; k < P; k += T)
        qhat[(size_t)c * P + k] = vec4<A>((A)sum[k][0], (A)sum[k][1], (A)sum[k][2]);
}

// qhat of the cells of one level from their children (NO points per direction).  A lane
// takes a column of the parent's proxies (kx, ky) and one child: a child's weight is read
// from LDS once for NO proxies (a lane per proxy read it for each: 1M blobs 40 us a level
// on average, now 27; 256 diatom colonies in FP64 68, now 38).  The children's sums are added
// in their order.
template <class A, int NO>
struct M2MShape {
    static constexpr int Q = NO * NO, P = Q * NO;
    static constexpr size_t bytes(int c) { return P * (sizeof(Vec4<A>) * c + 24); }
    static constexpr int C = bytes(8) <= 60 << 10 ? 8 : bytes(4) <= 60 << 10 ? 4 : 2;  // children at a time
    static constexpr int T = (C * Q + kWave - 1) / kWave * kWave;
};

template <class A, int NO>
__global__ __launch_bounds__((M2MShape<A, NO>::T)) void fmm_m2m_kernel(
    Geo g, const float *__restrict__ tabg, const int4 *__restrict__ cc,
    const int2 *__restrict__ kids, int cell0, Vec4<A> *__restrict__ qhat) {
    constexpr int n = NO, Q = M2MShape<A, NO>::Q, P = M2MShape<A, NO>::P, C = M2MShape<A, NO>::C,
                  T = M2MShape<A, NO>::T;
    __shared__ float tab[kTabSize];
    __shared__ Vec4<A> sq[C * P];
    __shared__ double sum[P][3];
    load_tab(tabg, tab);
    const int c = cell0 + blockIdx.x;
    const int tid = threadIdx.x, mine = tid / Q;
    const int kx = tid % Q / n, ky = tid % n;
    const int2 kr = kids[c];
    if (kr.y <= kr.x)
        for (int k = tid; k < P; k += T) sum[k][0] = sum[k][1] = sum[k][2] = 0.0;
    for (int ch0 = kr.x; ch0 < kr.y; ch0 += C) {
        const int cnt = min(C, kr.y - ch0);
        __syncthreads();
        for (int i = tid; i < cnt * P; i += T) sq[i] = qhat[(size_t)ch0 * P + i];
        __syncthreads();
        A f[n][3] = {};
        if (mine < cnt) {
            const int4 cci = cc[ch0 + mine];
            // t1[sigma][k][m] = l_k(sigma/2 + xi_m/2): the parent's polynomial at the
            // child's proxies (sigma = -1 for the lower child, the even coordinate)
            constexpr int kT = kFmmMaxOrder * kFmmMaxOrder;
            const float *tx = tab + kTabT1 + (cci.x & 1) * kT + kx * kFmmMaxOrder;
            const float *ty = tab + kTabT1 + (cci.y & 1) * kT + ky * kFmmMaxOrder;
            const float *tz = tab + kTabT1 + (cci.z & 1) * kT;
            float z[n][n];
#pragma unroll
            for (int kz = 0; kz < n; ++kz)
#pragma unroll
                for (int mz = 0; mz < n; ++mz) z[kz][mz] = tz[kz * kFmmMaxOrder + mz];
            const Vec4<A> *qc = sq + mine * P;
            for (int mx = 0; mx < n; ++mx)
                for (int my = 0; my < n; ++my) {
                    const float a = tx[mx] * ty[my];
#pragma unroll
                    for (int mz = 0; mz < n; ++mz) {
                        const Vec4<A> q = qc[(mx * n + my) * n + mz];
#pragma unroll
                        for (int kz = 0; kz < n; ++kz) {
                            const A w = (A)(a * z[kz][mz]);
                            f[kz][0] = fma(w, q.x, f[kz][0]);
                            f[kz][1] = fma(w, q.y, f[kz][1]);
                            f[kz][2] = fma(w, q.z, f[kz][2]);
                        }
                    }
                }
        }
        for (int s = 0; s < cnt; ++s) {
            if (s == mine)
#pragma unroll
                for (int kz = 0; kz < n; ++kz)
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        double &at = sum[tid % Q * n + kz][d];
                        at = s == 0 && ch0 == kr.x ? f[kz][d] : at + f[kz][d];
                    }
            __syncthreads();
        }
    }
    for (int k = tid; k < P; k += T)
        qhat[(size_t)c * P + k] = vec4<A>((A)sum[k][0], (A)sum[k][1], (A)sum[k][2]);
}

// the children at one level gain the parent's interpolant at their proxies (NO
// points per direction)
template <int NO>
__global__ __launch_bounds__(kFmmMaxP) void fmm_l2l_kernel(Geo g, const float *__restrict__ tabg,
                                                           const int4 *__restrict__ cc,
                                                           const int *__restrict__ parent,
                                                           int cell0, double *__restrict__ v) {
    __shared__ float tab[kTabSize];
    __shared__ double sv[3 * kFmmMaxP];  // the parent's values, read by every lane
    load_tab(tabg, tab);
    const int c = cell0 + blockIdx.x;
    const int m = threadIdx.x;
    constexpr int n = NO, P = NO * NO * NO;
    {
        const double *vp = v + (size_t)parent[c] * P * 3;
        for (int i = m; i < 3 * P; i += blockDim.x) sv[i] = vp[i];
    }
    __syncthreads();
    if (m >= P) return;
    const int mx = m / (n * n), my = (m / n) % n, mz = m % n;
    const int4 cci = cc[c];
    const float *tx = tab + kTabT1 + (cci.x & 1) * kFmmMaxOrder * kFmmMaxOrder + mx;
    const float *ty = tab + kTabT1 + (cci.y & 1) * kFmmMaxOrder * kFmmMaxOrder + my;
    const float *tz = tab + kTabT1 + (cci.z & 1) * kFmmMaxOrder * kFmmMaxOrder + mz;
    const double *vp = sv;
    double sx = 0.0, sy = 0.0, sz = 0.0;
    for (int kx = 0; kx < n; ++kx)
#pragma unroll
        for (int ky = 0; ky < n; ++ky) {
            const double a = (double)(tx[kx * kFmmMaxOrder] * ty[ky * kFmmMaxOrder]);
#pragma unroll
            for (int kz = 0; kz < n; ++kz) {
                const double wk = a * (double)tz[kz * kFmmMaxOrder];
                const double *pv = vp + 3 * ((kx * n + ky) * n + kz);
                sx = fma(wk, pv[0], sx);
                sy = fma(wk, pv[1], sy);
                sz = fma(wk, pv[2], sz);
            }
        }
    double *o = v + ((size_t)c * P + m) * 3;
    o[0] += sx;
    o[1] += sy;
    o[2] += sz;
}

// ---------------------------------------------------------------- single-blob bodies
// Generalised forces (f, tau) in two channels, f and tau / a (units of a), each
// carried by the channel-wise P2M, M2M and L2L kernels above; M2L and the near
// field apply the 6 x 6 generalised tensor (Sec. 2.4) between the channels.

template <class A>
__global__ void fmm_gather6_kernel(int M, const int *__restrict__ perm,
                                   const double *__restrict__ x6, double inv_a,
                                   Vec4<A> *__restrict__ sf, Vec4<A> *__restrict__ st) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= M) return;
    const double *x = x6 + 6 * (size_t)perm[k];
    sf[k] = vec4<A>((A)x[0], (A)x[1], (A)x[2]);
    st[k] = vec4<A>((A)(x[3] * inv_a), (A)(x[4] * inv_a), (A)(x[5] * inv_a));
}

// ---------------------------------------------------------------- host tree
inline uint64_t spread3(uint64_t x) {  // 21 bits -> every third bit
    x &= 0x1fffff;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}
inline uint64_t morton(int x, int y, int z) {
    return (spread3((uint64_t)x) << 2) | (spread3((uint64_t)y) << 1) | spread3((uint64_t)z);
}
inline int compact3(uint64_t x) {  // every third bit -> 21 bits (inverse of spread3)
    x &= 0x1249249249249249ull;
    x = (x | (x >> 2)) & 0x10c30c30c30c30c3ull;
    x = (x | (x >> 4)) & 0x100f00f00f00f00full;
    x = (x | (x >> 8)) & 0x1f0000ff0000ffull;
    x = (x | (x >> 16)) & 0x1f00000000ffffull;
    x = (x | (x >> 32)) & 0x1fffffull;
    return (int)x;
}

// host threads for a step over `items` items: at most 16 (one GPU's share of the
// host), one per `each` items; the environment variable ARB_HOST_THREADS (1..16)
// caps them (the tree does not depend on the count)
int step_threads(int64_t items, int each) {
    int hw = (int)std::max(1u, std::thread::hardware_concurrency());
    if (const char *e = std::getenv("ARB_HOST_THREADS")) {
        const int v = std::atoi(e);
        if (v >= 1 && v <= 16) hw = std::min(hw, v);
    }
    return (int)std::max<int64_t>(1, std::min<int64_t>(std::min(16, hw), items / each));
}
// for the O(N) steps of the tree build
int host_threads(int N) { return step_threads(N, 65536); }
// entries of the cells' lists per thread of a step over them
constexpr int kListStep = 65536;

// FNV-1a over the bytes of a vector
template <class V>
void fnv1a(uint64_t &h, const std::vector<V> &v) {
    const unsigned char *b = reinterpret_cast<const unsigned char *>(v.data());
    const size_t n = v.size() * sizeof(V);
    for (size_t i = 0; i < n; ++i) {
        h ^= b[i];
        h *= 0x100000001b3ull;
    }
}

// Host worker threads kept for the life of the process (started on first use,
// at most 15), so that the tree build's many short parallel steps do not each
// start and join threads.  One job at a time: a caller that finds the pool busy
// (another context building its tree on another thread) gets false and runs
// the step on threads of its own.  The pool is never destroyed; its idle
// workers wait on a condition variable until the process ends.
class HostPool {
  public:
    // slice(t) for t in [0, T): t = 0 on the caller's thread, the others on
    // workers; slice must not throw.  False (nothing run) when the pool is busy
    // or cannot start enough workers.
    bool run(int T, const std::function<void(int)> &slice) {
        std::unique_lock<std::mutex> busy(busy_, std::try_to_lock);
        if (!busy.owns_lock()) return false;
        {
            std::lock_guard<std::mutex> lk(mu_);
            try {
                while ((int)workers_.size() < T - 1) {
                    const int id = (int)workers_.size() + 1;
                    workers_.emplace_back([this, id] { worker(id); });
                }
            } catch (const std::system_error &) {
                return false;
            }
            job_ = &slice;
            job_T_ = T;
            pending_ = T - 1;
            ++gen_;
        }
        cv_.notify_all();
        slice(0);
        std::unique_lock<std::mutex> lk(mu_);
        done_.wait(lk, [this] { return pending_ == 0; });
        job_ = nullptr;
        return true;
    }

  private:
    void worker(int id) {
        uint64_t seen = 0;
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            cv_.wait(lk, [&] { return gen_ != seen; });
            seen = gen_;
            if (id >= job_T_) continue;
            const std::function<void(int)> *f = job_;
            lk.unlock();
            (*f)(id);
            lk.lock();
            if (--pending_ == 0) done_.notify_one();
        }
    }
    std::mutex busy_, mu_;
    std::condition_variable cv_, done_;
    std::vector<std::thread> workers_;
    const std::function<void(int)> *job_ = nullptr;
    int job_T_ = 0, pending_ = 0;
    uint64_t gen_ = 0;
};

HostPool &host_pool() {
    static HostPool *pool = new HostPool;  // never freed (see above)
    return *pool;
}

// f(t, i0, i1) on T contiguous slices of [0, N), slice t on thread t (of the
// host pool, or of threads started for this step when the pool is busy).  An
// exception in a slice is caught on its thread and rethrown on the caller's
// after every slice has ended; a slice whose thread cannot be started runs on
// the caller's thread (the result does not depend on where a slice runs).
template <class F>
void parallel_slices(int T, int N, F &&f) {
    if (T <= 1) {
        f(0, 0, N);
        return;
    }
    std::vector<std::exception_ptr> err((size_t)T);
    const std::function<void(int)> slice = [&f, &err, T, N](int t) {
        const int i0 = (int)((int64_t)N * t / T), i1 = (int)((int64_t)N * (t + 1) / T);
        try {
            f(t, i0, i1);
        } catch (...) {
            err[t] = std::current_exception();
        }
    };
    if (!host_pool().run(T, slice)) {
        std::vector<std::thread> th;
        th.reserve(T);
        for (int t = 0; t < T; ++t) {
            try {
                th.emplace_back(slice, t);
            } catch (const std::system_error &) {
                slice(t);
            }
        }
        for (auto &x : th) x.join();
    }
    for (auto &e : err)
        if (e) std::rethrow_exception(e);
}

// per-cell lists on host threads: f(c, out) appends the entries of item c to
// out for c in [0, n); ptr gets the prefix sums of their counts and out the
// entries joined in item order, as a loop over the items would give them
template <class V, class F>
void lists_by_item(int threads, int n, std::vector<int> &ptr, std::vector<V> &out, F &&f) {
    const int T = std::max(1, std::min(threads, n / 256));
    std::vector<std::vector<V>> part((size_t)T);
    ptr.assign((size_t)n + 1, 0);
    parallel_slices(T, n, [&](int t, int c0, int c1) {
        std::vector<V> &v = part[t];
        for (int c = c0; c < c1; ++c) {
            const size_t before = v.size();
            f(c, v);
            ptr[c + 1] = (int)(v.size() - before);
        }
    });
    for (int c = 0; c < n; ++c) ptr[c + 1] += ptr[c];
    out.clear();
    out.reserve((size_t)ptr[n]);
    for (const std::vector<V> &v : part) out.insert(out.end(), v.begin(), v.end());
}

// open-addressing map from the Morton keys of one level's cells (< 2^48) to
// their indices
struct CellHash {
    std::vector<uint64_t> keys;
    std::vector<int> vals;
    uint64_t mask = 0;
    static uint64_t mix(uint64_t x) {
        x ^= x >> 30;
        x *= 0xbf58476d1ce4e5b9ull;
        x ^= x >> 27;
        x *= 0x94d049bb133111ebull;
        return x ^ (x >> 31);
    }
    // the keys k[0..n) (distinct) with values base + i; up to `threads` host
    // threads claim slots with compare-and-swap, so the table's layout may depend
    // on their timing, but every lookup finds the same value
    void build(const uint64_t *k, int n, int base, int threads);
    // index of the cell with coordinates (x, y, z) at a level of side 2^l, or -1
    int get(int l, int x, int y, int z) const {
        const int lim = 1 << l;
        if (x < 0 || y < 0 || z < 0 || x >= lim || y >= lim || z >= lim) return -1;
        const uint64_t k = morton(x, y, z);
        for (uint64_t h = mix(k) & mask; keys[h] != ~0ull; h = (h + 1) & mask)
            if (keys[h] == k) return vals[h];
        return -1;
    }
};

void CellHash::build(const uint64_t *k, int n, int base, int threads) {
    size_t cap = 16;
    while (cap < 2 * (size_t)n) cap *= 2;
    mask = cap - 1;
    keys.assign(cap, ~0ull);
    vals.assign(cap, -1);
    const int T = std::max(1, std::min(threads, n / 16384));
    parallel_slices(T, n, [&](int, int i0, int i1) {
        for (int i = i0; i < i1; ++i) {
            uint64_t h = mix(k[i]) & mask;
            for (;;) {
                uint64_t empty = ~0ull;
                if (__atomic_compare_exchange_n(&keys[h], &empty, k[i], false, __ATOMIC_RELAXED,
                                                __ATOMIC_RELAXED)) {
                    vals[h] = base + i;
                    break;
                }
                h = (h + 1) & mask;
            }
        }
    });
}

// work items per cell of M2L's sparse part: one, or up to 8 when there are too few
// cells to fill the chip (about 2,048 items wanted)
int m2l_splits(int cells) {
    return std::max(1, std::min(8, (2048 + cells - 1) / std::max(cells, 1)));
}

}  // namespace

// the octree of N positions (units of length, host memory), built on the host
struct FmmPlan {
    int n = 0, P = 0, L = 0, ncell = 0, nleaf = 0;
    double o[3] = {0.0, 0.0, 0.0}, S = 0.0;  // root cube, units of length
    int64_t n_near_pairs = 0, n_m2l_pairs = 0;
    std::vector<int> perm, lvl, parent, il_ptr, il, near_ptr, nearl;
    std::vector<int4> cc;
    std::vector<int2> rng, kids, work;
    std::vector<float> tab;
};

// Host scratch of the tree build: grow-only arrays whose contents are not
// initialised (every entry used is written first), kept between builds so that
// their pages are allocated and touched once
template <class T>
struct HostArr {
    std::unique_ptr<T[]> p;
    size_t n = 0;
    T *get(size_t m) {
        if (m > n || !p) {
            p.reset(new T[std::max<size_t>(m, 1)]);
            n = std::max<size_t>(m, 1);
        }
        return p.get();
    }
};
// M2L's work (fmm_m2l.hip): per cell of levels 2..L the sparse listed cells and the
// slots of its dense entries, the dense entries grouped into batches, and the
// chunks of cells that share the slots' memory
struct M2LGroups {
    std::vector<int> sp_ptr, sp, sp_order, slot_ptr, count, zidx, blobs, sparse, listed, key;
    std::vector<int2> cols;
    std::vector<FmmBatch> batches;
    std::vector<FmmChunk> chunks;
    int max_slots = 0;  // of a chunk
};
// the near field's work (fmm_near.hip): blocks of targets (leaf, first target,
// targets, first slot) and, per leaf, the slots that other blocks fill for it
struct NearBlocks {
    std::vector<int4> blocks, by_leaf;
    std::vector<int> in_ptr, in, first, next;
    std::vector<int64_t> visited, per_block, cost;
    int64_t slots = 0;  // blobs' worth of slots (3 doubles each)
};
struct PlanScratch {
    HostArr<int> crd, idx, idx2;
    HostArr<uint64_t> key, key2;
    HostArr<unsigned char> first;
};

}  // namespace arb

// what a context keeps of its tree builds: the scratch, the last plan (its
// vectors' capacity is reused) and pinned host memory for the positions
struct arb::FmmHostCache {
    PlanScratch scratch;
    FmmPlan plan;
    M2LGroups m2l;
    NearBlocks near;
    double *hpos = nullptr;
    size_t hpos_n = 0;
    FmmHostCache() = default;
    FmmHostCache(const FmmHostCache &) = delete;
    FmmHostCache &operator=(const FmmHostCache &) = delete;
    ~FmmHostCache() {
        if (hpos) (void)hipHostFree(hpos);
    }
    // pinned room for n doubles (null when it cannot be allocated)
    double *positions(size_t n) {
        if (n <= hpos_n && hpos) return hpos;
        if (hpos) (void)hipHostFree(hpos);
        hpos = nullptr;
        hpos_n = 0;
        if (hipHostMalloc((void **)&hpos, n * sizeof(double), hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            hpos = nullptr;
            return nullptr;
        }
        hpos_n = n;
        return hpos;
    }
};

namespace arb {

int fmm_plan(FmmPlan &pl, PlanScratch &sc, int N, const double *h, double a, int n, int levels,
             int leaf, std::string *msg) {
    const int P = n * n * n;
    const int T = host_threads(N);
    // finite positions and the root cube (host threads over slices; min and max
    // are exact, so the result does not depend on the slicing)
    std::vector<double> bound(6 * (size_t)T);
    std::vector<char> bad((size_t)T, 0);
    parallel_slices(T, N, [&](int t, int i0, int i1) {
        // running bounds in registers, stored once (the threads' slots share
        // cache lines)
        double lo[3] = {h[0], h[1], h[2]}, up[3] = {h[0], h[1], h[2]};
        bool finite = true;
        for (int i = i0; i < i1; ++i)
            for (int d = 0; d < 3; ++d) {
                const double x = h[3 * (size_t)i + d];
                finite = finite && std::isfinite(x);
                lo[d] = std::min(lo[d], x);
                up[d] = std::max(up[d], x);
            }
        for (int d = 0; d < 3; ++d) {
            bound[6 * (size_t)t + d] = lo[d];
            bound[6 * (size_t)t + 3 + d] = up[d];
        }
        if (!finite) bad[t] = 1;
    });
    for (int t = 0; t < T; ++t)
        if (bad[t]) {
            *msg = "fast product: a position is not finite";
            return ARB_E_NAN;
        }
    double o[3] = {h[0], h[1], h[2]}, hi_d[3] = {h[0], h[1], h[2]}, ext = 0.0;
    for (int t = 0; t < T; ++t)
        for (int d = 0; d < 3; ++d) {
            o[d] = std::min(o[d], bound[6 * (size_t)t + d]);
            hi_d[d] = std::max(hi_d[d], bound[6 * (size_t)t + 3 + d]);
        }
    for (int d = 0; d < 3; ++d) ext = std::max(ext, hi_d[d] - o[d]);
    const double S = ext > 0.0 ? ext * (1.0 + 0x1p-20) : a;
    int Lhi = 0;  // deepest level with a cell side >= 2a
    while (Lhi < kFmmMaxLevel && S / std::ldexp(1.0, Lhi + 1) >= 2.0 * a) ++Lhi;
    // cell coordinates at level Lhi and Morton keys (host threads over slices;
    // the arrays are left uninitialised, so that their pages are first touched
    // by the threads that fill them)
    int *crd = sc.crd.get(3 * (size_t)N);
    uint64_t *key = sc.key.get(N), *key2 = sc.key2.get(N);
    int *idx = sc.idx.get(N), *idx2 = sc.idx2.get(N);
    const double scale = std::ldexp(1.0, Lhi);
    parallel_slices(T, N, [&](int, int i0, int i1) {
        for (int i = i0; i < i1; ++i) {
            int cq[3];
            for (int d = 0; d < 3; ++d) {
                const double u = (h[3 * (size_t)i + d] - o[d]) / S;
                cq[d] = (int)std::floor(u * scale);
                crd[3 * (size_t)i + d] = cq[d];
            }
            key[i] = morton(cq[0], cq[1], cq[2]);
            idx[i] = i;
        }
    });
    // stable LSD radix sort of the 3 Lhi-bit keys in the fewest passes of at
    // most 14 bits: blobs in Morton order, equal keys in ascending blob index.
    // Each thread counts and then scatters its own contiguous slice, at offsets
    // ordered by bucket and then by thread, which keeps the sort stable.
    {
        const int bits = 3 * Lhi, passes = (bits + 13) / 14;
        const int dbits = passes ? (bits + passes - 1) / passes : 0;
        const size_t B = (size_t)1 << dbits;
        const uint64_t mask = B - 1;
        std::vector<int> cnt((size_t)T * B);
        for (int ps = 0; ps < passes; ++ps) {
            const int shift = ps * dbits;
            parallel_slices(T, N, [&](int t, int i0, int i1) {
                int *c = cnt.data() + (size_t)t * B;
                std::fill(c, c + B, 0);
                for (int i = i0; i < i1; ++i) ++c[(key[i] >> shift) & mask];
            });
            int run = 0;
            for (size_t b = 0; b < B; ++b)
                for (int t = 0; t < T; ++t) {
                    const int m = cnt[(size_t)t * B + b];
                    cnt[(size_t)t * B + b] = run;
                    run += m;
                }
            parallel_slices(T, N, [&](int t, int i0, int i1) {
                int *c = cnt.data() + (size_t)t * B;
                for (int i = i0; i < i1; ++i) {
                    const int at = c[(key[i] >> shift) & mask]++;
                    key2[at] = key[i];
                    idx2[at] = idx[i];
                }
            });
            std::swap(key, key2);
            std::swap(idx, idx2);
        }
    }
    // the shallowest level at which sorted blob j starts a new cell (a cell
    // starts at every deeper level too): the highest differing key bit / 3
    unsigned char *first = sc.first.get(N);
    first[0] = 0;
    std::vector<int64_t> new_at_t((size_t)T * (Lhi + 2), 0), new_at(Lhi + 2, 0);
    parallel_slices(T, N, [&](int t, int i0, int i1) {
        int64_t *na = new_at_t.data() + (size_t)t * (Lhi + 2);
        for (int j = std::max(i0, 1); j < i1; ++j) {
            const uint64_t d = key[j] ^ key[j - 1];
            if (!d) {
                first[j] = (unsigned char)(Lhi + 1);  // same cell at every level
                continue;
            }
            const int hb = 63 - __builtin_clzll(d);
            first[j] = (unsigned char)(Lhi - hb / 3);
            ++na[first[j]];
        }
    });
    for (int t = 0; t < T; ++t)
        for (int l = 0; l < Lhi + 2; ++l) new_at[l] += new_at_t[(size_t)t * (Lhi + 2) + l];
    // the cells of levels 0..L with their blob ranges, parents and children, the
    // interaction lists, the adjacent leaves and the work items of leaf level L
    auto build = [&](int L, FmmPlan &q) -> int {
        // cells of every level in Morton order, with their blob ranges
        std::vector<std::vector<int>> starts_t((size_t)T * (L + 1));
        parallel_slices(T, N, [&](int t, int i0, int i1) {
            std::vector<int> *st = starts_t.data() + (size_t)t * (L + 1);
            for (int j = std::max(i0, 1); j < i1; ++j)
                for (int l = first[j]; l <= L; ++l) st[l].push_back(j);
        });
        std::vector<std::vector<int>> starts(L + 1, std::vector<int>(1, 0));
        for (int t = 0; t < T; ++t)
            for (int l = 0; l <= L; ++l) {
                const std::vector<int> &st = starts_t[(size_t)t * (L + 1) + l];
                starts[l].insert(starts[l].end(), st.begin(), st.end());
            }
        std::vector<int4> cc;
        std::vector<int2> rng;
        std::vector<uint64_t> pk;
        std::vector<int> lvl(L + 2, 0);
        for (int l = 0; l <= L; ++l) {
            lvl[l] = (int)cc.size();
            const int sh = 3 * (Lhi - l), dl = Lhi - l;
            const std::vector<int> &st = starts[l];
            for (size_t t = 0; t < st.size(); ++t) {
                const int j = st[t], e = t + 1 < st.size() ? st[t + 1] : N;
                const int i0 = idx[j];
                cc.push_back(make_int4(crd[3 * (size_t)i0] >> dl, crd[3 * (size_t)i0 + 1] >> dl,
                                       crd[3 * (size_t)i0 + 2] >> dl, l));
                rng.push_back(make_int2(j, e));
                pk.push_back(key[j] >> sh);
            }
        }
        lvl[L + 1] = (int)cc.size();
        const int ncell = (int)cc.size();
        std::vector<int> parent(ncell, -1);
        std::vector<int2> kids(ncell, make_int2(0, 0));
        for (int l = 1; l <= L; ++l) {
            int p = lvl[l - 1];
            for (int c = lvl[l]; c < lvl[l + 1]; ++c) {
                while (rng[p].y <= rng[c].x) ++p;
                parent[c] = p;
                if (kids[p].y == 0) kids[p] = make_int2(c, c + 1);
                else kids[p].y = c + 1;
            }
        }
        std::vector<CellHash> hash(L + 1);
        for (int l = 0; l <= L; ++l)
            hash[l].build(pk.data() + lvl[l], lvl[l + 1] - lvl[l], lvl[l], T);
        auto find = [&](int l, int x, int y, int z) -> int { return hash[l].get(l, x, y, z); };
        auto adjacent = [&](int c1, int c2) {
            return std::abs(cc[c1].x - cc[c2].x) <= 1 && std::abs(cc[c1].y - cc[c2].y) <= 1 &&
                   std::abs(cc[c1].z - cc[c2].z) <= 1;
        };
        // interaction lists (levels 2..L) and the adjacent leaves
        std::vector<int> il_ptr, il;
        lists_by_item(T, ncell, il_ptr, il, [&](int c, std::vector<int> &out) {
            const int l = cc[c].w;
            if (l < 2) return;
            const int4 pc = cc[parent[c]];
            for (int dx = -1; dx <= 1; ++dx)
                for (int dy = -1; dy <= 1; ++dy)
                    for (int dz = -1; dz <= 1; ++dz) {
                        const int q = find(l - 1, pc.x + dx, pc.y + dy, pc.z + dz);
                        if (q < 0) continue;
                        for (int ch = kids[q].x; ch < kids[q].y; ++ch)
                            if (!adjacent(ch, c)) out.push_back(ch);
                    }
        });
        const int leaf0 = lvl[L], nleaf = lvl[L + 1] - lvl[L];
        std::vector<int> near_ptr, nearl;
        lists_by_item(T, nleaf, near_ptr, nearl, [&](int i, std::vector<int> &out) {
            const int4 c4 = cc[leaf0 + i];
            for (int dx = -1; dx <= 1; ++dx)
                for (int dy = -1; dy <= 1; ++dy)
                    for (int dz = -1; dz <= 1; ++dz) {
                        const int q = find(L, c4.x + dx, c4.y + dy, c4.z + dz);
                        if (q >= 0) out.push_back(q);
                    }
        });
        std::vector<int2> work;
        for (int c = leaf0; c < leaf0 + nleaf; ++c)
            for (int k0 = rng[c].x; k0 < rng[c].y; k0 += kNearBlock) work.push_back(make_int2(c, k0));
        // per cell the blobs of its interaction list, and M2L's pair evaluations: n^3 per
        // proxy of each listed cell, or per blob when it holds fewer blobs than proxies
        const int Tl = step_threads((int64_t)il.size(), kListStep);
        std::vector<int64_t> listed((size_t)ncell), m2l((size_t)Tl);
        parallel_slices(Tl, ncell, [&](int t, int c0, int c1) {
            int64_t pairs = 0;
            for (int c = c0; c < c1; ++c) {
                int64_t m = 0;
                for (int e = il_ptr[c]; e < il_ptr[c + 1]; ++e) {
                    const int n = rng[il[e]].y - rng[il[e]].x;
                    m += n;
                    pairs += (int64_t)P * std::min(P, n);
                }
                listed[c] = m;
            }
            m2l[t] = pairs;
        });
        // every target sees every source exactly once: the adjacent leaves and the
        // interaction lists of its ancestors hold N blobs between them, and every
        // index handed to a kernel is in range
        const int Tn = step_threads((int64_t)nearl.size(), kListStep);
        std::vector<int64_t> pairs((size_t)Tn);
        std::vector<int> fault((size_t)Tn, 0);
        parallel_slices(Tn, nleaf, [&](int t, int i0, int i1) {
            int64_t near = 0;
            for (int i = i0; i < i1 && !fault[t]; ++i) {
                const int c = leaf0 + i;
                int64_t cnt = 0;
                for (int e = near_ptr[i]; e < near_ptr[i + 1]; ++e) {
                    const int q = nearl[e];
                    if (q < leaf0 || q >= leaf0 + nleaf) {
                        fault[t] = 1;
                        break;
                    }
                    cnt += rng[q].y - rng[q].x;
                }
                near += cnt * (rng[c].y - rng[c].x);
                for (int a2 = c; a2 >= 0 && cc[a2].w >= 2; a2 = parent[a2]) cnt += listed[a2];
                if (cnt != N && !fault[t]) fault[t] = 2;
            }
            pairs[t] = near;
        });
        for (int f : fault)
            if (f) {
                *msg = f == 1 ? "fast product: internal error (near list)"
                              : "fast product: internal error (cells do not partition the blobs)";
                return ARB_E_ARG;
            }
        q.L = L;
        q.ncell = ncell;
        q.nleaf = nleaf;
        q.n_m2l_pairs = std::accumulate(m2l.begin(), m2l.end(), int64_t(0));
        q.n_near_pairs = std::accumulate(pairs.begin(), pairs.end(), int64_t(0));
        q.lvl = std::move(lvl);
        q.cc = std::move(cc);
        q.rng = std::move(rng);
        q.parent = std::move(parent);
        q.kids = std::move(kids);
        q.il_ptr = std::move(il_ptr);
        q.il = std::move(il);
        q.near_ptr = std::move(near_ptr);
        q.nearl = std::move(nearl);
        q.work = std::move(work);
        return 0;
    };
    // leaf level
    int rc;
    if (Lhi < 2) {
        rc = build(0, pl);
    } else if (levels > 0) {
        rc = build(levels < 2 ? 0 : std::min(levels, Lhi), pl);
    } else if (leaf > 0) {
        // the shallowest level whose mean occupancy is at most `leaf`
        int L = Lhi;
        int64_t cells = 1;
        for (int l = 1; l <= Lhi; ++l) {
            cells += new_at[l];
            if (l >= 2 && (int64_t)N <= (int64_t)leaf * cells) {
                L = l;
                break;
            }
        }
        rc = build(L, pl);
    } else {
        // the level with the fewest pair evaluations: deeper from level 2 while
        // the count falls.  Counted level by level (the interaction lists of the
        // shallower levels are the same for every leaf level), then built once.
        // the cells of level l: each host thread finds the cell starts in its
        // slice of the sorted blobs, the slices' lists then joined in order
        // (each thread fills its own cells, at the offset of its slice; a cell's
        // coordinates are decoded from its Morton key)
        std::vector<std::vector<int>> st_t((size_t)T);
        std::vector<size_t> st_off((size_t)T + 1);
        std::vector<int> st_next((size_t)T);
        auto cells_of = [&](int l, std::vector<int4> &c4, std::vector<int2> &r2,
                            std::vector<uint64_t> &k) {
            parallel_slices(T, N, [&](int t, int i0, int i1) {
                std::vector<int> &v = st_t[t];
                v.clear();
                for (int j = i0; j < i1; ++j)
                    if (j == 0 || first[j] <= l) v.push_back(j);
            });
            st_off[0] = 0;
            for (int t = 0; t < T; ++t) st_off[t + 1] = st_off[t] + st_t[t].size();
            for (int t = T - 1, nx = N; t >= 0; --t) {  // first cell start after slice t
                st_next[t] = nx;
                if (!st_t[t].empty()) nx = st_t[t][0];
            }
            const size_t nc = st_off[T];
            c4.resize(nc);
            r2.resize(nc);
            k.resize(nc);
            const int sh = 3 * (Lhi - l);
            parallel_slices(T, T, [&](int t, int, int) {
                const std::vector<int> &v = st_t[t];
                const size_t c0 = st_off[t];
                for (size_t e = 0; e < v.size(); ++e) {
                    const uint64_t kc = key[v[e]] >> sh;
                    c4[c0 + e] = make_int4(compact3(kc >> 2), compact3(kc >> 1), compact3(kc), l);
                    r2[c0 + e] = make_int2(v[e], e + 1 < v.size() ? v[e + 1] : st_next[t]);
                    k[c0 + e] = kc;
                }
            });
        };
        std::vector<int4> pc, cc2;
        std::vector<int2> pr, rr;
        std::vector<uint64_t> pk2, kk2;
        CellHash ph, ch;
        cells_of(1, pc, pr, pk2);
        ph.build(pk2.data(), (int)pk2.size(), 0, T);
        int64_t m2l_total = 0, best = -1;
        int L = 2;
        for (int l = 2; l <= Lhi; ++l) {
            cells_of(l, cc2, rr, kk2);
            ch.build(kk2.data(), (int)kk2.size(), 0, T);
            // children of each parent (contiguous) and the parent of each cell
            std::vector<int2> kid(pc.size());
            std::vector<int> par(cc2.size());
            for (size_t p = 0, c = 0; p < pc.size(); ++p) {
                const size_t c0 = c;
                while (c < cc2.size() && rr[c].x < pr[p].y) par[c++] = (int)p;
                kid[p] = make_int2((int)c0, (int)c);
            }
            // integer counts over slices of the cells on host threads
            const int ncl = (int)cc2.size();
            const int Tc = std::max(1, std::min(T, ncl / 256));
            std::vector<int64_t> part(2 * (size_t)Tc, 0);
            parallel_slices(Tc, ncl, [&](int t, int c0, int c1) {
                int64_t m2l = 0, near = 0;
                for (int c = c0; c < c1; ++c) {
                    const int4 q = pc[par[c]];
                    int64_t adj = 0;
                    for (int dx = -1; dx <= 1; ++dx)
                        for (int dy = -1; dy <= 1; ++dy)
                            for (int dz = -1; dz <= 1; ++dz) {
                                const int g = ph.get(l - 1, q.x + dx, q.y + dy, q.z + dz);
                                if (g >= 0)
                                    for (int k = kid[g].x; k < kid[g].y; ++k)
                                        if (std::abs(cc2[k].x - cc2[c].x) > 1 ||
                                            std::abs(cc2[k].y - cc2[c].y) > 1 ||
                                            std::abs(cc2[k].z - cc2[c].z) > 1)
                                            m2l += (int64_t)P * std::min(P, rr[k].y - rr[k].x);
                                const int e =
                                    ch.get(l, cc2[c].x + dx, cc2[c].y + dy, cc2[c].z + dz);
                                if (e >= 0) adj += rr[e].y - rr[e].x;
                            }
                    near += adj * (rr[c].y - rr[c].x);
                }
                part[2 * (size_t)t] = m2l;
                part[2 * (size_t)t + 1] = near;
            });
            int64_t near_pairs = 0;
            for (int t = 0; t < Tc; ++t) {
                m2l_total += part[2 * (size_t)t];
                near_pairs += part[2 * (size_t)t + 1];
            }
            const int64_t cl = near_pairs + m2l_total;
            if (best >= 0 && cl >= best) break;
            best = cl;
            L = l;
            pc.swap(cc2);
            pr.swap(rr);
            pk2.swap(kk2);
            std::swap(ph, ch);
        }
        rc = build(L, pl);
    }
    if (rc) return rc;
    // Chebyshev points, Lagrange denominators, parent polynomials at child proxies
    std::vector<float> tab(kTabSize, 0.f);
    double xn[kFmmMaxOrder];
    for (int k = 0; k < n; ++k) xn[k] = std::cos((2 * k + 1) * kPi / (2 * n));
    for (int k = 0; k < n; ++k) {
        double den = 1.0;
        for (int j = 0; j < n; ++j)
            if (j != k) den *= xn[k] - xn[j];
        tab[kTabNode + k] = (float)xn[k];
        tab[kTabDen + k] = (float)(1.0 / den);
    }
    for (int sg = 0; sg < 2; ++sg)
        for (int k = 0; k < n; ++k)
            for (int m = 0; m < n; ++m) {
                const double u = (sg ? 0.5 : -0.5) + 0.5 * xn[m];
                double p = 1.0;
                for (int j = 0; j < n; ++j)
                    if (j != k) p *= (u - xn[j]) / (xn[k] - xn[j]);
                tab[kTabT1 + (sg * kFmmMaxOrder + k) * kFmmMaxOrder + m] = (float)p;
            }
    pl.n = n;
    pl.P = P;
    pl.o[0] = o[0];
    pl.o[1] = o[1];
    pl.o[2] = o[2];
    pl.S = S;
    pl.perm.assign(idx, idx + N);  // sorted position -> blob
    pl.tab = std::move(tab);
    return 0;
}

// Work items longest first when there are so few that the last ones to start decide
// when a launch ends (a few per compute unit; with more, neighbours stay together for
// the caches): cost[k] >= 0 of item k, the order in `order`; equal costs keep their order
// (a stable radix sort, 12 bits a pass)
constexpr int kSortItems = 16384;
template <class V>
static void longest_first(const std::vector<V> &cost, std::vector<int> &order) {
    const size_t n = cost.size();
    order.resize(n);
    for (size_t k = 0; k < n; ++k) order[k] = (int)k;
    if (n > kSortItems || n < 2) return;
    const V top = *std::max_element(cost.begin(), cost.end());
    std::vector<int> other(n), count;
    for (int shift = 0; shift < 63 && (uint64_t)top >> shift; shift += 12) {
        auto digit = [&](int k) { return (uint64_t)(top - cost[k]) >> shift & 4095; };
        count.assign(4097, 0);
        for (int k : order) ++count[digit(k) + 1];
        for (int d = 0; d < 4096; ++d) count[d + 1] += count[d];
        for (int k : order) other[count[digit(k)]++] = k;
        order.swap(other);
    }
}

// Groups the interaction lists for M2L.  Entries whose listed cell holds at least P
// blobs are dense: they get a slot each, numbered in list order within a chunk of
// target cells, and are sorted (counting sort, stable) by the key that fixes the
// tensor between the two proxy grids: the level, the cells' offset and, above the
// wall, the target cell's height.  Equal keys make batches of at most max_cols
// columns.  Host threads take slices of the cells, each with counts of its own, and
// place their entries in slice order, as one thread would.
static void group_m2l(const FmmPlan &pl, bool wall, int max_cols, int64_t chunk_slots,
                      M2LGroups &G) {
    G.batches.clear();
    G.chunks.clear();
    G.max_slots = 0;
    const int cell0 = pl.L >= 2 ? pl.lvl[2] : pl.ncell, nc = pl.ncell - cell0, P = pl.P;
    const int T = step_threads((int64_t)pl.il.size(), kListStep);
    // blobs of a cell when it is sparse, 0 when it is dense (the passes over the lists
    // do not branch on it: both kinds are mixed); strung: proxies, every cell counts as sparse
    const bool strung = pl.n == kFmmStrungOrder;
    G.sparse.resize((size_t)pl.ncell);
    for (int c = 0; c < pl.ncell; ++c) {
        const int m = pl.rng[c].y - pl.rng[c].x;
        G.sparse[c] = m < P ? m : (strung ? P : 0);
    }
    G.sp_ptr.assign((size_t)nc + 1, 0);
    G.slot_ptr.assign((size_t)nc + 1, 0);
    G.blobs.assign((size_t)nc, 0);
    parallel_slices(T, nc, [&](int, int i0, int i1) {
        for (int i = i0; i < i1; ++i) {
            const int e0 = pl.il_ptr[cell0 + i], e1 = pl.il_ptr[cell0 + i + 1];
            int d = 0, m = 0;
            for (int e = e0; e < e1; ++e) {
                const int n = G.sparse[pl.il[e]];
                d += n == 0;
                m += n;
            }
            G.slot_ptr[i + 1] = d;
            G.sp_ptr[i + 1] = e1 - e0 - d;
            G.blobs[i] = m;
        }
    });
    for (int i = 0; i < nc; ++i) {
        G.sp_ptr[i + 1] += G.sp_ptr[i];
        G.slot_ptr[i + 1] += G.slot_ptr[i];
    }
    // the sparse listed cells, and the dense one of each slot
    G.sp.resize((size_t)G.sp_ptr[nc]);
    G.listed.resize((size_t)G.slot_ptr[nc]);
    G.key.resize((size_t)G.slot_ptr[nc]);
    parallel_slices(T, nc, [&](int, int i0, int i1) {
        int *to[2] = {G.sp.data() + G.sp_ptr[i0], G.listed.data() + G.slot_ptr[i0]};
        for (int e = pl.il_ptr[cell0 + i0]; e < pl.il_ptr[cell0 + i1]; ++e) {
            const int q = pl.il[e];
            *to[G.sparse[q] == 0]++ = q;
        }
    });
    longest_first(G.blobs, G.sp_order);
    G.cols.resize((size_t)G.slot_ptr[nc]);
    for (int a = 0; a < nc;) {
        int b = a + 1;
        while (b < nc && G.slot_ptr[b + 1] - G.slot_ptr[a] <= chunk_slots) ++b;
        FmmChunk ch{a, b, (int)G.batches.size(), 0, G.slot_ptr[a]};
        for (int x = a; x < b;) {  // the cells of one level
            const int l = pl.cc[cell0 + x].w;
            int y = x + 1;
            while (y < b && pl.cc[cell0 + y].w == l) ++y;
            // the heights that occur, numbered
            int z0 = pl.cc[cell0 + x].z, z1 = z0, nz = 1;
            if (wall) {
                for (int i = x; i < y; ++i) {
                    z0 = std::min(z0, pl.cc[cell0 + i].z);
                    z1 = std::max(z1, pl.cc[cell0 + i].z);
                }
                G.zidx.assign((size_t)(z1 - z0 + 1), -1);
                nz = 0;
                for (int i = x; i < y; ++i) {
                    int &zi = G.zidx[pl.cc[cell0 + i].z - z0];
                    if (zi < 0) zi = nz++;
                }
            }
            const int base = G.slot_ptr[x], m = G.slot_ptr[y] - base, keys = nz * 343;
            // (summing up the counts takes less than placing the entries)
            const int Tr = std::max(1, std::min(step_threads(m, kListStep / 2), m / keys));
            G.count.assign((size_t)Tr * keys, 0);
            parallel_slices(Tr, y - x, [&](int t, int i0, int i1) {
                int *n = G.count.data() + (size_t)t * keys;
                for (int i = x + i0; i < x + i1; ++i) {
                    const int4 c = pl.cc[cell0 + i];
                    const int k0 = wall ? G.zidx[c.z - z0] * 343 : 0;
                    for (int e = G.slot_ptr[i]; e < G.slot_ptr[i + 1]; ++e) {
                        const int4 q = pl.cc[G.listed[e]];
                        const int k = k0 + ((c.x - q.x + 3) * 7 + (c.y - q.y + 3)) * 7 +
                                      (c.z - q.z + 3);
                        G.key[e] = k;
                        ++n[k];
                    }
                }
            });
            // counts to places: by key, then by slice; the key's batches on the way
            for (int zi = 0, run = base; zi < nz; ++zi) {
                int tz = 0;
                if (wall)
                    while (G.zidx[tz] != zi) ++tz;
                for (int d = 0; d < 343; ++d) {
                    const int k0 = run;
                    for (int t = 0; t < Tr; ++t) {
                        int &n = G.count[(size_t)t * keys + zi * 343 + d];
                        run += std::exchange(n, run);
                    }
                    for (int f = k0; f < run; f += max_cols)
                        G.batches.push_back(FmmBatch{f, std::min(max_cols, run - f), l,
                                                     wall ? z0 + tz : 0, d / 49 - 3,
                                                     (d / 7) % 7 - 3, d % 7 - 3, 0});
                }
            }
            parallel_slices(Tr, y - x, [&](int t, int i0, int i1) {
                int *at = G.count.data() + (size_t)t * keys;
                for (int e = G.slot_ptr[x + i0]; e < G.slot_ptr[x + i1]; ++e)
                    G.cols[at[G.key[e]]++] = make_int2(G.listed[e], e - ch.slot0);
            });
            x = y;
        }
        ch.batch1 = (int)G.batches.size();
        G.max_slots = std::max(G.max_slots, G.slot_ptr[b] - G.slot_ptr[a]);
        G.chunks.push_back(ch);
        a = b;
    }
}

// Blocks of at most kNearBlock targets of one leaf; with sym, the slots of each block: one
// per adjacent leaf after its own (in list order), |leaf| blobs each, and per leaf the
// slots that the blocks before fill for it, in the blocks' order by leaf.
static void near_blocks(const FmmPlan &pl, bool sym, NearBlocks &B) {
    const int leaf0 = pl.lvl[pl.L], n = pl.nleaf;
    const int T = step_threads((int64_t)pl.nearl.size(), kListStep);
    auto size = [&](int c) { return pl.rng[c].y - pl.rng[c].x; };
    auto count = [&](int c) { return (size(c) + kNearBlock - 1) / kNearBlock; };
    B.visited.resize((size_t)n);
    B.per_block.resize((size_t)n);
    parallel_slices(T, n, [&](int, int i0, int i1) {
        for (int i = i0; i < i1; ++i) {
            int64_t all = 0, after = 0;
            for (int e = pl.near_ptr[i]; e < pl.near_ptr[i + 1]; ++e) {
                const int q = pl.nearl[e];
                all += size(q);
                if (q > leaf0 + i) after += size(q);
            }
            B.visited[i] = sym ? after + size(leaf0 + i) : all;
            B.per_block[i] = sym ? after : 0;
        }
    });
    B.first.resize((size_t)n + 1);
    B.first[0] = 0;
    B.slots = 0;
    for (int i = 0; i < n; ++i) {
        B.first[i + 1] = B.first[i] + count(leaf0 + i);
        B.slots += count(leaf0 + i) * B.per_block[i];
    }
    B.in.clear();
    B.in_ptr.assign((size_t)n + 1, 0);
    const bool fits = B.slots <= kFmmNearSlots;  // else the caller takes the other form
    B.by_leaf.resize((size_t)B.first[n]);
    B.cost.resize((size_t)B.first[n]);
    for (int64_t i = 0, at = 0; i < n; ++i) {
        const int2 r = pl.rng[leaf0 + i];
        for (int b = B.first[i], t = r.x; t < r.y; ++b, t += kNearBlock) {
            B.by_leaf[b] = make_int4(leaf0 + (int)i, t, std::min(kNearBlock, r.y - t),
                                     fits ? (int)at : 0);
            B.cost[b] = B.visited[i];
            at += B.per_block[i];
        }
    }
    std::vector<int> order;
    longest_first(B.cost, order);
    B.blocks.resize(order.size());
    for (size_t k = 0; k < order.size(); ++k) B.blocks[k] = B.by_leaf[order[k]];
    if (!sym || !fits) return;
    // per thread the slots its leaves' blocks fill for each leaf, then their places
    B.next.assign((size_t)T * n, 0);
    parallel_slices(T, n, [&](int t, int i0, int i1) {
        int *c = B.next.data() + (size_t)t * n;
        for (int i = i0; i < i1; ++i)
            for (int e = pl.near_ptr[i]; e < pl.near_ptr[i + 1]; ++e)
                if (pl.nearl[e] > leaf0 + i) c[pl.nearl[e] - leaf0] += count(leaf0 + i);
    });
    int run = 0;
    for (int q = 0; q < n; ++q) {
        for (int t = 0; t < T; ++t) {
            int &c = B.next[(size_t)t * n + q];
            run += std::exchange(c, run);
        }
        B.in_ptr[q + 1] = run;
    }
    B.in.resize((size_t)run);
    parallel_slices(T, n, [&](int t, int i0, int i1) {
        int *c = B.next.data() + (size_t)t * n;
        for (int b = B.first[i0]; b < B.first[i1]; ++b) {
            const int leaf = B.by_leaf[b].x;
            int at = B.by_leaf[b].w;
            for (int e = pl.near_ptr[leaf - leaf0]; e < pl.near_ptr[leaf - leaf0 + 1]; ++e) {
                const int q = pl.nearl[e];
                if (q <= leaf) continue;
                B.in[c[q - leaf0]++] = at;
                at += size(q);
            }
        }
    });
}

// Whether the near field sums both directions of a pair at once: by the steps of its
// wavefronts over all pairs of adjacent leaves.  A pair of tiles takes 64 steps of 88
// instructions both ways, however few blobs its tiles hold, and one way a step of 71
// instructions per source for each direction.
// Products of order 3 both ways and one way in FP32, us: leaves of 15 blobs in space 443
// and 310, of 34 605 and 553, of 49 626 and 628, of 98 in a layer above the wall 710 and 794,
// of 68 516 and 512, of 49 406 and 345.  (With double sums alike above the wall; in space
// one way still wins at leaves of 81, 1,567 and 1,301.)
static bool near_both_ways(const FmmPlan &pl) {
    const int leaf0 = pl.lvl[pl.L];
    const int T = step_threads((int64_t)pl.nearl.size(), kListStep);
    std::vector<int64_t> steps(2 * (size_t)T);
    parallel_slices(T, pl.nleaf, [&](int t, int i0, int i1) {
        int64_t both = 0, one = 0;
        for (int i = i0; i < i1; ++i) {
            const int2 r = pl.rng[leaf0 + i];
            const int64_t mc = r.y - r.x, tc = (mc + 63) / 64;
            for (int e = pl.near_ptr[i]; e < pl.near_ptr[i + 1]; ++e) {
                const int q = pl.nearl[e];
                if (q <= leaf0 + i) continue;
                const int64_t mq = pl.rng[q].y - pl.rng[q].x, tq = (mq + 63) / 64;
                both += 64 * tc * tq;
                one += tc * mq + tq * mc;
            }
        }
        steps[2 * (size_t)t] = both;
        steps[2 * (size_t)t + 1] = one;
    });
    int64_t both = 0, one = 0;
    for (int t = 0; t < T; ++t) {
        both += steps[2 * (size_t)t];
        one += steps[2 * (size_t)t + 1];
    }
    return 88 * both < 71 * one;
}

int fmm_build(FmmState &F, hipStream_t s, int N, const double *pos_dev, const float4 *hi,
              const float4 *lo, double a, int order, int levels, int leaf, int channels, bool wall,
              std::string *msg) {
    F.N = 0;
    F.ready = false;
    const int n = order > 0 ? order : kFmmDefaultOrder;
    if (n < 2 || n > kFmmMaxOrder || levels < 0 || leaf < 0 || N < 0) {
        *msg = "fast product: order must be 2..8, levels and leaf >= 0";
        return ARB_E_ARG;
    }
    F.n = n;
    F.P = n * n * n;
    ++F.version;
    if (N == 0) {
        F.ready = true;
        return 0;
    }
    if (!F.host) F.host = std::make_shared<FmmHostCache>();
    FmmHostCache &hc = *F.host;
    std::vector<double> hpage;  // pageable fallback when pinned memory is refused
    double *h = hc.positions(3 * (size_t)N);
    if (!h) {
        hpage.resize(3 * (size_t)N);
        h = hpage.data();
    }
    if (hipMemcpyAsync(h, pos_dev, 3 * (size_t)N * sizeof(double), hipMemcpyDeviceToHost, s) !=
            hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
        *msg = "fast product: copying positions failed";
        return ARB_E_DEVICE;
    }
    FmmPlan &pl = hc.plan;
    const int prc = fmm_plan(pl, hc.scratch, N, h, a, n, levels, leaf, msg);
    if (prc) return prc;
    // upload
    const int P = F.P, ncell = pl.ncell;
    auto up = [&](DevBuf &b, const void *src, size_t bytes) -> bool {
        if (b.ensure(std::max<size_t>(bytes, 16)) != hipSuccess) return false;
        return bytes == 0 ||
               hipMemcpyAsync(b.p, src, bytes, hipMemcpyHostToDevice, s) == hipSuccess;
    };
    bool ok = up(F.perm, pl.perm.data(), pl.perm.size() * sizeof(int)) &&
              up(F.cc, pl.cc.data(), pl.cc.size() * sizeof(int4)) &&
              up(F.rng, pl.rng.data(), pl.rng.size() * sizeof(int2)) &&
              up(F.parent, pl.parent.data(), pl.parent.size() * sizeof(int)) &&
              up(F.kids, pl.kids.data(), pl.kids.size() * sizeof(int2)) &&
              up(F.near_ptr, pl.near_ptr.data(), pl.near_ptr.size() * sizeof(int)) &&
              up(F.nearl, pl.nearl.data(), pl.nearl.size() * sizeof(int)) &&
              up(F.work, pl.work.data(), pl.work.size() * sizeof(int2)) &&
              up(F.tab, pl.tab.data(), pl.tab.size() * sizeof(float)) &&
              F.shi.ensure((size_t)N * sizeof(float4)) == hipSuccess &&
              F.slo.ensure((size_t)N * sizeof(float4)) == hipSuccess &&
              F.slam.ensure((size_t)N * sizeof(double4)) == hipSuccess &&
              F.qhat.ensure((size_t)ncell * P * sizeof(double4)) == hipSuccess &&
              F.v.ensure((size_t)ncell * P * 3 * sizeof(double)) == hipSuccess &&
              (channels < 2 ||
               (F.slam2.ensure((size_t)N * sizeof(double4)) == hipSuccess &&
                F.qhat2.ensure((size_t)ncell * P * sizeof(double4)) == hipSuccess &&
                F.v2.ensure((size_t)ncell * P * 3 * sizeof(double)) == hipSuccess));
    // M2L's batches: 32 columns, 16 with the torque channel; slots of a chunk bounded
    M2LGroups &mg = hc.m2l;
    const int64_t slot_doubles = 3 * (int64_t)P * channels;
    group_m2l(pl, wall, channels == 2 ? 16 : 32,
              std::max<int64_t>(1, kFmmSlotBytes / (slot_doubles * 8)), mg);
    ok = ok && up(F.sp_ptr, mg.sp_ptr.data(), mg.sp_ptr.size() * sizeof(int)) &&
         up(F.sp, mg.sp.data(), mg.sp.size() * sizeof(int)) &&
         up(F.sp_order, mg.sp_order.data(), mg.sp_order.size() * sizeof(int)) &&
         up(F.slot_ptr, mg.slot_ptr.data(), mg.slot_ptr.size() * sizeof(int)) &&
         up(F.cols, mg.cols.data(), mg.cols.size() * sizeof(int2)) &&
         up(F.batches, mg.batches.data(), mg.batches.size() * sizeof(FmmBatch)) &&
         F.slots.ensure((size_t)mg.max_slots * slot_doubles * sizeof(double)) == hipSuccess;
    const int nc_m2l = pl.L >= 2 ? pl.lvl[pl.L + 1] - pl.lvl[2] : 0;
    const int splits = nc_m2l > 0 ? m2l_splits(nc_m2l) : 1;
    ok = ok && (splits == 1 ||
                F.vsplit.ensure((size_t)nc_m2l * splits * P * 3 * channels * sizeof(double)) ==
                    hipSuccess);
    ok = ok && F.own.ensure((size_t)N * 3 * channels * sizeof(double)) == hipSuccess;
    // near field: both directions of a pair at once for the 3-component tensor; one way,
    // without slots, with torques, where leaves are nearly empty, or when the slots would
    // outgrow kFmmNearSlots or the memory that the rest leaves
    NearBlocks &nb = hc.near;
    bool near_sym = channels == 1 && near_both_ways(pl);
    near_blocks(pl, near_sym, nb);
    if (near_sym && ok &&
        (nb.slots > kFmmNearSlots ||
         F.near_slots.ensure((size_t)nb.slots * 3 * sizeof(double)) != hipSuccess)) {
        (void)hipGetLastError();
        near_sym = false;
        near_blocks(pl, false, nb);
    }
    ok = ok && up(F.blocks, nb.blocks.data(), nb.blocks.size() * sizeof(int4)) &&
         up(F.in_ptr, nb.in_ptr.data(), nb.in_ptr.size() * sizeof(int)) &&
         up(F.in, nb.in.data(), nb.in.size() * sizeof(int));
    if (!ok) {
        *msg = "fast product: device allocation or copy failed";
        return ARB_E_DEVICE;
    }
    fmm_sort_pos_kernel<<<(N + 255) / 256, 256, 0, s>>>(N, F.perm.as<int>(), hi, lo,
                                                         F.shi.as<float4>(), F.slo.as<float4>());
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
        *msg = "fast product: device error while sorting positions";
        return ARB_E_DEVICE;
    }
    F.L = pl.L;
    F.lvl = pl.lvl;
    F.chunks = mg.chunks;
    F.splits = splits;
    F.o[0] = pl.o[0] / a;
    F.o[1] = pl.o[1] / a;
    F.o[2] = pl.o[2] / a;
    F.S = pl.S / a;
    F.ncell = pl.ncell;
    F.nleaf = pl.nleaf;
    F.nwork = (int)pl.work.size();
    F.n_blocks = (int)nb.blocks.size();
    F.near_sym = near_sym;
    F.n_il = (int64_t)pl.il.size();
    F.n_m2l_pairs = pl.n_m2l_pairs;
    F.n_near_pairs = pl.n_near_pairs;
    F.channels = channels;
    F.N = N;
    F.ready = true;
    return 0;
}

namespace {

template <bool WALL, class A>
void fmm_run(const FmmState &F, hipStream_t s, const double *lam, double *partial) {
    const int N = F.N, L = F.L, P = F.P;
    const Geo g{F.o[0], F.o[1], F.o[2], F.S, F.n, P};
    const int B = round_up(P, kWave);
    const float *tab = F.tab.as<float>();
    Vec4<A> *slam = F.slam.as<Vec4<A>>(), *qhat = F.qhat.as<Vec4<A>>();
    fmm_gather_lam_kernel<A><<<(N + 255) / 256, 256, 0, s>>>(N, F.perm.as<int>(), lam, slam);
    if (L >= 2) {
        with_order(F.n, [&](auto o) {
            constexpr int n = decltype(o)::value;
            fmm_p2m_kernel<A, n><<<F.lvl[L + 1] - F.lvl[L], P2MShape<n>::T, 0, s>>>(
                g, tab, F.cc.as<int4>(), F.rng.as<int2>(), F.lvl[L], F.shi.as<float4>(),
                F.slo.as<float4>(), slam, qhat);
            for (int l = L - 1; l >= 2; --l)
                fmm_m2m_kernel<A, n><<<F.lvl[l + 1] - F.lvl[l], M2MShape<A, n>::T, 0, s>>>(
                    g, tab, F.cc.as<int4>(), F.kids.as<int2>(), F.lvl[l], qhat);
        });
        fmm_m2l(F, s, 1, WALL, std::is_same_v<A, double>);
        with_order(F.n, [&](auto o) {
            for (int l = 3; l <= L; ++l)
                fmm_l2l_kernel<decltype(o)::value><<<F.lvl[l + 1] - F.lvl[l], B, 0, s>>>(
                    g, tab, F.cc.as<int4>(), F.parent.as<int>(), F.lvl[l], F.v.as<double>());
        });
    }
    fmm_near(F, s, 1, WALL, std::is_same_v<A, double>, partial);
}

}  // namespace

void fmm_apply(const FmmState &F, hipStream_t s, bool wall, bool fp64, const double *lam,
               double *partial) {
    if (F.N == 0) return;
    if (wall)
        fp64 ? fmm_run<true, double>(F, s, lam, partial) : fmm_run<true, float>(F, s, lam, partial);
    else
        fp64 ? fmm_run<false, double>(F, s, lam, partial)
             : fmm_run<false, float>(F, s, lam, partial);
}

}  // namespace arb

namespace arb {

namespace {

template <class A>
void fmm_run6(const FmmState &F, hipStream_t s, const double *x6, double inv_a, double *partial) {
    const int M = F.N, L = F.L, P = F.P;
    const Geo g{F.o[0], F.o[1], F.o[2], F.S, F.n, P};
    const int B = round_up(P, kWave);
    const float *tab = F.tab.as<float>();
    Vec4<A> *sf = F.slam.as<Vec4<A>>(), *st = F.slam2.as<Vec4<A>>();
    Vec4<A> *qf = F.qhat.as<Vec4<A>>(), *qt = F.qhat2.as<Vec4<A>>();
    double *vu = F.v.as<double>(), *vw = F.v2.as<double>();
    fmm_gather6_kernel<A><<<(M + 255) / 256, 256, 0, s>>>(M, F.perm.as<int>(), x6, inv_a, sf, st);
    if (L >= 2) {
        with_order(F.n, [&](auto o) {
            constexpr int n = decltype(o)::value;
            for (int ch = 0; ch < 2; ++ch)
                fmm_p2m_kernel<A, n><<<F.lvl[L + 1] - F.lvl[L], P2MShape<n>::T, 0, s>>>(
                    g, tab, F.cc.as<int4>(), F.rng.as<int2>(), F.lvl[L], F.shi.as<float4>(),
                    F.slo.as<float4>(), ch ? st : sf, ch ? qt : qf);
            for (int l = L - 1; l >= 2; --l)
                for (int ch = 0; ch < 2; ++ch)
                    fmm_m2m_kernel<A, n><<<F.lvl[l + 1] - F.lvl[l], M2MShape<A, n>::T, 0, s>>>(
                        g, tab, F.cc.as<int4>(), F.kids.as<int2>(), F.lvl[l], ch ? qt : qf);
        });
        fmm_m2l(F, s, 2, false, std::is_same_v<A, double>);
        with_order(F.n, [&](auto o) {
            for (int l = 3; l <= L; ++l)
                for (int ch = 0; ch < 2; ++ch)
                    fmm_l2l_kernel<decltype(o)::value><<<F.lvl[l + 1] - F.lvl[l], B, 0, s>>>(
                        g, tab, F.cc.as<int4>(), F.parent.as<int>(), F.lvl[l], ch ? vw : vu);
        });
    }
    fmm_near(F, s, 2, false, std::is_same_v<A, double>, partial);
}

}  // namespace

void fmm_apply6(const FmmState &F, hipStream_t s, bool fp64, const double *x6, double inv_a,
                double *partial) {
    if (F.N == 0) return;
    fp64 ? fmm_run6<double>(F, s, x6, inv_a, partial) : fmm_run6<float>(F, s, x6, inv_a, partial);
}

}  // namespace arb

int arb_fmm_plan(int N, const double *pos, double a, int order, int levels, int leaf,
                 arb_fmm_stats *out) {
    using namespace arb;
    if (N < 0 || (N > 0 && !pos) || !(a > 0.0) || !out ||
        (order != 0 && (order < 2 || order > kFmmMaxOrder)) || levels < 0 ||
        levels > kFmmMaxLevel || leaf < 0)
        return ARB_E_ARG;
    const int n = order > 0 ? order : kFmmDefaultOrder;
    *out = arb_fmm_stats{};
    out->order = n;
    if (N == 0) return ARB_OK;
    const auto t0 = std::chrono::steady_clock::now();
    // one scratch kept for the process (plans on several threads at once: the
    // others take scratch of their own for the call)
    static std::mutex mu;
    static PlanScratch kept;
    FmmPlan pl;
    int rc = 0;
    try {
        std::string msg;
        std::unique_lock<std::mutex> lk(mu, std::try_to_lock);
        if (lk.owns_lock()) {
            rc = fmm_plan(pl, kept, N, pos, a, n, levels, leaf, &msg);
        } else {
            PlanScratch own;
            rc = fmm_plan(pl, own, N, pos, a, n, levels, leaf, &msg);
        }
    } catch (...) {  // host allocation or worker-thread failure: no exception crosses the ABI
        return ARB_E_HOST;
    }
    if (rc) return rc;
    out->levels = pl.L;
    out->cells = pl.ncell;
    out->leaves = pl.nleaf;
    out->near_pairs = pl.n_near_pairs;
    out->interactions = (long long)pl.il.size();
    out->m2l_pairs = pl.n_m2l_pairs;
    out->build_ms =
        std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    uint64_t h = 0xcbf29ce484222325ull;
    fnv1a(h, pl.perm);
    fnv1a(h, pl.lvl);
    fnv1a(h, pl.parent);
    fnv1a(h, pl.il_ptr);
    fnv1a(h, pl.il);
    fnv1a(h, pl.near_ptr);
    fnv1a(h, pl.nearl);
    fnv1a(h, pl.cc);
    fnv1a(h, pl.rng);
    fnv1a(h, pl.kids);
    fnv1a(h, pl.work);
    fnv1a(h, pl.tab);
    out->plan_hash = (unsigned long long)h;
    return ARB_OK;
}
