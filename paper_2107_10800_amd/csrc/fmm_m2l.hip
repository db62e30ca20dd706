// M2L of the fast product (fmm.hip): v^c_k = sum over the interaction list of c of
// the pair tensor between c's proxies and the listed cell's, or its blobs when it
// holds fewer blobs than proxies.  Two kernels share the work:
//
//  * listed cells with their proxies ("dense" entries).  The tensor between two
//    proxy grids depends only on the level, the cells' integer offset and, above
//    the wall, the target cell's height, so the entries with the same key are one
//    matrix (3 n^3 x 3 n^3, 6 n^3 with torques) against many columns: a
//    contraction, done on the matrix cores.  The host groups the entries by key
//    into batches of at most 16 CT columns; a wavefront holds 16 target proxies
//    against the batch's columns.  At each step every lane evaluates the tensor
//    of one pair (proxy l mod 16 of the tile, source proxy 4 st + l / 16) once, and
//    its 9 entries (30 with torques) are the A operands of one matrix instruction
//    each per 16 columns, in the instruction's own lane layout, so nothing is
//    exchanged between lanes.  Each column's result goes to a slot of its own, and
//    fmm_m2l_sum_kernel adds a cell's slots in list order: no atomics, products
//    repeat bit for bit.
//    Bound by the matrix cores: 9 instructions of 1,024 FMAs (30 with torques) per 64
//    pairs and 16 columns, against about 60 VALU instructions to form the operands,
//    shared by up to 32 columns.  8,192 bacteria (94,550 dense entries, n = 6): 1.03 ms
//    = 77 TFLOP/s; pair by pair on the VALU these entries took about 6.8 ms.  Diatom
//    colonies, double sums: 0.90 ms (2.5 ms before); 4,096 shells with torques 1.86 ms
//    (4.1 ms).
//  * sparse entries (P2L): the blobs of a cell's sparse listed cells, strung
//    together and dealt evenly to lane groups of n^2 lanes, each lane holding the
//    KZ target proxies of one (x, y), so that the differences in the plane are
//    formed once per blob and lane.  VALU-bound: 1.87 ms for 1.48e9 pairs of the
//    bacteria (7.9e11 pairs/s).
//
// At order 2 (8 proxies: half a matrix tile, and results as many as weights) every listed
// cell is strung, the dense ones with their proxies, and a cell takes one wavefront: 150,000
// blobs in clusters 212 us, in a thin layer 35, against 391 and 81 with batches (and 311 and
// 47 before there were any).
//
// Every pair is well separated (r > 2a: cells at least a side apart, side >= 2a, and
// proxies inside their cells), so the overlap branch is left out.
#include <algorithm>

#include "fmm_device.h"

namespace arb {

namespace {

typedef float accf __attribute__((ext_vector_type(4)));
typedef double accd __attribute__((ext_vector_type(4)));
template <class A>
using Acc = std::conditional_t<std::is_same_v<A, float>, accf, accd>;

__device__ __forceinline__ accf mfma16(float a, float b, accf c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ accd mfma16(double a, double b, accd c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// row of accumulator element e in lane l (column l mod 16)
__device__ __forceinline__ int acc_row(int l, int e, float) { return 4 * (l >> 4) + e; }
__device__ __forceinline__ int acc_row(int l, int e, double) { return 4 * e + (l >> 4); }

// wall pair coefficients of a well-separated pair, float
__device__ __forceinline__ PairCoef<float> wall_coef(float dx, float dy, float dz, float zi,
                                                     const TargetZ<float> &zs, float zj,
                                                     float &Rz) {
    constexpr CoefF cf = kUnitCoefF;
    const float dxy2 = fmaf(dx, dx, dy * dy);
    const float rinv = rsq_f32(fmaf(dz, dz, dxy2));
    Rz = zi + zj;
    const float h2 = 2.f * zj;
    return wall_pair_coef<float, CoefF, false>(0.f, rinv, dxy2, zs, zj, h2, -(h2 * h2), Rz,
                                               rsq_f32(fmaf(Rz, Rz, dxy2)), cf);
}

// the 3 x 3 tensor (row-major) of a well-separated pair: coefficients in float,
// entries in A
template <bool WALL, class A>
__device__ __forceinline__ void entries3(float dx, float dy, float dz, float zi,
                                         const TargetZ<float> &zs, float zj, A *m) {
    if constexpr (WALL) {
        float Rzf;
        const PairCoef<float> w = wall_coef(dx, dy, dz, zi, zs, zj, Rzf);
        const A x = (A)dx, y = (A)dy, z = (A)dz, R = (A)Rzf, b = (A)w.b, c2 = (A)w.c2;
        const A px = (c2 + b) * x, py = (c2 + b) * y;
        const A q = fma(c2, z, b * R);
        const A qc = q + (A)w.c, qd = q + (A)w.d;
        m[0] = fma(px, x, (A)w.cA);
        m[1] = m[3] = px * y;
        m[4] = fma(py, y, (A)w.cA);
        m[2] = x * qc;
        m[5] = y * qc;
        m[6] = x * qd;
        m[7] = y * qd;
        m[8] = fma(R, fma(b, R, (A)w.c + (A)w.d), fma(c2 * z, z, (A)w.cAe));
    } else {
        constexpr CoefF cf = kUnitCoefF;
        const float rinv = rsq_f32(fmaf(dz, dz, fmaf(dx, dx, dy * dy)));
        const float rinv2 = rinv * rinv, rinv3 = rinv * rinv2;
        const A c1 = (A)fmaf(cf.k1, rinv3, rinv), c2 = (A)fmaf(-cf.k2, rinv3 * rinv2, rinv3);
        const A x = (A)dx, y = (A)dy, z = (A)dz;
        const A px = c2 * x, py = c2 * y;
        m[0] = fma(px, x, c1);
        m[4] = fma(py, y, c1);
        m[8] = fma(c2 * z, z, c1);
        m[1] = m[3] = px * y;
        m[2] = m[6] = px * z;
        m[5] = m[7] = py * z;
    }
}

// generalised tensor of a well-separated pair: translation and rotation blocks
// (symmetric: xx, xy, xz, yy, yz, zz) and the couplings c_r r
template <class A>
__device__ __forceinline__ void entries6(float dx, float dy, float dz, A *tr, A *ro, A *e) {
    constexpr RotCoef<float> c = kUnitRotCoef;
    const float rinv = rsq_f32(fmaf(dz, dz, fmaf(dx, dx, dy * dy)));
    const float rinv2 = rinv * rinv, rinv3 = rinv * rinv2, rinv5 = rinv3 * rinv2;
    const A c1 = (A)fmaf(c.k1, rinv3, rinv), c2 = (A)fmaf(-c.k2, rinv5, rinv3);
    const A cr = (A)rinv3, d1 = (A)(-0.5f * rinv3), d2 = (A)(1.5f * rinv5);
    const A x = (A)dx, y = (A)dy, z = (A)dz;
    e[0] = cr * x;
    e[1] = cr * y;
    e[2] = cr * z;
    const A px = c2 * x, py = c2 * y, sx = d2 * x, sy = d2 * y;
    tr[0] = fma(px, x, c1);
    tr[1] = px * y;
    tr[2] = px * z;
    tr[3] = fma(py, y, c1);
    tr[4] = py * z;
    tr[5] = fma(c2 * z, z, c1);
    ro[0] = fma(sx, x, d1);
    ro[1] = sx * y;
    ro[2] = sx * z;
    ro[3] = fma(sy, y, d1);
    ro[4] = sy * z;
    ro[5] = fma(d2 * z, z, d1);
}

// One wavefront: a tile of 16 target proxies against a batch's columns, independent of
// the others of its workgroup (no barrier: with the weights staged in LDS by the
// workgroup, barriers and the uneven share of tiles per SIMD left the matrix cores
// idle half the time).  The weights are read straight in the B operand's layout,
// 4 consecutive proxies of 16 cells at a time (64-byte runs), the next step's in
// flight while this one's are used; the tiles of a batch run side by side and share
// them in the caches.  Float sums run over kFmmRun sources and are promoted to
// double, as in the direct sums.
constexpr int kDenseWaves = 4;

template <bool WALL, int CH, class A, int CT, int NO>
__global__ __launch_bounds__(64 * kDenseWaves) __attribute__((amdgpu_waves_per_eu(4)))
void fmm_m2l_dense_kernel(
    Geo g, const float *__restrict__ tabg, const FmmBatch *__restrict__ batches, int tasks,
    int items, const int2 *__restrict__ cols, const Vec4<A> *__restrict__ qf,
    const Vec4<A> *__restrict__ qt, double *__restrict__ slots) {
    constexpr int P = NO * NO * NO, tiles = (P + 15) / 16, NB = 3 * CH;
    constexpr int steps = (P + 3) / 4, run = kFmmRun / 4;
    constexpr bool F32 = std::is_same_v<A, float>;
    const int item = xcd_item(items);
    if (item < 0) return;
    __shared__ float tab[kTabSize];
    __shared__ float4 s_off[kDenseWaves][P];
    load_tab(tabg, tab);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int task = item * kDenseWaves + wv;
    if (task >= tasks) return;  // the whole wavefront; no barrier follows
    const FmmBatch b = batches[task / tiles];
    const double side = ldexp(g.S, -b.level), w = 0.5 * side;
    float4 *off = s_off[wv];
    for (int m = lane; m < P; m += 64)
        off[m] = make_float4((float)(w * tab[kTabNode + m / (NO * NO)]),
                             (float)(w * tab[kTabNode + (m / NO) % NO]),
                             (float)(w * tab[kTabNode + m % NO]), 0.f);
    __builtin_amdgcn_wave_barrier();  // LDS of one wavefront completes in order
    // this lane's target proxy (A operand row l mod 16 of the tile)
    const int tile = task % tiles;
    const int kq = lane >> 4, cl = lane & 15;
    const int k = min(tile * 16 + cl, P - 1);
    const float4 ok4 = off[k];
    const float ax = (float)((double)b.dx * side) + ok4.x;
    const float ay = (float)((double)b.dy * side) + ok4.y;
    const float az = (float)((double)b.dz * side) + ok4.z;
    const float zi = (float)(centre(g.oz, side, b.tz) + w * (double)tab[kTabNode + k % NO]);
    const TargetZ<float> zs = target_z(zi);
    const float zc = (float)centre(g.oz, side, b.tz - b.dz);
    const bool two = CT > 1 && b.count > 16;
    // a column past the batch's last reads the last one's weights (its results are
    // not stored)
    const Vec4<A> *src[CT], *srt[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const size_t q = (size_t)cols[b.first + min(16 * ct + cl, b.count - 1)].x * P;
        src[ct] = qf + q;
        srt[ct] = CH == 2 ? qt + q : nullptr;
    }
    Vec4<A> bf[CT], bt[CH == 2 ? CT : 1];
    auto fetch = [&](int st) {
        const int m = 4 * st + kq;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            if (ct > 0 && !two) break;
            bf[ct] = src[ct][min(m, P - 1)];
            if constexpr (CH == 2) bt[ct] = srt[ct][min(m, P - 1)];
        }
        if (P % 4 != 0 && m >= P) {  // no source proxy: zero weights
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                bf[ct] = vec4<A>(0, 0, 0);
                if constexpr (CH == 2) bt[ct] = vec4<A>(0, 0, 0);
            }
        }
    };
    Acc<A> acc[CT][NB] = {};
    double sum[F32 ? CT : 1][F32 ? NB : 1][4] = {};
    fetch(0);
#pragma unroll 1
    for (int st0 = 0; st0 < steps; st0 += run) {
#pragma unroll 1
        for (int st = st0; st < min(st0 + run, steps); ++st) {
            Vec4<A> f[CT], t[CH == 2 ? CT : 1];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                f[ct] = bf[ct];
                if constexpr (CH == 2) t[ct] = bt[ct];
            }
            if (st + 1 < steps) fetch(st + 1);
            const float4 o = off[min(4 * st + kq, P - 1)];
            const float dx = ax - o.x, dy = ay - o.y, dz = az - o.z;
            if constexpr (CH == 1) {
                A m[9];
                entries3<WALL, A>(dx, dy, dz, zi, zs, zc + o.z, m);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    if (ct > 0 && !two) break;
                    const A bv[3] = {f[ct].x, f[ct].y, f[ct].z};
#pragma unroll
                    for (int j = 0; j < 3; ++j)
#pragma unroll
                        for (int i = 0; i < 3; ++i)
                            acc[ct][i] = mfma16(m[3 * i + j], bv[j], acc[ct][i]);
                }
            } else {
                A tr[6], ro[6], e[3];
                entries6<A>(dx, dy, dz, tr, ro, e);
                constexpr int sy[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
                const A bv[6] = {f[0].x, f[0].y, f[0].z, t[0].x, t[0].y, t[0].z};
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        acc[0][i] = mfma16(tr[sy[i][j]], bv[j], acc[0][i]);
                        acc[0][3 + i] = mfma16(ro[sy[i][j]], bv[3 + j], acc[0][3 + i]);
                    }
                // u += t x e, w += f x e:  (v x e)_i = v_{i+1} e_{i+2} - v_{i+2} e_{i+1}
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
                    acc[0][i] = mfma16(e[i2], bv[3 + i1], acc[0][i]);
                    acc[0][3 + i] = mfma16(e[i2], bv[i1], acc[0][3 + i]);
                    acc[0][i] = mfma16(-e[i1], bv[3 + i2], acc[0][i]);
                    acc[0][3 + i] = mfma16(-e[i1], bv[i2], acc[0][3 + i]);
                }
            }
        }
        if constexpr (F32) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int i = 0; i < NB; ++i) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) sum[ct][i][q] += (double)acc[ct][i][q];
                    acc[ct][i] = Acc<A>{};
                }
        }
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int col = 16 * ct + cl;
        if (col >= b.count) continue;
        double *o = slots + (size_t)cols[b.first + col].y * (3 * CH * P);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = tile * 16 + acc_row(lane, q, A(0));
            if (row >= P) continue;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                double v;
                if constexpr (F32)
                    v = sum[ct][i][q];
                else
                    v = acc[ct][i][q];
                o[(size_t)(i / 3) * 3 * P + 3 * row + i % 3] = v;
            }
        }
    }
}

// shape of the sparse kernel for order n: KZ proxies of one (x, y) per lane, n^3 / KZ
// lanes per group, as many groups as fill the workgroup's wavefronts, at most
// kFmmRun staged blobs per group.  KZ = n, but half of it at n = 6 and 8: the KZ
// pairs are independent chains, and the 128 registers of 4 wavefronts per SIMD hold
// three of them side by side (2.05 ms on the bacteria; 1.87 with the longest lists
// first) but not six, which the compiler then runs one after the other (2.60 ms; so do 5
// or 6 wavefronts per SIMD: 2.47 ms).  Workgroups are whole multiples of 4 wavefronts: 6
// load two of the four SIMDs twice as much (3.30 ms).  (Order 2, with little to do per
// cell: one wavefront; 150,000 blobs in clusters and strays with 4 754 us, with 1 428.)
template <int NO>
struct SparseShape {
    static constexpr int P = NO * NO * NO, KZ = NO == 6 || NO == 8 ? NO / 2 : NO;
    static constexpr int lanes = P / KZ;
    static constexpr int block = NO == 6 ? 512 : (NO == 2 ? 64 : 256), groups = block / lanes;
    static constexpr int chunk = groups * kFmmRun < block ? groups * kFmmRun : block;
    // groups whose sums are joined at a time
    static constexpr int join = NO == 2 ? 16 : (NO == 3 ? 14 : (NO == 4 ? 8 : 1));
    // order 2: dense listed cells are strung too, with their proxies
    static constexpr bool all = NO == kFmmStrungOrder;
};
constexpr int kMaxListed = 189;  // cells of an interaction list (6^3 - 3^3)

// the blobs of the sparse listed cells of one target cell; a cell's blobs may be
// split over `splits` consecutive items, each with a place of its own in vpart
template <bool WALL, int CH, class A, int NO>
__global__ __launch_bounds__(SparseShape<NO>::block)
__attribute__((amdgpu_waves_per_eu(CH == 1 ? 4 : 3)))
void fmm_p2l_kernel(
    Geo g, const float *__restrict__ tabg, const int4 *__restrict__ cc,
    const int *__restrict__ sp_ptr, const int *__restrict__ sp, const int *__restrict__ order,
    int cell0, int items, int splits,
    const int2 *__restrict__ rng, const float4 *__restrict__ shi, const float4 *__restrict__ slo,
    const Vec4<A> *__restrict__ sf, const Vec4<A> *__restrict__ st,
    const Vec4<A> *__restrict__ qf, const Vec4<A> *__restrict__ qt, double *__restrict__ vu,
    double *__restrict__ vw, double *__restrict__ vpart) {
    using Sh = SparseShape<NO>;
    constexpr int P = Sh::P, C = Sh::chunk, NB = 3 * CH, KZ = Sh::KZ, block = Sh::block;
    constexpr bool F32 = std::is_same_v<A, float>;
    const int item = xcd_item(items);
    if (item < 0) return;
    __shared__ float tab[kTabSize];
    __shared__ int s_start[kMaxListed], s_pre[kMaxListed + 1], s_wave[block / kWave];
    __shared__ float4 s_off[C];
    __shared__ Vec4<A> s_f[C], s_t[CH == 2 ? C : 1];
    __shared__ double s_sum[NB][P];
    __shared__ unsigned char s_id[Sh::all ? C : 1];
    load_tab(tabg, tab);
    const int tid = threadIdx.x;
    const int ci = order[item / splits], part = item % splits, c = cell0 + ci;
    const int4 ct = cc[c];
    const double side = ldexp(g.S, -ct.w), w = 0.5 * side;
    const int e0 = sp_ptr[ci], ne = sp_ptr[ci + 1] - e0;
    for (int i = tid; i < NB * P; i += block) s_sum[i / P][i % P] = 0.0;
    // prefix sums of the listed cells' source counts, an entry per thread (a wavefront alone
    // in turns)
    static_assert(block == kWave || block >= kMaxListed);
    if (tid == 0) s_pre[0] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < ne; i0 += block) {
        const int i = i0 + tid;
        int v = 0;
        if (i < ne) {
            const int q = sp[e0 + i];
            const int2 r = rng[q];
            s_start[i] = r.x;
            v = r.y - r.x;
            if (Sh::all && v >= P) {  // proxies: ~cell in place of the first blob
                s_start[i] = ~q;
                v = P;
            }
        }
        for (int off = 1; off < kWave; off <<= 1) {
            const int u = __shfl_up(v, off);
            if ((tid & 63) >= off) v += u;
        }
        if constexpr (block > kWave) {
            if ((tid & 63) == 63) s_wave[tid >> 6] = v;
            __syncthreads();
            for (int q = 0; q < (tid >> 6); ++q) v += s_wave[q];
        } else {
            v += s_pre[i0];
        }
        if (i < ne) s_pre[i + 1] = v;
        __syncthreads();
    }
    const int total = s_pre[ne];
    if (total == 0 && splits == 1) {
        for (int i = tid; i < 3 * P; i += block) {
            vu[(size_t)c * 3 * P + i] = 0.0;
            if constexpr (CH == 2) vw[(size_t)c * 3 * P + i] = 0.0;
        }
        return;
    }
    const int j1 = (int)((int64_t)total * (part + 1) / splits);
    // proxies k0 .. k0 + KZ - 1 of this lane: one (x, y), consecutive z
    const int grp = tid / Sh::lanes, k0 = tid % Sh::lanes * KZ, kxy = k0 / NO, kz0 = k0 % NO;
    const bool act = grp < Sh::groups;
    const float okx = (float)(w * tab[kTabNode + kxy / NO]),
                oky = (float)(w * tab[kTabNode + kxy % NO]);
    const double cx = centre(g.ox, side, ct.x), cy = centre(g.oy, side, ct.y),
                 cz = centre(g.oz, side, ct.z);
    const F2 hx = split(cx), hy = split(cy), hz = split(cz);
    float okz[KZ], zi[KZ];
#pragma unroll
    for (int kz = 0; kz < KZ; ++kz) {
        okz[kz] = (float)(w * tab[kTabNode + kz0 + kz]);
        zi[kz] = (float)(cz + w * (double)tab[kTabNode + kz0 + kz]);
    }
    // double sums: float runs are promoted after each chunk
    A run[KZ][NB] = {};
    double sum[F32 ? KZ : 1][F32 ? NB : 1] = {};
    for (int j0 = (int)((int64_t)total * part / splits); j0 < j1; j0 += C) {
        const int cnt = min(C, j1 - j0);
        __syncthreads();
        if constexpr (Sh::all) {  // at most P = 8 sources a cell: each marks its own
            for (int i = tid; i < ne; i += block)
                for (int k = max(s_pre[i], j0); k < min(s_pre[i + 1], j0 + cnt); ++k)
                    s_id[k - j0] = (unsigned char)i;
            __syncthreads();
        }
        if (tid < cnt) {
            // the listed cell that holds blob j0 + tid of the string
            int lo = 0;
            if constexpr (Sh::all) {
                lo = s_id[tid];
            } else {
                int up = ne;
                while (up - lo > 1) {
                    const int mid = (lo + up) >> 1;
                    if (s_pre[mid] <= j0 + tid)
                        lo = mid;
                    else
                        up = mid;
                }
            }
            const int k = j0 + tid - s_pre[lo], first = s_start[lo];
            if (Sh::all && first < 0) {
                const int q = ~first;
                const int4 cs = cc[q];
                const float oz = (float)(w * tab[kTabNode + k % NO]);
                s_off[tid] = make_float4(
                    (float)((double)(cs.x - ct.x) * side) + (float)(w * tab[kTabNode + k / (NO * NO)]),
                    (float)((double)(cs.y - ct.y) * side) + (float)(w * tab[kTabNode + (k / NO) % NO]),
                    (float)((double)(cs.z - ct.z) * side) + oz,
                    (float)centre(g.oz, side, cs.z) + oz);
                s_f[tid] = qf[(size_t)q * P + k];
                if constexpr (CH == 2) s_t[tid] = qt[(size_t)q * P + k];
            } else {
                const int j = first + k;
                const float4 h = shi[j], l = slo[j];
                // offset from the target cell's centre, and the blob's height
                s_off[tid] = make_float4((h.x - hx.h) + (l.x - hx.l), (h.y - hy.h) + (l.y - hy.l),
                                         (h.z - hz.h) + (l.z - hz.l), h.z + l.z);
                s_f[tid] = sf[j];
                if constexpr (CH == 2) s_t[tid] = st[j];
            }
        }
        __syncthreads();
        if (!act) continue;
#pragma unroll 1
        for (int s = grp; s < cnt; s += Sh::groups) {
            const float4 o = s_off[s];
            const Vec4<A> F = s_f[s];
            const float dx = okx - o.x, dy = oky - o.y;
            if constexpr (CH == 1) {
#pragma unroll
                for (int kz = 0; kz < KZ; ++kz) {
                    const float dz = okz[kz] - o.z;
                    if constexpr (WALL) {
                        float Rz;
                        const PairCoef<float> pc =
                            wall_coef(dx, dy, dz, zi[kz], target_z(zi[kz]), o.w, Rz);
                        const PairCoef<A> pa{(A)pc.cA, (A)pc.cAe, (A)pc.c2, (A)pc.b,
                                             (A)pc.c,  (A)pc.d,   (A)pc.e,  (A)pc.h2};
                        wall_pair_apply<A>(pa, pa.c, pa.d, (A)dx, (A)dy, (A)dz, (A)Rz, F.x, F.y,
                                           F.z, run[kz][0], run[kz][1], run[kz][2]);
                    } else {
                        constexpr CoefF cf = kUnitCoefF;
                        const float rinv = rsq_f32(fmaf(dz, dz, fmaf(dx, dx, dy * dy)));
                        const float rinv2 = rinv * rinv, rinv3 = rinv * rinv2;
                        const A c1 = (A)fmaf(cf.k1, rinv3, rinv);
                        const A c2 = (A)fmaf(-cf.k2, rinv3 * rinv2, rinv3);
                        const A t = c2 * fma((A)dx, F.x, fma((A)dy, F.y, (A)dz * F.z));
                        run[kz][0] = fma(c1, F.x, fma(t, (A)dx, run[kz][0]));
                        run[kz][1] = fma(c1, F.y, fma(t, (A)dy, run[kz][1]));
                        run[kz][2] = fma(c1, F.z, fma(t, (A)dz, run[kz][2]));
                    }
                }
            } else {
                const Vec4<A> Tq = s_t[s];
#pragma unroll
                for (int kz = 0; kz < KZ; ++kz) {
                    constexpr RotCoef<float> rc = kUnitRotCoef;
                    const float dz = okz[kz] - o.z;
                    const float rinv = rsq_f32(fmaf(dz, dz, fmaf(dx, dx, dy * dy)));
                    const float rinv2 = rinv * rinv, rinv3 = rinv * rinv2, rinv5 = rinv3 * rinv2;
                    const RotTerms<A> kt{(A)fmaf(rc.k1, rinv3, rinv), (A)fmaf(-rc.k2, rinv5, rinv3),
                                         (A)rinv3, (A)(-0.5f * rinv3), (A)(1.5f * rinv5)};
                    rot_one_way<A>(kt, (A)dx, (A)dy, (A)dz, F.x, F.y, F.z, Tq.x, Tq.y, Tq.z,
                                   run[kz]);
                }
            }
        }
        if constexpr (F32) {
#pragma unroll
            for (int kz = 0; kz < KZ; ++kz)
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    sum[kz][i] += (double)run[kz][i];
                    run[kz][i] = 0.f;
                }
        }
    }
    // the groups' sums, added in group order; those of the many small groups of low orders
    // through LDS, several at a time (a barrier per group: 945 us for order 3 on a slab of
    // 100,000 blobs in leaves of 2, 28 groups; now 827)
    if constexpr (Sh::join > 1) {
        __shared__ double s_join[Sh::join][NB * P];
        for (int g0 = 0; g0 < Sh::groups; g0 += Sh::join) {
            if (grp >= g0 && grp < min(g0 + Sh::join, Sh::groups)) {
#pragma unroll
                for (int kz = 0; kz < KZ; ++kz)
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        if constexpr (F32)
                            s_join[grp - g0][i * P + k0 + kz] = sum[kz][i];
                        else
                            s_join[grp - g0][i * P + k0 + kz] = run[kz][i];
                    }
            }
            __syncthreads();
            const int cnt = min(Sh::join, Sh::groups - g0);
            for (int i = tid; i < NB * P; i += block) {
                double t = s_sum[i / P][i % P];
                for (int q = 0; q < cnt; ++q) t += s_join[q][i];
                s_sum[i / P][i % P] = t;
            }
            __syncthreads();
        }
    } else {
        for (int gr = 0; gr < Sh::groups; ++gr) {
            if (grp == gr) {
#pragma unroll
                for (int kz = 0; kz < KZ; ++kz)
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        if constexpr (F32)
                            s_sum[i][k0 + kz] += sum[kz][i];
                        else
                            s_sum[i][k0 + kz] += run[kz][i];
                    }
            }
            __syncthreads();
        }
    }
    for (int i = tid; i < 3 * P; i += block) {
        if (splits == 1) {
            vu[(size_t)c * 3 * P + i] = s_sum[i % 3][i / 3];
            if constexpr (CH == 2) vw[(size_t)c * 3 * P + i] = s_sum[3 + i % 3][i / 3];
        } else {
            double *o = vpart + ((size_t)ci * splits + part) * NB * P + i;
            o[0] = s_sum[i % 3][i / 3];
            if constexpr (CH == 2) o[3 * P] = s_sum[3 + i % 3][i / 3];
        }
    }
}

// v of the cells [c0, c0 + gridDim.x) (counted from cell0): the sparse part, or
// its split parts in order, plus the cell's slots in list order
__global__ __launch_bounds__(256) void fmm_m2l_sum_kernel(int cell0, int c0, int P3, int channels,
                                                          int splits,
                                                          const int *__restrict__ slot_ptr,
                                                          int slot0,
                                                          const double *__restrict__ slots,
                                                          const double *__restrict__ vpart,
                                                          double *__restrict__ vu,
                                                          double *__restrict__ vw) {
    const int ci = c0 + blockIdx.x, W = P3 * channels;
    const int s0 = slot_ptr[ci] - slot0, s1 = slot_ptr[ci + 1] - slot0;
    for (int i = blockIdx.y * blockDim.x + threadIdx.x; i < W; i += blockDim.x * gridDim.y) {
        double *v = (i < P3 ? vu : vw) + (size_t)(cell0 + ci) * P3 + i % P3;
        double t = 0.0;
        if (splits == 1)
            t = *v;
        else
            for (int j = 0; j < splits; ++j) t += vpart[((size_t)ci * splits + j) * W + i];
        const double *s = slots + (size_t)s0 * W + i;
#pragma unroll 4
        for (int j = s0; j < s1; ++j, s += W) t += *s;
        *v = t;
    }
}

template <bool WALL, int CH, class A>
void run_m2l(const FmmState &F, hipStream_t s) {
    const int P = F.P, L = F.L;
    const Geo g{F.o[0], F.o[1], F.o[2], F.S, F.n, P};
    const float *tab = F.tab.as<float>();
    const Vec4<A> *sf = F.slam.as<Vec4<A>>(), *st = F.slam2.as<Vec4<A>>();
    const Vec4<A> *qf = F.qhat.as<Vec4<A>>(), *qt = F.qhat2.as<Vec4<A>>();
    double *vu = F.v.as<double>(), *vw = F.v2.as<double>();
    const int cell0 = F.lvl[2], nc = F.lvl[L + 1] - cell0, splits = F.splits;
    const int W = 3 * P * CH;
    with_order(F.n, [&](auto o) {
        constexpr int NO = decltype(o)::value;
        fmm_p2l_kernel<WALL, CH, A, NO>
            <<<round_up(nc * splits, 8 * kXcdChunk), SparseShape<NO>::block, 0, s>>>(
                g, tab, F.cc.as<int4>(), F.sp_ptr.as<int>(), F.sp.as<int>(), F.sp_order.as<int>(), cell0,
                nc * splits,
                splits, F.rng.as<int2>(), F.shi.as<float4>(), F.slo.as<float4>(), sf, st, qf, qt, vu, vw,
                F.vsplit.as<double>());
        for (const FmmChunk &ch : F.chunks) {
            const int tasks = (ch.batch1 - ch.batch0) * ((NO * NO * NO + 15) / 16);
            const int items = (tasks + kDenseWaves - 1) / kDenseWaves;
            if (items > 0)
                fmm_m2l_dense_kernel<WALL, CH, A, (CH == 1 ? 2 : 1), NO>
                    <<<round_up(items, 8 * kXcdChunk), 64 * kDenseWaves, 0, s>>>(
                        g, tab, F.batches.as<FmmBatch>() + ch.batch0, tasks, items,
                        F.cols.as<int2>(), qf, qt, F.slots.as<double>());
            if (items > 0 || splits > 1)
                fmm_m2l_sum_kernel<<<dim3(ch.cell1 - ch.cell0, (W + 255) / 256),
                                     std::min(256, round_up(W, kWave)), 0, s>>>(cell0, ch.cell0, 3 * P, CH, splits,
                                          F.slot_ptr.as<int>(), ch.slot0, F.slots.as<double>(),
                                          F.vsplit.as<double>(), vu, vw);
        }
    });
}

}  // namespace

void fmm_m2l(const FmmState &F, hipStream_t s, int channels, bool wall, bool fp64) {
    if (channels == 2) {
        fp64 ? run_m2l<false, 2, double>(F, s) : run_m2l<false, 2, float>(F, s);
    } else if (wall) {
        fp64 ? run_m2l<true, 1, double>(F, s) : run_m2l<true, 1, float>(F, s);
    } else {
        fp64 ? run_m2l<false, 1, double>(F, s) : run_m2l<false, 1, float>(F, s);
    }
}

}  // namespace arb
