// Near field of the fast product (fmm.hip): direct sums over the adjacent leaves, and
// the pass that adds everything up per blob.
//
// A workgroup takes a block of up to 64 targets of one leaf against the leaves adjacent
// to it, its 4 wavefronts taking the source tiles (64 blobs of one adjacent leaf, each
// staged in the wavefront's own LDS) in turn, without barriers, so that small leaves
// and small trees still fill the chip.  The host lists up to 16,384 blocks longest first:
// with 12 per compute unit the last ones left 19 % of the time idle.
//
// Forces (3 components): the tensor of a pair serves both directions (M_ji = M_ij^T),
// so a block visits only the adjacent leaves after its own in cell order (and its
// own, one way) and sums both sides: as in the dense symmetric kernel the source-side
// sums follow their sources around the wavefront, lane l meeting source l + s at step
// s.  A block's source-side sums go to a slot of their own per (block, leaf); the
// last pass adds a blob's slots in the order of the blocks' leaves, so products repeat bit
// for bit.
// VALU-bound: 88 instructions per unordered pair against 2 x 71 one way; 8,192
// bacteria 3.54 -> 2.58 ms (issue rate at its limit, 1.46 per clock and CU), diatom
// colonies with double sums 0.89 -> 0.52 ms.  Blocks of 256 targets with their source
// sums joined in LDS write a quarter of the slots but wait on barriers: 2.98 ms.
// Where most leaves fill less than about half a tile, a wavefront's 64 steps both ways
// cost more than a step per source: such trees are summed one way (near_both_ways in
// fmm.hip), by an instance of its own without the second copy of the tile and the source
// sums, whose LDS and registers left a third of the wavefronts (100,000 blobs above the
// wall in leaves of 9: 784 us both ways, 237 one way; 500,000 in space in leaves of 15 with
// double sums: 1,149 us in the two-way instance, 854 in its own).
// Single-blob bodies (6 components) are summed one way, the tensor's few coefficients
// being a small part of a pair: 4,096 shells 3.19 -> 1.74 ms.  (Two targets per lane,
// to halve the LDS reads, leave too few blocks: 2.39 against 2.11 ms before the blocks
// were ordered.)
//
// Float sums run over at most kFmmRun blobs and are promoted to double.
#include <algorithm>

#include "fmm_device.h"

namespace arb {

namespace {

constexpr int kNearWaves = 4;
constexpr int kMaxNear = 27;  // adjacent cells, itself included

// free-space RPY coefficients c1, c2 (units of a) of M = c1 I + c2 r r^T
__device__ __forceinline__ void free_coef(float r2, float rinv, float &c1, float &c2) {
    constexpr CoefF c = kUnitCoefF;
    const float rinv2 = rinv * rinv, rinv3 = rinv * rinv2;
    c1 = fmaf(c.k1, rinv3, rinv);
    c2 = fmaf(-c.k2, rinv3 * rinv2, rinv3);
    ARB_IF_ANY_OVERLAP(r2 <= c.four_a2)
    if (r2 <= c.four_a2) {
        const float rv = r2 > 0.f ? rinv : 0.f;
        c1 = fmaf(-c.n2, r2 * rv, c.n1);
        c2 = rv * c.n3;
    }
    ARB_END_IF_ANY
}

template <class A>
__device__ __forceinline__ PairCoef<A> widen(const PairCoef<float> &p) {
    return PairCoef<A>{(A)p.cA, (A)p.cAe, (A)p.c2, (A)p.b, (A)p.c, (A)p.d, (A)p.e, (A)p.h2};
}

// f += M(d) lj, and with BOTH b += M(d)^T li: tensor coefficients in float, applied in A
template <bool WALL, bool BOTH, class A>
__device__ __forceinline__ void pair_acc(float dx, float dy, float dz, const TargetZ<float> &zsc,
                                         float zi, float zj, float h2, float mh22,
                                         const Vec4<A> &lj, const Vec4<A> &li, A *f, A *b) {
    const float dxy2 = fmaf(dx, dx, dy * dy);
    const float r2 = fmaf(dz, dz, dxy2);
    const float rinv = rsq_f32(r2);
    if constexpr (WALL) {
        const float Rz = zi + zj;
        const float Ri = rsq_f32(fmaf(Rz, Rz, dxy2));
        const PairCoef<A> p =
            widen<A>(wall_pair_coef<float>(r2, rinv, dxy2, zsc, zj, h2, mh22, Rz, Ri, kUnitCoefF));
        wall_pair_apply<A>(p, p.c, p.d, (A)dx, (A)dy, (A)dz, (A)Rz, lj.x, lj.y, lj.z, f[0], f[1],
                           f[2]);
        if constexpr (BOTH)
            wall_pair_apply<A>(p, p.d, p.c, (A)dx, (A)dy, (A)dz, (A)Rz, li.x, li.y, li.z, b[0],
                               b[1], b[2]);
    } else {
        float c1f, c2f;
        free_coef(r2, rinv, c1f, c2f);
        const A c1 = (A)c1f, c2 = (A)c2f, x = (A)dx, y = (A)dy, z = (A)dz;
        const A tj = c2 * fma(x, lj.x, fma(y, lj.y, z * lj.z));
        f[0] = fma(c1, lj.x, fma(tj, x, f[0]));
        f[1] = fma(c1, lj.y, fma(tj, y, f[1]));
        f[2] = fma(c1, lj.z, fma(tj, z, f[2]));
        if constexpr (BOTH) {
            const A ti = c2 * fma(x, li.x, fma(y, li.y, z * li.z));
            b[0] = fma(c1, li.x, fma(ti, x, b[0]));
            b[1] = fma(c1, li.y, fma(ti, y, b[1]));
            b[2] = fma(c1, li.z, fma(ti, z, b[2]));
        }
    }
}

// acc += N(d) (f, t): tensor coefficients in float (a = 1), applied in A
template <class A>
__device__ __forceinline__ void rot_acc(float dx, float dy, float dz, const Vec4<A> &f,
                                        const Vec4<A> &t, A *acc) {
    const float r2 = fmaf(dz, dz, fmaf(dx, dx, dy * dy));
    const RotTerms<float> k = rot_terms<float>(r2, rsq_f32(r2), kUnitRotCoef);
    const RotTerms<A> ka{(A)k.c1, (A)k.c2, (A)k.cr, (A)k.d1, (A)k.d2};
    rot_one_way<A>(ka, (A)dx, (A)dy, (A)dz, f.x, f.y, f.z, t.x, t.y, t.z, acc);
}

// v of lane (l + 1) mod 64 for lane l, as in the dense symmetric kernels: the wall's
// loop is VALU-bound and shuffles through the LDS crossbar, the free-space loop moves
// by DPP (wave_rol:1)
template <bool WALL>
__device__ __forceinline__ float next_lane(float v, int src) {
    if (WALL) return __shfl(v, src);
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x134, 0xF, 0xF, false));
}
template <bool WALL>
__device__ __forceinline__ double next_lane(double v, int src) {
    if (WALL) return __shfl(v, src);
    const long long q = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(q & 0xffffffffll), 0x134, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(q >> 32), 0x134, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// work[item] = (leaf, first target, targets, first slot); near: the adjacent leaves;
// own[c][k]: the sums of sorted blob k over its own leaf and (SYM) the adjacent leaves
// after it, or (!SYM) all adjacent leaves; slots: per block, for each adjacent leaf
// after its own in list order, 3 x |leaf| source-side sums (component-major)
template <bool WALL, int CH, bool SYM, class A>
__global__ __launch_bounds__(64 * kNearWaves) void fmm_near_kernel(
    int N, const int2 *__restrict__ rng, const int *__restrict__ near_ptr,
    const int *__restrict__ near, int leaf0, const int4 *__restrict__ work, int items,
    const float4 *__restrict__ shi, const float4 *__restrict__ slo,
    const Vec4<A> *__restrict__ sf, const Vec4<A> *__restrict__ st, double *__restrict__ own,
    double *__restrict__ slots) {
    constexpr int NB = 3 * CH, W = kNearWaves;
    const int item = xcd_item(items);
    if (item < 0) return;
    // a source tile per wavefront, twice over for the rotation (SYM)
    constexpr int TS = SYM ? 128 : 64;
    __shared__ float4 s_pos[(2 * W * TS * 16 > W * NB * 64 * 8 ? 2 * W * TS : W * NB * 32)];
    float4(*s_hi)[TS] = reinterpret_cast<float4(*)[TS]>(s_pos), (*s_lo)[TS] = s_hi + W;
    __shared__ Vec4<A> s_f[W][TS], s_t[CH == 2 ? W : 1][64];
    __shared__ A s_comb[SYM ? W : 1][2][3][SYM ? 64 : 1];
    __shared__ int s_beg[kMaxNear], s_cnt[kMaxNear], s_first[kMaxNear + 1], s_slot[kMaxNear];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int4 it = work[item];
    const int c = it.x, nt = it.z;
    // the visited leaves: blob ranges, running counts of their tiles and slots
    if (w == 0) {
        const int e0 = near_ptr[c - leaf0], ne = near_ptr[c - leaf0 + 1] - e0;
        int cnt = 0, q = -1;
        if (lane < ne) {
            q = near[e0 + lane];
            const int2 r = rng[q];
            cnt = SYM && q < c ? 0 : r.y - r.x;
            s_beg[lane] = r.x;
            s_cnt[lane] = cnt;
        }
        int tiles = (cnt + 63) / 64, sl = q > c ? cnt : 0;
        const int own_sl = sl;
        for (int off = 1; off < 32; off <<= 1) {
            const int a = __shfl_up(tiles, off), b = __shfl_up(sl, off);
            if (lane >= off) {
                tiles += a;
                sl += b;
            }
        }
        if (lane < ne) {
            s_first[lane + 1] = tiles;
            s_slot[lane] = SYM && q > c ? it.w + sl - own_sl : -1;
        }
        if (lane == 0) s_first[0] = 0;
        if (lane >= ne && lane < kMaxNear) s_first[lane + 1] = tiles;
    }
    const int i = it.y + lane;
    const bool act = lane < nt;
    float4 th = make_float4(-1e6f, -1e6f, 10.f, 20.f), tl = make_float4(0.f, 0.f, 0.f, 0.f);
    Vec4<A> lt = vec4<A>(0, 0, 0);
    if (act) {
        th = shi[i];
        tl = slo[i];
        if (SYM) lt = sf[i];
    }
    const float zi = th.z + tl.z;
    const TargetZ<float> zsc = target_z(zi);
    const int src = (lane + 1) & 63;
    double u[NB] = {};
    __syncthreads();
    const int T = s_first[kMaxNear];
    // every wavefront stages, sums and stores its own source tiles: only its own LDS
    // accesses have to stay in order
    auto sync = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int t = w, e = 0; t < T; t += W) {
        while (s_first[e + 1] <= t) ++e;  // the tile's leaf
        const int j0 = 64 * (t - s_first[e]), cnt = s_cnt[e];
        sync();
        {
            const int j = s_beg[e] + j0 + lane;
            float4 h = make_float4(1e6f, 1e6f, 10.f, 20.f);
            float4 l = make_float4(0.f, 0.f, 0.f, -400.f);
            Vec4<A> f = vec4<A>(0, 0, 0);
            const bool ok = j0 + lane < cnt;
            if (ok) {
                h = shi[j];
                l = slo[j];
                f = sf[j];
            }
            s_hi[w][lane] = h;
            s_lo[w][lane] = l;
            s_f[w][lane] = f;
            if constexpr (SYM) {
                s_hi[w][lane + 64] = h;
                s_lo[w][lane + 64] = l;
                s_f[w][lane + 64] = f;
            }
            if constexpr (CH == 2) s_t[w][lane] = ok ? st[j] : vec4<A>(0, 0, 0);
        }
        sync();
        const int slot = SYM ? s_slot[e] : -1;
        {
            const float4 *ph = s_hi[w], *pl = s_lo[w];
            const Vec4<A> *pf = s_f[w];
            if (slot < 0) {
                const int nj = min(64, cnt - j0);
                for (int k0 = 0; k0 < nj; k0 += kFmmRun) {
                    const int k1 = min(k0 + kFmmRun, nj);
                    A f[NB] = {};
#pragma unroll 2
                    for (int k = k0; k < k1; ++k) {
                        const float4 sh = ph[k], sl = pl[k];
                        const float dx = (th.x - sh.x) + (tl.x - sl.x);
                        const float dy = (th.y - sh.y) + (tl.y - sl.y);
                        const float dz = (th.z - sh.z) + (tl.z - sl.z);
                        if constexpr (CH == 1)
                            pair_acc<WALL, false, A>(dx, dy, dz, zsc, zi, sh.z, sh.w, sl.w, pf[k],
                                                     lt, f, nullptr);
                        else
                            rot_acc<A>(dx, dy, dz, pf[k], s_t[w][k], f);
                    }
#pragma unroll
                    for (int q = 0; q < NB; ++q) u[q] += (double)f[q];
                }
            } else if constexpr (SYM) {
                // lane l meets source l + s; after 32 steps it holds the sums of
                // source l + 32, after 64 those of source l
#pragma unroll 1
                for (int h = 0; h < 2; ++h) {
                    A f[3] = {}, b[3] = {};
#pragma unroll 2
                    for (int k = lane + 32 * h, s = 0; s < 32; ++s, ++k) {
                        const float4 sh = ph[k], sl = pl[k];
                        const float dx = (th.x - sh.x) + (tl.x - sl.x);
                        const float dy = (th.y - sh.y) + (tl.y - sl.y);
                        const float dz = (th.z - sh.z) + (tl.z - sl.z);
                        pair_acc<WALL, true, A>(dx, dy, dz, zsc, zi, sh.z, sh.w, sl.w, pf[k], lt,
                                                f, b);
#pragma unroll
                        for (int q = 0; q < 3; ++q) b[q] = next_lane<WALL>(b[q], src);
                    }
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        u[q] += (double)f[q];
                        s_comb[w][h][q][h ? lane : (lane + 32) & 63] = b[q];
                    }
                }
            }
        }
        if constexpr (SYM) {
            if (slot < 0) continue;
            sync();
            if (j0 + lane < cnt) {
                double *o = slots + (size_t)slot * 3 + j0 + lane;
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    o[(size_t)q * cnt] =
                        (double)s_comb[w][0][q][lane] + (double)s_comb[w][1][q][lane];
            }
        }
    }
    // the wavefronts' sums, added in their order (through the staged positions' memory)
    double(*s_own)[NB][64] = reinterpret_cast<double(*)[NB][64]>(s_pos);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NB; ++q) s_own[w][q][lane] = u[q];
    __syncthreads();
    if (w > 0 || !act) return;
    for (int k = 1; k < W; ++k)
#pragma unroll
        for (int q = 0; q < NB; ++q) u[q] += s_own[k][q][lane];
#pragma unroll
    for (int q = 0; q < NB; ++q) own[(size_t)q * N + i] = u[q];
}

// Lagrange polynomials l_0..l_{n-1}(u) at the Chebyshev points (product form)
template <int NO>
__device__ __forceinline__ void lag_all(const float *tab, float u, float *l) {
#pragma unroll
    for (int k = 0; k < NO; ++k) {
        float p = tab[kTabDen + k];
#pragma unroll
        for (int j = 0; j < NO; ++j)
            if (j != k) p *= u - tab[kTabNode + j];
        l[k] = p;
    }
}

// per blob (64 of one leaf per workgroup): the near field's own sums, its slots in
// block order and the leaf's interpolant; partial[c][i] in the original blob order
template <int CH, int NO>
__global__ __launch_bounds__(64) void fmm_finish_kernel(
    Geo g, const float *__restrict__ tabg, int N, int far, const int4 *__restrict__ cc,
    const int2 *__restrict__ rng, int leaf0, const int2 *__restrict__ work, int items,
    const int *__restrict__ perm, const float4 *__restrict__ shi, const float4 *__restrict__ slo,
    const int *__restrict__ in_ptr, const int *__restrict__ in, const double *__restrict__ own,
    const double *__restrict__ slots, const double *__restrict__ vu,
    const double *__restrict__ vw, double *__restrict__ partial) {
    constexpr int NB = 3 * CH;
    const int item = xcd_item(items);
    if (item < 0) return;
    __shared__ float tab[kTabSize];
    load_tab(tabg, tab);
    const int2 wk = work[item];
    const int c = wk.x, i = wk.y + threadIdx.x;
    const int2 r = rng[c];
    if (i >= r.y) return;
    double u[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) u[q] = own[(size_t)q * N + i];
    if (CH == 1 && in_ptr) {
        const int cnt = r.y - r.x, j = i - r.x;
        const int e1 = in_ptr[c - leaf0 + 1];
#pragma unroll 2
        for (int e = in_ptr[c - leaf0]; e < e1; ++e) {
            const double *s = slots + (size_t)in[e] * 3 + j;
            u[0] += s[0];
            u[1] += s[cnt];
            u[2] += s[2 * (size_t)cnt];
        }
    }
    if (far) {
        const int4 ci = cc[c];
        const double side = ldexp(g.S, -ci.w);
        const F2 cx = split(centre(g.ox, side, ci.x)), cy = split(centre(g.oy, side, ci.y)),
                 cz = split(centre(g.oz, side, ci.z));
        const float iw = (float)(2.0 / side);
        const float4 th = shi[i], tl = slo[i];
        float lx[NO], ly[NO], lz[NO];
        lag_all<NO>(tab, ((th.x - cx.h) + (tl.x - cx.l)) * iw, lx);
        lag_all<NO>(tab, ((th.y - cy.h) + (tl.y - cy.l)) * iw, ly);
        lag_all<NO>(tab, ((th.z - cz.h) + (tl.z - cz.l)) * iw, lz);
        const double *pu = vu + (size_t)c * (3 * NO * NO * NO);
        const double *pw = CH == 2 ? vw + (size_t)c * (3 * NO * NO * NO) : nullptr;
        double s[NB] = {};
#pragma unroll
        for (int kx = 0; kx < NO; ++kx)
#pragma unroll 1
            for (int ky = 0; ky < NO; ++ky) {
                float b = 0.f;
#pragma unroll
                for (int k = 0; k < NO; ++k) b = k == ky ? lx[kx] * ly[k] : b;
                const int q0 = 3 * (kx * NO + ky) * NO;
#pragma unroll
                for (int kz = 0; kz < NO; ++kz) {
                    const double wk2 = (double)(b * lz[kz]);
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        s[q] = fma(wk2, pu[q0 + 3 * kz + q], s[q]);
                        if constexpr (CH == 2) s[3 + q] = fma(wk2, pw[q0 + 3 * kz + q], s[3 + q]);
                    }
                }
            }
#pragma unroll
        for (int q = 0; q < NB; ++q) u[q] += s[q];
    }
    const size_t o = (size_t)perm[i];
#pragma unroll
    for (int q = 0; q < NB; ++q) partial[(size_t)q * N + o] = u[q];
}

template <bool WALL, int CH, class A>
void run_near(const FmmState &F, hipStream_t s, double *partial) {
    const int N = F.N, leaf0 = F.lvl[F.L];
    const Geo g{F.o[0], F.o[1], F.o[2], F.S, F.n, F.P};
    const bool sym = CH == 1 && F.near_sym;
    auto go = [&](auto both) {
        fmm_near_kernel<WALL, CH, decltype(both)::value, A>
            <<<round_up(F.n_blocks, 8 * kXcdChunk), 64 * kNearWaves, 0, s>>>(
                N, F.rng.as<int2>(), F.near_ptr.as<int>(), F.nearl.as<int>(), leaf0,
                F.blocks.as<int4>(), F.n_blocks, F.shi.as<float4>(), F.slo.as<float4>(),
                F.slam.as<Vec4<A>>(), F.slam2.as<Vec4<A>>(), F.own.as<double>(),
                F.near_slots.as<double>());
    };
    if (sym)
        go(std::bool_constant<CH == 1>());
    else
        go(std::false_type());
    with_order(F.n, [&](auto o) {
        fmm_finish_kernel<CH, decltype(o)::value><<<round_up(F.nwork, 8 * kXcdChunk), 64, 0, s>>>(
            g, F.tab.as<float>(), N, F.L >= 2 ? 1 : 0, F.cc.as<int4>(), F.rng.as<int2>(), leaf0,
            F.work.as<int2>(), F.nwork, F.perm.as<int>(), F.shi.as<float4>(), F.slo.as<float4>(),
            sym ? F.in_ptr.as<int>() : nullptr, F.in.as<int>(), F.own.as<double>(),
            F.near_slots.as<double>(), F.v.as<double>(), F.v2.as<double>(), partial);
    });
}

}  // namespace

void fmm_near(const FmmState &F, hipStream_t s, int channels, bool wall, bool fp64,
              double *partial) {
    if (channels == 2) {
        fp64 ? run_near<false, 2, double>(F, s, partial) : run_near<false, 2, float>(F, s, partial);
    } else if (wall) {
        fp64 ? run_near<true, 1, double>(F, s, partial) : run_near<true, 1, float>(F, s, partial);
    } else {
        fp64 ? run_near<false, 1, double>(F, s, partial) : run_near<false, 1, float>(F, s, partial);
    }
}

}  // namespace arb
