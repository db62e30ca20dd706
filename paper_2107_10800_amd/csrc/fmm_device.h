// Device helpers of the fast product shared by its translation units (fmm.hip:
// tree, P2M, M2M, L2L; fmm_m2l.hip: M2L; fmm_near.hip: near field, L2P).
#pragma once
#include <type_traits>

#include "rot_device.h"

namespace arb {

constexpr int kTabNode = 0, kTabDen = kFmmMaxOrder, kTabT1 = 2 * kFmmMaxOrder;
constexpr int kTabSize = 2 * kFmmMaxOrder + 2 * kFmmMaxOrder * kFmmMaxOrder;
constexpr int kFmmRun = 32;  // sources per float partial sum

template <class A>
using Vec4 = std::conditional_t<std::is_same_v<A, float>, float4, double4>;

template <class A>
__device__ __forceinline__ Vec4<A> vec4(A x, A y, A z) {
    Vec4<A> r;
    r.x = x;
    r.y = y;
    r.z = z;
    r.w = A(0);
    return r;
}

struct Geo {
    double ox, oy, oz, S;  // root cube in units of a
    int n, P;
};

__device__ __forceinline__ void load_tab(const float *__restrict__ g, float *tab) {
    for (int i = threadIdx.x; i < kTabSize; i += blockDim.x) tab[i] = g[i];
    __syncthreads();
}

// the item of this workgroup when the launch has round_up(items, 8 kXcdChunk)
// workgroups: consecutive workgroups are dealt round-robin to the 8 XCDs, so
// this gives each XCD runs of kXcdChunk consecutive items (neighbouring cells in
// Morton order, which read the same leaves and multipole weights, share its
// L2), the runs dealt round-robin to keep the XCDs' loads even; -1 past the end
constexpr int kXcdChunk = 16;
__device__ __forceinline__ int xcd_item(int items) {
    const int x = blockIdx.x % 8, j = blockIdx.x / 8;
    const int it = (j / kXcdChunk) * 8 * kXcdChunk + x * kXcdChunk + j % kXcdChunk;
    return it < items ? it : -1;
}

// a double split into float hi + lo
struct F2 {
    float h, l;
};
__device__ __forceinline__ F2 split(double x) {
    const float h = (float)x;
    return F2{h, (float)(x - (double)h)};
}

__device__ __forceinline__ double centre(double o, double side, int i) {
    return o + ((double)i + 0.5) * side;
}

inline int round_up(int x, int m) { return (x + m - 1) / m * m; }

// calls f with the order n (2..kFmmMaxOrder, checked when the options are
// read) as a compile-time constant, for the kernels whose loops unroll over it
template <class F> void with_order(int n, F &&f) {
    static_assert(kFmmMaxOrder == 8, "cases 2..8");
    switch (n) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
    }
}

}  // namespace arb
