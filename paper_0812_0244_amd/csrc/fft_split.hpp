// Transforms of a length L = R1 R2 done as two register DFTs with one exchange
// through LDS (R1 <= R2 <= 27).  Index n = j + R2 r (j < R2, r < R1), frequency
// k = k1 + R1 k2 (k1 < R1, k2 < R2):
//   step one   item (line, j):  y_j[k1] = W_L^(j k1) sum_r x[j + R2 r] W_R1^(r k1)
//   step two   item (line, k1): X[k1 + R1 k2] = sum_j y_j[k1] W_R2^(j k2)
// and for the inverse the two steps in the opposite order with conjugate
// factors.  Step one's inputs (and step two's outputs) are rows of the grid,
// so they go between global memory and registers directly; y_j[k1] sits at
// LDS slot k1 R2 + j, and a step reads and writes the slots of its own item
// only.  A line thus crosses LDS once instead of once per radix pass and at
// both ends, and any length runs from one kernel per radix class: the
// radices are wave-uniform run-time values that select an unrolled DFT.
#pragma once

#include "fft_fast.hpp"
#include "tile_io.hpp"

namespace vdwnl {

// Radices of the split transforms.  A kernel is compiled for a largest radix
// (its class) since the largest DFT sets the registers of all its lengths:
// up to 10 (most lengths to 100), 16 (to 256), 20 (to 400) and 27 (to 405).
constexpr int kSplitRadices[] = {1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27};
constexpr int kSplitClassMax[] = {10, 16, 20, 27};
constexpr int kZClassMax[] = {10, 16, 20, 25};      // (the fused axis-1 pass: lengths to 204)
constexpr int kNumSplitClasses = 4;
constexpr int kSplitMaxLen = 405;

// The most even split of n into two radices, r1 <= r2 (false: none).
inline bool split_radices(int n, int &r1, int &r2) {
    r1 = r2 = 0;
    if (n < 1 || n > kSplitMaxLen) return false;
    for (int a : kSplitRadices)
        for (int b : kSplitRadices)
            if (a <= b && a * b == n && (r2 == 0 || b < r2)) { r1 = a; r2 = b; }
    return r2 != 0;
}

// Class of a length's split (index of kSplitClassMax), or kLenGeneric: no split.
inline int split_class(int n) {
    int r1, r2;
    if (!split_radices(n, r1, r2)) return kLenGeneric;
    for (int c = 0; c < kNumSplitClasses; ++c)
        if (r2 <= kSplitClassMax[c]) return c;
    return kLenGeneric;
}

// log2 of the lanes along a tile (16-byte chunks of a row, or derivative
// lines) in the passes with an item per thread: 16, or 8 where 16 R2 threads
// would exceed a workgroup.
constexpr int tile_lanes(int rmax) { return 16 * rmax <= kMaxThreads ? 4 : 3; }

// f(integral_constant<R>) for the run-time radix r <= RMAX (uniform).
template <int RMAX, typename F>
__device__ __forceinline__ void with_radix(int r, F &&f) {
#define VDWNL_RADIX(R) case R: if constexpr (R <= RMAX) f(std::integral_constant<int, R>{}); break;
    switch (__builtin_amdgcn_readfirstlane(r)) {
        VDWNL_RADIX(1) VDWNL_RADIX(2) VDWNL_RADIX(3) VDWNL_RADIX(4) VDWNL_RADIX(5) VDWNL_RADIX(6)
        VDWNL_RADIX(8) VDWNL_RADIX(9) VDWNL_RADIX(10) VDWNL_RADIX(12) VDWNL_RADIX(15) VDWNL_RADIX(16)
        VDWNL_RADIX(18) VDWNL_RADIX(20) VDWNL_RADIX(24) VDWNL_RADIX(25) VDWNL_RADIX(27)
        default: break;
    }
#undef VDWNL_RADIX
}

// Division of items and positions by a run-time length: x / d as the high
// half of x m, m = floor(2^32 / d) + 1, exact while x d < 2^32 (items of a tile
// and positions in a row stay below 2^16, as do the divisors).  A run-time
// integer division takes some twenty instructions, several times per thread.
// m comes from the host with the plan (0 for d = 1).
constexpr uint32_t div_magic(int d) { return d > 1 ? 0xffffffffu / (uint32_t)d + 1u : 0u; }
struct FastDiv {
    uint32_t m;
    __device__ __forceinline__ int operator()(int x) const { return m ? (int)__umulhi((uint32_t)x, m) : x; }
};

// 16-byte chunks of complex values: two in FP32, one in FP64.
template <typename T> struct Chunk;
template <> struct Chunk<float> {
    using V = float4;
    static constexpr int N = 2;
    __device__ __forceinline__ static void split(const float4 &v, float2 *c) { c[0] = mk<float>(v.x, v.y); c[1] = mk<float>(v.z, v.w); }
    __device__ __forceinline__ static float4 join(const float2 *c) { return make_float4(c[0].x, c[0].y, c[1].x, c[1].y); }
};
template <> struct Chunk<double> {
    using V = double2;
    static constexpr int N = 1;
    __device__ __forceinline__ static void split(const double2 &v, double2 *c) { c[0] = v; }
    __device__ __forceinline__ static double2 join(const double2 *c) { return c[0]; }
};

// W_L^(j k), k = 1 .. R-1 (sign S: -1 as tabulated, +1 conjugate), the factors
// between the two steps for item j; tw: the length's table in global memory
// (every item of a wave reads a few entries of it, from cache)
template <typename T, int S, int R>
__device__ __forceinline__ void split_twiddles(C2<T> *w, const C2<T> *tw, int j) {
#pragma unroll
    for (int k = 1; k < R; ++k) {
        w[k - 1] = gld(tw)[j * k];
        if (S > 0) w[k - 1].y = -w[k - 1].y;
    }
}

// The same from a copy of the table in LDS.
template <typename T, int S, int R>
__device__ __forceinline__ void lds_twiddles(C2<T> *w, const C2<T> *tw, int j) {
#pragma unroll
    for (int k = 1; k < R; ++k) {
        w[k - 1] = tw[j * k];
        if (S > 0) w[k - 1].y = -w[k - 1].y;
    }
}

}  // namespace vdwnl
