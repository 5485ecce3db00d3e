// Copies between global memory and LDS tiles.  Each thread issues a batch of
// U independent loads before it writes any of them to LDS, so a wave keeps
// U requests per lane in flight instead of waiting on each one; row/column
// indices advance incrementally (no integer division per element).  The
// loads of a batch are unconditional (a load under a branch, even a
// wave-uniform one, is waited for where the branch joins, so the batch would
// go out one load at a time): a step past the end of the tile re-reads the
// tile's first element and its value is dropped.
#pragma once

#include "fft_fast.hpp"

namespace vdwnl {

constexpr int kUnroll = 8;

// The kernels reach global memory through pointers held in memory (the
// per-grid descriptors), which the compiler would access with flat
// instructions; those also count as LDS operations, so every LDS wait would
// also wait for outstanding global loads.  These casts make the accesses
// global ones.
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
#else   // the host pass only parses device code
template <typename T>
using gptr = T *;
#endif
template <typename T>
__device__ __forceinline__ gptr<const T> gld(const T *p) { return (gptr<const T>)p; }
template <typename T>
__device__ __forceinline__ gptr<T> gst(T *p) { return (gptr<T>)p; }

// Position (row l, column w) of flat element index i in rows of W columns,
// advanced by kThreads per step.
struct RowCursor {
    int l, w, dl, dw, W;
    __device__ __forceinline__ RowCursor(int i, int W_) : W(W_) {
        l = i / W_;
        w = i - l * W_;
        dl = kThreads / W_;
        dw = kThreads - dl * W_;
    }
    __device__ __forceinline__ void step() {
        w += dw;
        l += dl;
        if (w >= W) { w -= W; ++l; }
    }
};

// FP32 complex rows moved as 16-byte pairs when the row width, the global row
// stride and the global base allow it (W even, gstr even, g 16-byte aligned);
// LDS rows keep any stride (the pair is written as two 8-byte elements).
__device__ __forceinline__ bool pairable(const void *g, size_t gstr, int W) {
    return ((W | (int)(gstr & 1)) & 1) == 0 && (reinterpret_cast<uintptr_t>(g) & 15) == 0;
}

// Transposed copies: global rows l < nrows of W contiguous elements go to
// LDS lines w < W with element l at lds[w * lpitch + l] (lines contiguous, for
// FFTs along l with unit element stride).
template <int U = kUnroll>
__device__ __forceinline__ void rows_in_t(float2 *lds, int lpitch, const float2 *__restrict__ g, size_t gstr,
                                          int nrows, int W) {
    if (!pairable(g, gstr, W)) {
        const int total = nrows * W;
        RowCursor cur(threadIdx.x, W);
        for (int base = threadIdx.x; base < total; base += U * kThreads) {
            float rx[U], ry[U];
            int o[U];
    #pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool on = base + u * kThreads < total;
                const float2 v = gld(g)[on ? (size_t)cur.l * gstr + cur.w : 0];
                rx[u] = v.x;
                ry[u] = v.y;
                o[u] = on ? cur.w * lpitch + cur.l : -1;
                cur.step();
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (o[u] >= 0) lds[o[u]] = make_float2(rx[u], ry[u]);
        }
        return;
    }
    const int Wp = W / 2, total = nrows * Wp;
    const float4 *gp = reinterpret_cast<const float4 *>(g);
    const size_t gp_str = gstr / 2;
    RowCursor cur(threadIdx.x, Wp);
    for (int base = threadIdx.x; base < total; base += U * kThreads) {
        float4 r[U];
        int o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = base + u * kThreads < total;
            r[u] = gld(gp)[on ? (size_t)cur.l * gp_str + cur.w : 0];
            o[u] = on ? 2 * cur.w * lpitch + cur.l : -1;
            cur.step();
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (o[u] >= 0) {
                lds[o[u]] = make_float2(r[u].x, r[u].y);
                lds[o[u] + lpitch] = make_float2(r[u].z, r[u].w);
            }
    }
}

template <int U = kUnroll>
__device__ __forceinline__ void rows_out_t(float2 *__restrict__ g, size_t gstr, const float2 *lds, int lpitch,
                                           int nrows, int W) {
    if (!pairable(g, gstr, W)) {
        const int total = nrows * W;
        RowCursor cur(threadIdx.x, W);
        for (int base = threadIdx.x; base < total; base += U * kThreads) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (base + u * kThreads < total) gst(g)[(size_t)cur.l * gstr + cur.w] = lds[cur.w * lpitch + cur.l];
                cur.step();
            }
        }
        return;
    }
    const int Wp = W / 2, total = nrows * Wp;
    float4 *gp = reinterpret_cast<float4 *>(g);
    const size_t gp_str = gstr / 2;
    RowCursor cur(threadIdx.x, Wp);
    for (int base = threadIdx.x; base < total; base += U * kThreads) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + u * kThreads < total) {
                const float2 a = lds[2 * cur.w * lpitch + cur.l], b = lds[(2 * cur.w + 1) * lpitch + cur.l];
                gst(gp)[(size_t)cur.l * gp_str + cur.w] = make_float4(a.x, a.y, b.x, b.y);
            }
            cur.step();
        }
    }
}

template <int U = kUnroll>
__device__ __forceinline__ void rows_in_t(double2 *lds, int lpitch, const double2 *__restrict__ g, size_t gstr,
                                          int nrows, int W) {
    const int total = nrows * W;
    RowCursor cur(threadIdx.x, W);
    for (int base = threadIdx.x; base < total; base += U * kThreads) {
        double rx[U], ry[U];
        int o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = base + u * kThreads < total;
            const double2 v = gld(g)[on ? (size_t)cur.l * gstr + cur.w : 0];
            rx[u] = v.x;
            ry[u] = v.y;
            o[u] = on ? cur.w * lpitch + cur.l : -1;
            cur.step();
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (o[u] >= 0) lds[o[u]] = make_double2(rx[u], ry[u]);
    }
}

template <int U = kUnroll>
__device__ __forceinline__ void rows_out_t(double2 *__restrict__ g, size_t gstr, const double2 *lds, int lpitch,
                                           int nrows, int W) {
    const int total = nrows * W;
    RowCursor cur(threadIdx.x, W);
    for (int base = threadIdx.x; base < total; base += U * kThreads) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + u * kThreads < total) gst(g)[(size_t)cur.l * gstr + cur.w] = lds[cur.w * lpitch + cur.l];
            cur.step();
        }
    }
}

}  // namespace vdwnl
