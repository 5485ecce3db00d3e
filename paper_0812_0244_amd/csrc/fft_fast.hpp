// In-register DFTs with compile-time twiddles, the ordering of one wave's LDS
// accesses, and the radix orders of the lengths (the schedule's listing).
#pragma once

#include <utility>

#include "fft_lds.hpp"

namespace vdwnl {

// ---------------------------------------------------------------- compile-time trigonometry

namespace ct {
constexpr double kPi = 3.14159265358979323846264338327950288;
constexpr double sin_poly(double x) {   // |x| <= pi/4
    double x2 = x * x, term = x, sum = x;
    for (int n = 1; n < 14; ++n) {
        term *= -x2 / ((2.0 * n) * (2.0 * n + 1.0));
        sum += term;
    }
    return sum;
}
constexpr double cos_poly(double x) {
    double x2 = x * x, term = 1.0, sum = 1.0;
    for (int n = 1; n < 14; ++n) {
        term *= -x2 / ((2.0 * n - 1.0) * (2.0 * n));
        sum += term;
    }
    return sum;
}
// cos and sin of 2 pi m / n (m, n integers), exact to double rounding
constexpr double cos2pi(int m, int n) {
    m %= n;
    if (m < 0) m += n;
    // quadrant q with angle = q pi/2 + r, |r| <= pi/4
    const int q = (4 * m + n / 2) / n;                 // nearest multiple of n/4
    const double r = 2.0 * kPi * ((double)m / n - (double)q / 4.0);
    switch (q & 3) {
        case 0: return cos_poly(r);
        case 1: return -sin_poly(r);
        case 2: return -cos_poly(r);
        default: return sin_poly(r);
    }
}
constexpr double sin2pi(int m, int n) {
    m %= n;
    if (m < 0) m += n;
    const int q = (4 * m + n / 2) / n;
    const double r = 2.0 * kPi * ((double)m / n - (double)q / 4.0);
    switch (q & 3) {
        case 0: return sin_poly(r);
        case 1: return cos_poly(r);
        case 2: return -sin_poly(r);
        default: return -cos_poly(r);
    }
}
constexpr int gcd(int a, int b) { return b == 0 ? a : gcd(b, a % b); }
}  // namespace ct

// ---------------------------------------------------------------- in-register DFTs

// X_q = sum_r v_r exp(S 2 pi i r q / R), in place
template <typename T, int R, int S>
struct Dft {
    // R = P Q, P the first base radix dividing R
    static constexpr int P = (R % 4 == 0) ? 4 : (R % 2 == 0) ? 2 : (R % 5 == 0) ? 5 : 3;
    static constexpr int Q = R / P;
    __device__ __forceinline__ static void run(C2<T> *v) {
        C2<T> y[R];
#pragma unroll
        for (int n2 = 0; n2 < Q; ++n2) {
            C2<T> a[P];
#pragma unroll
            for (int n1 = 0; n1 < P; ++n1) a[n1] = v[Q * n1 + n2];
            Dft<T, P, S>::run(a);
#pragma unroll
            for (int k1 = 0; k1 < P; ++k1) {
                const int e = n2 * k1;
                if (e % R == 0) {
                    y[n2 * P + k1] = a[k1];
                } else {
                    const T c = (T)ct::cos2pi(e, R), s = (T)(S * ct::sin2pi(e, R));
                    y[n2 * P + k1] = mk<T>(a[k1].x * c - a[k1].y * s, a[k1].x * s + a[k1].y * c);
                }
            }
        }
#pragma unroll
        for (int k1 = 0; k1 < P; ++k1) {
            C2<T> b[Q];
#pragma unroll
            for (int n2 = 0; n2 < Q; ++n2) b[n2] = y[n2 * P + k1];
            Dft<T, Q, S>::run(b);
#pragma unroll
            for (int k2 = 0; k2 < Q; ++k2) v[k1 + P * k2] = b[k2];
        }
    }
};
template <typename T, int S> struct Dft<T, 1, S> { __device__ __forceinline__ static void run(C2<T> *) {} };
template <typename T, int S> struct Dft<T, 2, S> { __device__ __forceinline__ static void run(C2<T> *v) { dft2<T>(v); } };
template <typename T, int S> struct Dft<T, 3, S> { __device__ __forceinline__ static void run(C2<T> *v) { dft3<T>(v, (T)S); } };
template <typename T, int S> struct Dft<T, 4, S> {
    __device__ __forceinline__ static void run(C2<T> *v) { dft4<T>(v[0], v[1], v[2], v[3], (T)S); }
};
template <typename T, int S> struct Dft<T, 5, S> { __device__ __forceinline__ static void run(C2<T> *v) { dft5<T>(v, (T)S); } };
template <typename T, int S> struct Dft<T, 8, S> { __device__ __forceinline__ static void run(C2<T> *v) { dft8<T>(v, (T)S); } };

// ---------------------------------------------------------------- wave ordering

// Order the wave's LDS accesses.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- lengths

// Lengths with radix orders (vdwnl_radix_order), which are also those whose
// axis-3 passes are compiled for the length; class kLenGeneric: any other.
constexpr int kFastLens[] = {24, 32, 48, 64, 96, 128, 160, 320};
constexpr int kNumLenClasses = 9;
constexpr int kLenGeneric = 8;

__host__ __device__ constexpr int len_class(int n) {
    for (int i = 0; i < kLenGeneric; ++i)
        if (kFastLens[i] == n) return i;
    return kLenGeneric;
}

// Radix orders of each length class.  The transforms run as splits into two
// radices (fft_split.hpp) whatever order a schedule names; the lists describe
// the factorisations vdwnl_radix_order reports.  Entries end at the first
// zero.
constexpr int kMaxVariants = 6;
constexpr int kRadixOrders[kNumLenClasses][kMaxVariants][5] = {
    {{4, 3, 2}},
    {{8, 4}, {4, 8}},
    {{4, 4, 3}, {3, 4, 4}},
    {{8, 8}, {4, 4, 4}, {16, 4}, {4, 16}},
    {{4, 4, 2, 3}, {2, 4, 4, 3}, {3, 4, 4, 2}},
    {{8, 4, 4}, {4, 4, 8}, {2, 8, 8}, {4, 8, 4},
     {16, 8}, {8, 16}},
    {{4, 4, 2, 5}, {5, 4, 4, 2}},
    {{4, 4, 4, 5}, {5, 4, 4, 4}},
    {},
};

__host__ __device__ constexpr int num_radices(int lc, int v) {
    int n = 0;
    while (n < 5 && kRadixOrders[lc][v][n] != 0) ++n;
    return n;
}

__host__ __device__ constexpr int num_variants(int lc) {
    int v = 0;
    while (v < kMaxVariants && num_radices(lc, v) > 0) ++v;
    return v;
}

constexpr int kNumVariants[kNumLenClasses] = {num_variants(0), num_variants(1), num_variants(2), num_variants(3),
                                              num_variants(4), num_variants(5), num_variants(6), num_variants(7),
                                              1};

// The radix sequence of class lc, order v (host side), into r[]; its length.
inline int radix_order_of(int lc, int v, int *r) {
    const int n = num_radices(lc, v);
    for (int i = 0; i < n; ++i) r[i] = kRadixOrders[lc][v][i];
    return n;
}

}  // namespace vdwnl
