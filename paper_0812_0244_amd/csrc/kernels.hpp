// HIP kernels of libvdwnl (gfx950), as templates in the working precision T;
// kernels_f32_{x,y,z}.hip and kernels_f64_{x,y,z}.hip instantiate them per pass
// family (compiled in parallel).  One evaluation of E_c^nl and v_nl is eleven
// passes over the grid with the spectral gradient (its gradient and
// divergence one pass per grid axis each), seven with finite differences;
// each pass is one launch per group of grids (by the classes their axis lengths
// split into, fft_split.hpp, and the kind of cell) that covers every grid of
// the group (a workgroup reads its work item from a tile list); gradient
// directions that do not wait for each other share one launch, and the energies
// are summed by the first workgroups of the inverse axis-2 pass.
//
// The 20 theta / u fields (the bulk of the traffic), the local chain and the
// divergence of w are computed in the working precision T (float or double).
// The spectral gradient of n always transforms in FP64: the gradient term of
// v_nl multiplies grad n by a factor that grows as 1/n, so FP32 rounding of a
// spectral grad n in the low-density regions would dominate the error of v.
//
// Fields are transformed with three 1-D FFT passes: along axis 3 (the
// contiguous one, real-to-complex by pairing two real lines into one complex
// line), axis 2 and axis 1.  Spectra keep all components of one k point
// together ([N1][N2][N3/2+1][V] complex), so the axis-1 pass of the 20 theta
// spectra holds every component of its k points in LDS and can apply the
// per-k kernel matrix between its forward and inverse FFTs.
#pragma once

#include "common.hpp"
#include "fft_split.hpp"

namespace vdwnl {

// ---------------------------------------------------------------- helpers

// Elementary functions of the local chain.  FP64: the device library.  FP32
// (arguments positive and normal there): built on the hardware base-2
// logarithm and exponential (v_log_f32, v_exp_f32), square root and
// reciprocal, each within about an ulp, in a few instructions where the
// library's general versions (special values, denormals, extra-precise
// arithmetic) take tens to a hundred.
__device__ __forceinline__ float hw_log(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }
__device__ __forceinline__ float hw_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }
template <typename T> __device__ __forceinline__ T dev_cbrt(T x);
template <> __device__ __forceinline__ float dev_cbrt(float x) {
    // 2^(log2(x)/3), then one Newton step for r^3 = x
    const float r = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(x) * (1.0f / 3.0f));
    return r + (x * __builtin_amdgcn_rcpf(r * r) - r) * (1.0f / 3.0f);
}
template <> __device__ __forceinline__ double dev_cbrt(double x) { return cbrt(x); }
template <typename T> __device__ __forceinline__ T dev_sqrt(T x);
template <> __device__ __forceinline__ float dev_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
template <> __device__ __forceinline__ double dev_sqrt(double x) { return sqrt(x); }
// 1/x: the hardware reciprocal in FP32 (within 1 ulp), a division in FP64
template <typename T> __device__ __forceinline__ T rcp(T x);
template <> __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
// FP64: the hardware estimate refined by two Newton-Raphson steps
// r <- r + r (1 - x r) (each doubles the correct bits; within an ulp or so
// of 1/x for normal x, against about fifteen instructions for a division)
template <> __device__ __forceinline__ double rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
template <typename T> __device__ __forceinline__ T dev_log1p(T x);
template <> __device__ __forceinline__ float dev_log1p(float x) {
    // log(u) x / (u - 1) with u = 1 + x as rounded: the quotient restores what
    // the rounding of 1 + x lost (Goldberg 1991, Theorem 4); x itself when u = 1
    const float u = 1.0f + x, d = u - 1.0f;
    return d == 0.0f ? x : hw_log(u) * (x * __builtin_amdgcn_rcpf(d));
}
template <> __device__ __forceinline__ double dev_log1p(double x) { return log1p(x); }
template <typename T> __device__ __forceinline__ T dev_exp(T x);
template <> __device__ __forceinline__ float dev_exp(float x) { return hw_exp(x); }
template <> __device__ __forceinline__ double dev_exp(double x) { return exp(x); }
template <typename T> __device__ __forceinline__ T dev_expm1(T x);
template <> __device__ __forceinline__ float dev_expm1(float x) {
    // |x| < 1/2: x (1 + x/2! + ... + x^8/9!) (Taylor; the rest is below 1e-9
    // relative); elsewhere exp(x) - 1, where no cancellation can hurt
    float p = 1.0f / 362880.0f;
    p = p * x + 1.0f / 40320.0f;
    p = p * x + 1.0f / 5040.0f;
    p = p * x + 1.0f / 720.0f;
    p = p * x + 1.0f / 120.0f;
    p = p * x + 1.0f / 24.0f;
    p = p * x + 1.0f / 6.0f;
    p = p * x + 0.5f;
    p = p * x + 1.0f;
    return fabsf(x) < 0.5f ? x * p : hw_exp(x) - 1.0f;
}
template <> __device__ __forceinline__ double dev_expm1(double x) { return expm1(x); }

__device__ __forceinline__ int freq_abs(int k, int N) { return k <= N - k ? k : N - k; }

// Sum over the workgroup in a fixed order (at most eight waves); result valid
// in thread 0.
__device__ __forceinline__ double block_sum(double v) {
    __shared__ double red[8];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < ((int)blockDim.x + 63) / 64; ++w) s += red[w];
    __syncthreads();
    return s;
}

// ---------------------------------------------------------------- q0 and the spline basis

// q0(n, |grad n|^2) before saturation and its partials (Dion et al. form,
// Perdew-Wang 1992 correlation), then the saturation of Eq. (Sat).
template <typename T, bool DERIV>
struct LocalQ {
    T q0, Q, dqdn, ndqds;    // ndqds = n dq0/dsigma (dq0/dsigma alone overflows FP32 at small n)
    T kf, eps, deps_dn;      // k_F, the LDA eps_c and (DERIV) d eps_c/dn

    __device__ __forceinline__ void eval(T n, T sigma, double qc, double iqc, int mc, const T *invm) {
        const T pi = (T)3.14159265358979323846;
        const T A = (T)0.031091, a1 = (T)0.21370;
        const T b1 = (T)7.5957, b2 = (T)3.5876, b3 = (T)1.6382, b4 = (T)0.49294;
        const T zg = (T)(0.8491 / 36.0);   // -Z_ab / 36
        // k_F = (3 pi^2 n)^(1/3), r_s = (3 / (4 pi n))^(1/3): one cube root
        const T cn = dev_cbrt<T>(n), icn = rcp<T>(cn), in = rcp<T>(n);
        kf = (T)3.0936677262801355 * cn;                  // (3 pi^2)^(1/3)
        const T rs = (T)0.6203504908994001 * icn;         // (3 / (4 pi))^(1/3)
        const T srs = dev_sqrt<T>(rs);
        const T P = b1 * srs + b2 * rs + b3 * rs * srs + b4 * rs * rs;
        const T iP2A = rcp<T>((T)2 * A * P);
        const T L = dev_log1p<T>(iP2A);
        eps = (T)-2 * A * ((T)1 + a1 * rs) * L;
        // sigma / (k_F n^2) as ((sigma / n) / n) / k_F: finite in FP32 wherever
        // |grad n| / n is, down to n_min (1 / (k_F n^2) alone is not below 1e-17)
        const T ikf = rcp<T>(kf);
        const T grad_term = zg * ((sigma * in) * in) * ikf;
        const T qraw = kf - ((T)4 * pi / (T)3) * eps + grad_term;
        if (DERIV) {
            const T dP = (T)0.5 * b1 * rcp<T>(srs) + b2 + (T)1.5 * b3 * srs + (T)2 * b4 * rs;
            const T deps_drs = (T)-2 * A * a1 * L + (T)2 * A * ((T)1 + a1 * rs) * dP * rcp<T>(P * ((T)2 * A * P + (T)1));
            deps_dn = deps_drs * (-rs * in * ((T)1 / (T)3));
            dqdn = kf * in * ((T)1 / (T)3) - ((T)4 * pi / (T)3) * deps_dn - ((T)7 / (T)3) * grad_term * in;
            ndqds = zg * ikf * in;
        }
        // h(x, x_c) = x_c (1 - exp(-S)), S = sum_{m<=m_c} (x/x_c)^m / m (Horner),
        // dh/dx = exp(-S) sum_{m<m_c} (x/x_c)^m.  1 - exp(-S) as -expm1(-S)
        // keeps its relative accuracy for small S.  S from 80 up (exp(-S) <
        // 2e-35), or overflowing, saturates: h = x_c, dh/dx = 0.  Below that
        // the derivative series stays under 80 m_c^2: no overflow in FP32.
        const T y = qraw * (T)iqc;
        T S = (T)0;
        for (int m = mc; m >= 1; --m) S = S * y + invm[m];
        S *= y;
        if (!(S < (T)80)) {
            q0 = (T)qc;
            Q = (T)0;
            if (DERIV) { dqdn = (T)0; ndqds = (T)0; }   // (their products with Q vanish)
        } else {
            q0 = (T)(-qc) * dev_expm1<T>(-S);
            if (DERIV) {
                T D = (T)0;
                for (int m = mc - 1; m >= 0; --m) D = D * y + (T)1;
                Q = dev_exp<T>(-S) * D;
            } else {
                Q = (T)0;
            }
        }
    }
};

// Largest finite value of T.
template <typename T>
__device__ __forceinline__ constexpr T finite_max() {
    if constexpr (sizeof(T) == 4) return __FLT_MAX__;
    else return __DBL_MAX__;
}

// The semilocal terms of Eq. (Exc) at one point, from n, sigma = |grad n|^2
// and the k_F, eps_c (and d eps_c/dn) of LocalQ.  Exchange: the revPBE GGA,
// e_x = e_u F_x(s) with e_u = -3 k_F n / (4 pi), s^2 = sigma / (4 k_F^2 n^2),
// F_x = 1 + kappa - kappa / (1 + mu s^2 / kappa), kappa = 1.245,
// mu = 0.066725 pi^2 / 3; correlation: the LDA e_c = n eps_c.
template <typename T>
struct Semilocal {
    T ex, ec;                // energies per volume
    T dn, ds;                // d(e_x + e_c)/dn, d e_x/dsigma (DERIV)
    template <bool DERIV>
    __device__ __forceinline__ void eval(T n, T sigma, const LocalQ<T, DERIV> &lq) {
        const T kappa = (T)1.245, mu = (T)(0.066725 * 3.14159265358979323846 * 3.14159265358979323846 / 3.0);
        const T in = rcp<T>(n), ikf = rcp<T>(lq.kf);
        const T eu = (T)(-3.0 / (4.0 * 3.14159265358979323846)) * lq.kf * n;
        // s^2 = sigma / (4 k_F^2 n^2), ordered to stay finite at small n; where
        // it still overflows (or is huge) F_x has reached 1 + kappa
        const T s2 = ((sigma * in) * in) * ((T)0.25 * ikf * ikf);
        const bool flat = !(s2 < (T)1e30);
        const T iden = flat ? (T)0 : rcp<T>((T)1 + (mu / kappa) * s2);
        const T fx = (T)1 + kappa - kappa * iden;
        ex = eu * fx;
        ec = n * lq.eps;
        if (DERIV) {
            const T dfx = mu * iden * iden;                  // dF_x / ds^2
            const T dfx_s2 = flat ? (T)0 : dfx * s2;
            // d e_u/dn = (4/3) e_u / n, d s^2/dn = -(8/3) s^2 / n;
            // d e_x/dsigma = e_u F_x' / (4 k_F^2 n^2) = -3 F_x' / (16 pi k_F n)
            dn = ((T)(4.0 / 3.0) * fx - (T)(8.0 / 3.0) * dfx_s2) * eu * in + lq.eps + n * lq.deps_dn;
            ds = (T)(-3.0 / (16.0 * 3.14159265358979323846)) * dfx * rcp<T>(lq.kf * n);
        }
    }
};

// Natural cubic cardinal splines p_a(q) on the q mesh (Eq. fofx and the text
// after it), M[j][a] (second derivative at q_j of p_a) in LDS.  On the
// interval j (a = (q_{j+1} - q)/h, b = 1 - a)
//   p_a  = a d_aj + b d_a,j+1 + ((a^3 - a) M[j][a] + (b^3 - b) M[j+1][a]) h^2/6
//   p_a' = (d_a,j+1 - d_aj)/h + ((1 - 3a^2) M[j][a] + (3b^2 - 1) M[j+1][a]) h/6
// and below q_1 the linear continuation p_a(q_1) + (q - q_1) p_a'(q_1).  Both
// are written p_a = A0 d_aj + A1 d_a,j+1 + C0 M[j][a] + C1 M[j+1][a] and
// p_a' = B0 d_aj + B1 d_a,j+1 + D0 M[j][a] + D1 M[j+1][a] with per-point
// scalars, so sums over a reduce to two dot products with rows of M.
template <typename T>
struct SplineW {
    int j;
    T A0, A1, C0, C1;
    T B0, B1, D0, D1;

    __device__ __forceinline__ void locate(T q0, const T *qm, int nq) {
        // one path for every case (the struct then stays in registers)
        const bool below = q0 < qm[0];
        int lo = 0, hi = nq - 1;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (qm[mid] <= q0) lo = mid; else hi = mid;
        }
        j = lo;
        const T ql = qm[lo], qh = qm[lo + 1];
        const T h = qh - ql, ih = rcp<T>(h), h6 = h * (T)(1.0 / 6.0);
        const T a = below ? (T)1 : (qh - q0) * ih;
        const T b = (T)1 - a;
        const T dq = below ? q0 - ql : (T)0;
        B0 = -ih;
        B1 = ih;
        D0 = ((T)1 - (T)3 * a * a) * h6;
        D1 = ((T)3 * b * b - (T)1) * h6;
        A0 = a + dq * B0;
        A1 = b + dq * B1;
        C0 = (a * a * a - a) * h * h6 + dq * D0;
        C1 = (b * b * b - b) * h * h6 + dq * D1;
    }
};

// q mesh, spline second derivatives and 1/m into LDS (in T); all loads are
// issued before any store (indices clamped, the stores guarded).  At least
// 128 threads.
template <typename T>
__device__ __forceinline__ void load_consts(const Consts *cst, T *qm, T *Mm, T *invm) {
    static_assert(kNQ * kNQ <= 4 * 128 && kNQ <= 128 && kMaxMc < 128, "four steps, one and one");
    const int i = threadIdx.x, nt = blockDim.x;
    const gptr<const double> q = gld(cst->q), M = gld(cst->M), im = gld(cst->invm);
    const double a = q[min(i, kNQ - 1)], c = im[min(i, kMaxMc)];
    double m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) m[u] = M[min(i + u * nt, kNQ * kNQ - 1)];
    if (i < kNQ) qm[i] = (T)a;
    if (i <= kMaxMc) invm[i] = (T)c;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (i + u * nt < kNQ * kNQ) Mm[i + u * nt] = (T)m[u];
}

// ---------------------------------------------------------------- axis-3 passes

// Axis-3 tiles: B whole rows, the 20 fields in pairs (theta_2m + i theta_2m+1,
// one complex line each), as split transforms in LDS.  Element n of a row
// (later slot (r, j), n = j + R2 r, and frequency slot (k1, k2)) holds its ten
// pair values contiguously: a point's thread moves them 16 bytes at a time, a
// transform item is one pair line, and ten lanes run along the pairs.  Each
// R2 elements are followed by a padding that keeps the lanes of neighbouring
// items on different banks.
// Compile-time radices (CR1 CR2 = the length; 0: run-time ones) turn the
// positions and strides of the common lengths into constants.
// Both passes are bound by vector ALU issue (0.85 and 0.92 of the cycles at
// 128^3 in FP32): the local chain, some 800 instructions a point.  Against whole lines in radix passes (theta, assembly,
// traced): 90 x 100 x 108 in FP32 87 -> 43 us and 90 -> 36, 96^3 39 -> 31 and
// 37 -> 31, 160 x 160 x 320 337 -> 265 and 330 -> 328; lost at two lengths that had
// compile-time plans: 128^3 60 -> 60 and 55 -> 66, sixteen 64^3 109 -> 130 and
// 117 -> 139.
template <typename T, int CR1, int CR2>
struct XTile {
    static constexpr int kP = kNQ / 2;                        // pair lines per row
    static constexpr int eb = kP * (int)sizeof(C2<T>);        // bytes per element
    const FftPlan &p;
    __device__ __forceinline__ explicit XTile(const FftPlan &p_) : p(p_) {}
    __device__ __forceinline__ int R1() const { if constexpr (CR1 > 0) return CR1; else return p.r1; }
    __device__ __forceinline__ int R2() const { if constexpr (CR1 > 0) return CR2; else return p.r2; }
    __device__ __forceinline__ int len() const { if constexpr (CR1 > 0) return CR1 * CR2; else return p.n; }
    __device__ __forceinline__ int by1(int x) const { if constexpr (CR1 > 0) return x / CR1; else return FastDiv{p.d1}(x); }
    __device__ __forceinline__ int by2(int x) const { if constexpr (CR1 > 0) return x / CR2; else return FastDiv{p.d2}(x); }
    __device__ __forceinline__ int byn(int x) const { if constexpr (CR1 > 0) return x / (CR1 * CR2); else return FastDiv{p.dn}(x); }
    __device__ __forceinline__ int gs() const { return __mul24(R2(), eb) + (__mul24(1 - R2(), eb) & 255); }   // bytes per R2 elements
    __device__ __forceinline__ int rs() const { return __mul24(R1(), gs()); }                            // and per row
    __device__ __forceinline__ int elem(int n) const { const int r = by2(n); return __mul24(r, gs()) + __mul24(n - __mul24(r, R2()), eb); }
    __device__ __forceinline__ int freq(int k) const { const int k2 = by1(k); return __mul24(k - __mul24(k2, R1()), gs()) + __mul24(k2, eb); }
};

// Both steps of the transform of a tile's B rows, in place: forward (S = -1)
// elements -> frequency slots, inverse (S = 1) back; tw: the length's table in
// LDS.  Synchronised by the caller before; synchronises between the steps and
// after.
template <typename T, int S, int RMAX, int CR1, int CR2>
__device__ __forceinline__ void xtile_fft(unsigned char *buf, const XTile<T, CR1, CR2> &X, int B, const C2<T> *tw) {
    constexpr int P = XTile<T, CR1, CR2>::kP;
    const int nt = blockDim.x;
    auto radix = [&](auto Cc, int r, auto &&f) {
        if constexpr (decltype(Cc)::value > 0) f(Cc);
        else with_radix<RMAX>(r, f);
    };
    auto one = [&]() {      // over r (or k1) at residue j
        for (int it = threadIdx.x; it < B * X.R2() * P; it += nt) {
            const int q = it / P, m = it - q * P, rb = X.by2(q), j = q - __mul24(rb, X.R2());
            unsigned char *lb = buf + __mul24(rb, X.rs()) + j * X.eb + m * (int)sizeof(C2<T>);
            radix(std::integral_constant<int, CR1>{}, X.R1(), [&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
                C2<T> x[R], w[R];
#pragma unroll
                for (int r = 0; r < R; ++r) x[r] = *reinterpret_cast<const C2<T> *>(lb + r * X.gs());
                Dft<T, R, S>::run(x);
                if (S < 0) lds_twiddles<T, S, R>(w, tw, j);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    *reinterpret_cast<C2<T> *>(lb + r * X.gs()) = (S > 0 || r == 0) ? x[r] : cmul(x[r], w[r - 1]);
            });
        }
        __syncthreads();
    };
    auto two = [&]() {      // over j (or k2) at k1
        for (int it = threadIdx.x; it < B * X.R1() * P; it += nt) {
            const int q = it / P, m = it - q * P, rb = X.by1(q), k1 = q - __mul24(rb, X.R1());
            unsigned char *lb = buf + __mul24(rb, X.rs()) + __mul24(k1, X.gs()) + m * (int)sizeof(C2<T>);
            radix(std::integral_constant<int, CR2>{}, X.R2(), [&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
                C2<T> x[R], w[R];
#pragma unroll
                for (int j = 0; j < R; ++j) x[j] = *reinterpret_cast<const C2<T> *>(lb + j * X.eb);
                Dft<T, R, S>::run(x);
                if (S > 0) lds_twiddles<T, S, R>(w, tw, k1);
#pragma unroll
                for (int j = 0; j < R; ++j)
                    *reinterpret_cast<C2<T> *>(lb + j * X.eb) = (S < 0 || j == 0) ? x[j] : cmul(x[j], w[j - 1]);
            });
        }
        __syncthreads();
    };
    if (S < 0) { one(); two(); }
    else { two(); one(); }
}

// theta_a = n p_a(q0) from n and the stored grad n, Delta E partials, R2C of
// the 20 theta rows.  tile: a = first row, b = rows, slot = partial.
template <typename T, int RMAX, int CR1, int CR2>
__global__ void __launch_bounds__(kMaxThreads, sizeof(T) == 8 ? 2 : RMAX <= 16 ? 5 : 4) k_x_theta(const InstDev *insts, const Tile *tiles, const Consts *cst,
                                                        const void *twv) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    const XTile<T, CR1, CR2> X(I.p3);
    const int N3 = X.len(), N3h = N3 / 2 + 1, row0 = t.a, B = t.b, nt = blockDim.x;
    const size_t N = (size_t)I.n1 * I.n2 * I.n3;
    C2<T> *tw = reinterpret_cast<C2<T> *>(smem + B * X.rs());
    T *qm = reinterpret_cast<T *>(tw + N3);
    T *Mm = qm + kNQ;
    T *invm = Mm + kNQ * kNQ;
    int *fo = reinterpret_cast<int *>(invm + kMaxMc + 1);     // (run-time radices) slot of every frequency
    // density and grad n of this thread's first point, fetched first (used
    // after the constants arrive); unconditional loads, clamped to the tile: a
    // load under a branch would be waited for where the branch joins
    const int npt = B * N3;
    const size_t p0 = (size_t)row0 * N3;
    const gptr<const T> nin = gld(reinterpret_cast<const T *>(I.n) + p0);
    const gptr<const T> gin = gld(reinterpret_cast<const T *>(I.grad) + p0);
    const int i_first = min((int)threadIdx.x, npt - 1);
    const T n_first = nin[i_first], gx_f = gin[i_first], gy_f = gin[N + i_first], gz_f = gin[2 * N + i_first];
    load_consts<T>(cst, qm, Mm, invm);
    load_twiddles<T>(tw, I.p3, reinterpret_cast<const C2<T> *>(twv));
    if (CR1 == 0)
        for (int k = threadIdx.x; k < N3; k += nt) fo[k] = X.freq(k);
    __syncthreads();

    const double c_qc = cst->qc, c_iqc = cst->iqc, c_cs = cst->cs, c_nmin = cst->nmin;
    const int c_mc = cst->mc;
    const bool semilocal = I.semilocal != 0;
    double de = 0.0, dex = 0.0, dec = 0.0;
    for (int idx = threadIdx.x; idx < npt; idx += nt) {
        const int rb = X.byn(idx), k = idx - __mul24(rb, N3);
        const bool first = idx == (int)threadIdx.x;
        const T nv = first ? n_first : nin[idx];
        const C2<T> g01 = mk<T>(first ? gx_f : gin[idx], first ? gy_f : gin[N + idx]);
        const C2<T> g2 = mk<T>(first ? gz_f : gin[2 * N + idx], (T)0);
        C2<T> *thc = reinterpret_cast<C2<T> *>(smem + __mul24(rb, X.rs()) + X.elem(k));   // the point's ten pairs
        // a density the method is not defined for (negative, NaN, infinite):
        // flag the grid (its energies come out NaN, the call reports it)
        if (!(nv >= (T)0 && nv <= finite_max<T>())) gst(I.bad)[0] = 1;
        if (nv >= (T)c_nmin) {
            LocalQ<T, false> lq;
            const T sigma = g01.x * g01.x + g01.y * g01.y + g2.x * g2.x;
            lq.eval(nv, sigma, c_qc, c_iqc, c_mc, invm);
            if (semilocal) {
                Semilocal<T> sl;
                sl.eval(nv, sigma, lq);
                dex += (double)sl.ex;
                dec += (double)sl.ec;
            }
            SplineW<T> sw;
            sw.locate(lq.q0, qm, kNQ);
            const T *Mj = Mm + sw.j * kNQ;
            const T nC0 = nv * sw.C0, nC1 = nv * sw.C1;
            // (16 bytes a store: lanes 80 or 160 bytes apart on different banks)
#pragma unroll
            for (int h = 0; h < kNQ / 2 / Chunk<T>::N; ++h) {
                C2<T> a[Chunk<T>::N];
#pragma unroll
                for (int q = 0; q < Chunk<T>::N; ++q) {
                    const int m = Chunk<T>::N * h + q;
                    a[q] = mk<T>(nC0 * Mj[2 * m] + nC1 * Mj[kNQ + 2 * m], nC0 * Mj[2 * m + 1] + nC1 * Mj[kNQ + 2 * m + 1]);
                }
                reinterpret_cast<typename Chunk<T>::V *>(thc)[h] = Chunk<T>::join(a);
            }
            // the interpolating parts A0 d_aj + A1 d_a,j+1 touch components j and
            // j + 1: rewrite the pair (j even) or the two pairs (j odd) that hold
            // them (same thread, so after the loop's stores)
            const int j0 = sw.j, m0 = j0 >> 1;
            const bool odd = (j0 & 1) != 0;
            const T nA0 = nv * sw.A0, nA1 = nv * sw.A1;
            const T *M0 = Mj + 2 * m0, *M1 = Mj + kNQ + 2 * m0;
            thc[m0] = mk<T>(nC0 * M0[0] + nC1 * M1[0] + (odd ? (T)0 : nA0), nC0 * M0[1] + nC1 * M1[1] + (odd ? nA0 : nA1));
            if (odd) thc[m0 + 1] = mk<T>(nC0 * M0[2] + nC1 * M1[2] + nA1, nC0 * M0[3] + nC1 * M1[3]);
            const T iq = rcp<T>(lq.q0);
            de += (double)((T)c_cs * nv * nv * iq * iq * iq);
        } else {
#pragma unroll
            for (int m = 0; m < kNQ / 2; ++m) thc[m] = mk<T>((T)0, (T)0);
        }
    }
    __syncthreads();
    xtile_fft<T, -1, RMAX, CR1, CR2>(smem, X, B, tw);

    // pair line m of row rb holds theta_{2m} + i theta_{2m+1}: its values at
    // k and N3 - k give both spectra at k, written together (item idx =
    // (rb N3h + k) 10 + m lands at spectrum element 2 idx)
    C2<T> *out = reinterpret_cast<C2<T> *>(I.spec) + (size_t)row0 * N3h * kNQ;
    auto by3h = [&](int x) { if constexpr (CR1 > 0) return x / (CR1 * CR2 / 2 + 1); else return FastDiv{I.dn3h}(x); };
    for (int idx = threadIdx.x; idx < B * N3h * (kNQ / 2); idx += nt) {
        const int q = idx / (kNQ / 2), m = idx - q * (kNQ / 2), rb = by3h(q), k = q - __mul24(rb, N3h);
        const unsigned char *Z = smem + __mul24(rb, X.rs()) + m * (int)sizeof(C2<T>);
        const int kc = k == 0 ? 0 : N3 - k;
        const C2<T> z = *reinterpret_cast<const C2<T> *>(Z + (CR1 > 0 ? X.freq(k) : fo[k]));
        const C2<T> zc = cconj(*reinterpret_cast<const C2<T> *>(Z + (CR1 > 0 ? X.freq(kc) : fo[kc])));
        const T ex = (z.x + zc.x) * (T)0.5, ey = (z.y + zc.y) * (T)0.5;
        const T ox = (z.y - zc.y) * (T)0.5, oy = -(z.x - zc.x) * (T)0.5;
        C2<T> *o = out + 2 * (size_t)idx;
        if constexpr (sizeof(T) == 4) gst(reinterpret_cast<float4 *>(o))[0] = make_float4(ex, ey, ox, oy);
        else { gst(o)[0] = mk<T>(ex, ey); gst(o)[1] = mk<T>(ox, oy); }
    }
    const double s = block_sum(de);
    double sx = 0.0, sc = 0.0;
    if (semilocal) {                 // (uniform over the workgroup)
        sx = block_sum(dex);
        sc = block_sum(dec);
    }
    if (threadIdx.x == 0) {
        I.part_de[t.slot] = s;
        I.part_sl[2 * t.slot] = sx;
        I.part_sl[2 * t.slot + 1] = sc;
    }
}

// The u spectra of B rows (axis 3 half spectra, [B][N3h][kNQ] complex at sp)
// into the frequency slots, ready for the inverse axis-3 FFT: u_{2m} + i u_{2m+1}
// of row rb, from the spectra at k (< N3/2 + 1) both the value at k and, by
// Hermitian symmetry, at N3 - k.  Item idx = (rb N3h + k) 10 + m reads spectrum
// elements 2 idx, 2 idx + 1; about five steps per thread: batches of six (four in FP64).
template <typename T, int CR1, int CR2>
__device__ __forceinline__ void u_lines_in(unsigned char *buf, const XTile<T, CR1, CR2> &X, const C2<T> *sp, int B,
                                           uint32_t dn3h) {
    constexpr int U = sizeof(T) == 4 ? 6 : 4, P = XTile<T, CR1, CR2>::kP;
    const int N3 = X.len(), N3h = N3 / 2 + 1;
    auto by3h = [&](int x) { if constexpr (CR1 > 0) return x / (CR1 * CR2 / 2 + 1); else return FastDiv{dn3h}(x); };
    const int total = B * N3h * P, nt = blockDim.x;
    const gptr<const C2<T>> g = gld(sp);
    for (int base = threadIdx.x; base < total; base += U * nt) {
        T ax[U], ay[U], bx[U], by[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = base + u * nt;
            const size_t e = idx < total ? 2 * (size_t)idx : 0;   // (unconditional loads)
            if constexpr (sizeof(T) == 4) {
                const float4 v = *(gptr<const float4>)(g + e);
                ax[u] = v.x; ay[u] = v.y; bx[u] = v.z; by[u] = v.w;
            } else {
                const C2<T> a = g[e], b = g[e + 1];
                ax[u] = a.x; ay[u] = a.y; bx[u] = b.x; by[u] = b.y;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = base + u * nt;
            if (idx >= total) continue;
            const int q = idx / P, m = idx - q * P, rb = by3h(q), k = q - __mul24(rb, N3h);
            unsigned char *Z = buf + __mul24(rb, X.rs()) + m * (int)sizeof(C2<T>);
            *reinterpret_cast<C2<T> *>(Z + X.freq(k)) = mk<T>(ax[u] - by[u], ay[u] + bx[u]);
            // conj(a) + i conj(b)
            if (k != 0 && 2 * k != N3) *reinterpret_cast<C2<T> *>(Z + X.freq(N3 - k)) = mk<T>(ax[u] + by[u], -ay[u] + bx[u]);
        }
    }
}

// C2R of the 20 u_a rows; v_loc = sum_a u_a dtheta_a/dn + de/dn;
// w = g grad n with g = sum_a u_a 2 n p'_a Q dq/dsigma + de/dsigma-part,
// stored in place of grad n as its lattice components q_c (the divergence
// passes take them).  tile: a = first row, b = rows.
template <typename T, int RMAX, int CR1, int CR2>
__global__ void __launch_bounds__(kMaxThreads, sizeof(T) == 8 ? (RMAX <= 16 || CR1 > 0 ? 3 : 2) : RMAX <= 16 ? 5 : 4) k_x_assemble(const InstDev *insts, const Tile *tiles, const Consts *cst,
                                                           const void *twv) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    const XTile<T, CR1, CR2> X(I.p3);
    const int N3 = X.len(), N3h = N3 / 2 + 1, row0 = t.a, B = t.b, nt = blockDim.x;
    const size_t N = (size_t)I.n1 * I.n2 * I.n3;
    C2<T> *tw = reinterpret_cast<C2<T> *>(smem + B * X.rs());
    T *qm = reinterpret_cast<T *>(tw + N3);
    T *Mm = qm + kNQ;
    T *invm = Mm + kNQ * kNQ;
    load_twiddles<T>(tw, I.p3, reinterpret_cast<const C2<T> *>(twv));
    // n and grad n of this thread's first point, fetched first (used after the FFT)
    const int npt = B * N3;
    const size_t p0 = (size_t)row0 * N3;
    const gptr<const T> nin = gld(reinterpret_cast<const T *>(I.n) + p0);
    const gptr<const T> grad = gld(reinterpret_cast<const T *>(I.grad) + p0);
    // (unconditional loads, clamped to the tile: a load under a branch would
    // be waited for where the branch joins)
    const int i_first = min((int)threadIdx.x, npt - 1);
    const T n_f = nin[i_first], gx_f = grad[i_first], gy_f = grad[N + i_first], gz_f = grad[2 * N + i_first];
    u_lines_in(smem, X, reinterpret_cast<const C2<T> *>(I.spec) + (size_t)row0 * N3h * kNQ, B, I.dn3h);
    load_consts<T>(cst, qm, Mm, invm);
    __syncthreads();
    xtile_fft<T, 1, RMAX, CR1, CR2>(smem, X, B, tw);

    const double c_qc = cst->qc, c_iqc = cst->iqc, c_cs = cst->cs, c_nmin = cst->nmin;
    const int c_mc = cst->mc;
    const bool semilocal = I.semilocal != 0;
    const gptr<T> vloc = gst(reinterpret_cast<T *>(I.vloc) + p0);
    for (int idx = threadIdx.x; idx < npt; idx += nt) {
        const int rb = X.byn(idx), k = idx - __mul24(rb, N3);
        const bool first = idx == (int)threadIdx.x;
        const T nv = first ? n_f : nin[idx];
        const T gx = first ? gx_f : grad[idx], gy = first ? gy_f : grad[N + idx], gz = first ? gz_f : grad[2 * N + idx];
        T vl = (T)0, gs = (T)0;
        if (nv >= (T)c_nmin) {
            LocalQ<T, true> lq;
            const T sigma = gx * gx + gy * gy + gz * gz;
            lq.eval(nv, sigma, c_qc, c_iqc, c_mc, invm);
            SplineW<T> sw;
            sw.locate(lq.q0, qm, kNQ);
            const T cn = nv * lq.Q * lq.dqdn;
            // sum_a u_a p_a and sum_a u_a p_a' through S0 = sum_a u_a M[j][a], S1 = sum_a u_a M[j+1][a]
            const T *Mj = Mm + sw.j * kNQ;
            T S0 = (T)0, S1 = (T)0;
            const C2<T> *uc = reinterpret_cast<const C2<T> *>(smem + __mul24(rb, X.rs()) + X.elem(k));   // the point's ten pairs
            const T *u = reinterpret_cast<const T *>(uc);
#pragma unroll
            for (int h = 0; h < kNQ / 2 / Chunk<T>::N; ++h) {
                C2<T> up[Chunk<T>::N];
                Chunk<T>::split(reinterpret_cast<const typename Chunk<T>::V *>(uc)[h], up);
#pragma unroll
                for (int q = 0; q < Chunk<T>::N; ++q) {
                    const int m = Chunk<T>::N * h + q;
                    S0 += up[q].x * Mj[2 * m] + up[q].y * Mj[2 * m + 1];
                    S1 += up[q].x * Mj[kNQ + 2 * m] + up[q].y * Mj[kNQ + 2 * m + 1];
                }
            }
            const int j0 = sw.j, j1 = sw.j + 1;
            const T uj = u[j0], uj1 = u[j1];
            const T su = sw.A0 * uj + sw.A1 * uj1 + sw.C0 * S0 + sw.C1 * S1;
            const T sdu = sw.B0 * uj + sw.B1 * uj1 + sw.D0 * S0 + sw.D1 * S1;
            // dtheta_a/dn = p_a + n p'_a Q dq/dn ; dtheta_a/dgrad n = 2 n p'_a Q dq/dsigma grad n
            const T q0 = lq.q0, cs = (T)c_cs;
            const T iq = rcp<T>(q0), iq3 = iq * iq * iq, iq4 = iq3 * iq;
            vl = su + cn * sdu + (T)2 * cs * nv * iq3 - (T)3 * cs * nv * nv * iq4 * lq.Q * lq.dqdn;
            gs = (T)2 * lq.Q * lq.ndqds * sdu - (T)6 * cs * nv * iq4 * lq.Q * lq.ndqds;
            if (semilocal) {
                // the semilocal terms: de/dgrad n = 2 de/dsigma grad n
                Semilocal<T> sl;
                sl.eval(nv, sigma, lq);
                vl += sl.dn;
                gs += (T)2 * sl.ds;
            }
        }
        vloc[idx] = vl;
        // the lattice components q_c = sum_x W[c][x] w_x of w in place of
        // grad n (each point is read and written by its own thread)
        const double gsd = (double)gs;
        const double wx = gsd * (double)gx, wy = gsd * (double)gy, wz = gsd * (double)gz;
        const gptr<T> wout = gst(reinterpret_cast<T *>(I.grad) + p0);
#pragma unroll
        for (int c = 0; c < 3; ++c)
            wout[c * N + idx] = (T)(I.fdW[c][0] * wx + I.fdW[c][1] * wy + I.fdW[c][2] * wz);
    }
}

// ---------------------------------------------------------------- finite-difference passes

// Central differences on the periodic grid in the working precision:
// d_c f_i = sum_s c_s (f_{i + s e_c} - f_{i - s e_c}), s = 1..M, along the grid
// (lattice) axis c; grad n = sum_c W[c] d_c n with W[c][x] = N_c b_c,x / (2 pi).
// Neighbour indices wrap once (M <= 4 <= every edge).  Tiles are runs of
// whole axis-3 lines: a = first row (i1 N2 + i2), b = rows.  Offsets are
// 32-bit (a grid and its three fields stay below 2^31 elements).

// offset of the neighbour s steps up (down) an axis of n points with element
// stride st from index i (one wrap at most)
__device__ __forceinline__ int fd_up(int i, int s, int n, int st) { return i + s < n ? s * st : (s - n) * st; }
__device__ __forceinline__ int fd_dn(int i, int s, int n, int st) { return i >= s ? -s * st : (n - s) * st; }

template <typename T, int M>
__device__ __forceinline__ T fd_diff(gptr<const T> f, int i, int n, int st, const T *c) {
    T acc = (T)0;
#pragma unroll
    for (int s = 1; s <= M; ++s) acc += c[s - 1] * (f[fd_up(i, s, n, st)] - f[fd_dn(i, s, n, st)]);
    return acc;
}

template <typename T, int M>
__device__ __forceinline__ void fd_grad_tile(const InstDev &I, int row0, int B) {
    const int N1 = I.n1, N2 = I.n2, N3 = I.n3;
    const int plane = N2 * N3, N = N1 * plane;
    const gptr<const T> n = gld(reinterpret_cast<const T *>(I.n));
    const gptr<T> g = gst(reinterpret_cast<T *>(I.grad));
    T c[M];
#pragma unroll
    for (int s = 0; s < M; ++s) c[s] = (T)I.fdc[s];
    T Wm[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int x = 0; x < 3; ++x) Wm[a][x] = (T)I.fdW[a][x];
    const int npt = B * N3;
    const int drow = kThreads / N3, dk = kThreads - drow * N3;
    int idx = threadIdx.x;
    if (idx >= npt) return;
    int rb = idx / N3, i3 = idx - rb * N3, row = row0 + rb;
    int i1 = row / N2, i2 = row - i1 * N2;
    for (; idx < npt; idx += kThreads) {
        const int p = row * N3 + i3;
        const gptr<const T> f = n + p;
        const T d1 = fd_diff<T, M>(f, i1, N1, plane, c);
        const T d2 = fd_diff<T, M>(f, i2, N2, N3, c);
        const T d3 = fd_diff<T, M>(f, i3, N3, 1, c);
#pragma unroll
        for (int a = 0; a < 3; ++a) g[a * N + p] = Wm[0][a] * d1 + Wm[1][a] * d2 + Wm[2][a] * d3;
        // next point: kThreads = drow N3 + dk further on
        i3 += dk;
        row += drow;
        i2 += drow;
        if (i3 >= N3) { i3 -= N3; ++row; ++i2; }
        while (i2 >= N2) { i2 -= N2; ++i1; }
    }
}

// v = v_loc - sum_c d_c q_c, q_c = sum_x W[c][x] w_x in the grad n buffer
// (Eq. (Vi): the sum over j of w_j . d(grad n_j)/dn_i is the transpose of the
// gradient operator applied to w, minus the same stencils since they are
// antisymmetric).
template <typename T, int M>
__device__ __forceinline__ void fd_div_tile(const InstDev &I, int row0, int B) {
    const int N1 = I.n1, N2 = I.n2, N3 = I.n3;
    const int plane = N2 * N3, N = N1 * plane;
    const gptr<const T> w = gld(reinterpret_cast<const T *>(I.grad));
    const gptr<const T> vloc = gld(reinterpret_cast<const T *>(I.vloc));
    const gptr<T> v = gst(reinterpret_cast<T *>(I.v));
    T c[M];
#pragma unroll
    for (int s = 0; s < M; ++s) c[s] = (T)I.fdc[s];
    const int npt = B * N3;
    const int drow = kThreads / N3, dk = kThreads - drow * N3;
    int idx = threadIdx.x;
    if (idx >= npt) return;
    int rb = idx / N3, i3 = idx - rb * N3, row = row0 + rb;
    int i1 = row / N2, i2 = row - i1 * N2;
    for (; idx < npt; idx += kThreads) {
        const int p = row * N3 + i3;
        const T d1 = fd_diff<T, M>(w + p, i1, N1, plane, c);
        const T d2 = fd_diff<T, M>(w + N + p, i2, N2, N3, c);
        const T d3 = fd_diff<T, M>(w + 2 * N + p, i3, N3, 1, c);
        v[p] = vloc[p] - (d1 + d2 + d3);
        i3 += dk;
        row += drow;
        i2 += drow;
        if (i3 >= N3) { i3 -= N3; ++row; ++i2; }
        while (i2 >= N2) { i2 -= N2; ++i1; }
    }
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_fd_grad(const InstDev *insts, const Tile *tiles) {
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    // (the grid's first pass: clear its bad-density flag before the theta pass)
    if (t.a == 0 && threadIdx.x == 0) gst(I.bad)[0] = 0;
    switch (I.fdm) {
        case 1: fd_grad_tile<T, 1>(I, t.a, t.b); break;
        case 2: fd_grad_tile<T, 2>(I, t.a, t.b); break;
        case 3: fd_grad_tile<T, 3>(I, t.a, t.b); break;
        case 4: fd_grad_tile<T, 4>(I, t.a, t.b); break;
        default: break;
    }
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_fd_div(const InstDev *insts, const Tile *tiles) {
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    switch (I.fdm) {
        case 1: fd_div_tile<T, 1>(I, t.a, t.b); break;
        case 2: fd_div_tile<T, 2>(I, t.a, t.b); break;
        case 3: fd_div_tile<T, 3>(I, t.a, t.b); break;
        case 4: fd_div_tile<T, 4>(I, t.a, t.b); break;
        default: break;
    }
}

// ---------------------------------------------------------------- per-axis spectral derivatives

// The spectral gradient of Eq. (Vi) multiplies the transform of n by i G_x,
// G = sum_c m_c b_c with the Nyquist index m_c = N_c/2 taken as zero: a sum
// of one-axis multipliers, so grad n = sum_c W[c] d_c n exactly, with d_c n
// = F_c^-1[i (2 pi m_c / N_c) F_c n] the derivative along grid axis c alone
// (in grid-index units; W[c][x] = N_c b_c,x / (2 pi)) and F_c the 1-D DFT
// along that axis; the divergence of the gradient term of v is likewise
// sum_c d_c q_c with q_c = sum_x W[c][x] w_x.  One pass per axis: pairs of
// real lines as one complex line (the one-axis operator is real), forward
// DFT, i kappa_m (Nyquist zero; the inverse's 1/N folded in), inverse DFT.
// MODE 0 (gradient, FP64 lines): n -> d_c n; MODE 1 (divergence, lines in
// the working precision): q_c -> the potential, v = v_loc - sum_c d_c q_c.

// The lines of a tile as split transforms (fft_split.hpp): step two of the
// forward transform, the factors i kappa_m and step two of the inverse stay in
// the registers of one item, so a line crosses LDS twice.  One kernel takes
// every axis (run-time strides), so the three independent gradient passes of
// an orthorhombic grid are one launch.  Bound by the latency of its few
// dependent steps on small grids, by memory on large ones (against lines held
// in LDS, traced: the three gradient directions together 41 -> 12 us at 96^3 and
// 84 -> 16 at 90 x 100 x 108 in FP32, 193 -> 81 at 160 x 160 x 320; the three
// divergence passes 39 -> 22, 77 -> 26 and 134 -> 80).  The FP32 gradient of the
// two largest classes does not fit its registers: 12 bytes a lane go to scratch
// in the class of radices to 20 and 64 in that to 27, in every direction of the
// launch (128 x 125 x 128: 54 -> 36 us all the same).
// tile: slot = axis (3, 2, 1); lanes = tile_lanes of the axis's R2.
//   axis 3: a = first row (i1 N2 + i2), b = rows (even, <= 2 << lanes; rows 2p, 2p+1
//     form line p).  MODE 0: grad[2] = W[2][2] d_3 n (orthorhombic) or d_3 n
//     (general cells: the axis-1 pass combines); the grid's first tile, it
//     also clears the bad-density flag.  MODE 1: v = v_loc - d_3 q_3 (q_3 in
//     grad[2]).
//   axes 2, 1 (lines along i2 at element stride N3, along i1 at N2 N3): a =
//     the other outer index (i1, or i2), b = first i3, c = number of
//     consecutive i3 (<= 2 << lanes; pairs form one line, an odd last one stands
//     alone).  MODE 0, axis 2: grad[1] = W[1][1] d_2 n (orthorhombic) or d_2 n
//     (general).  MODE 0, axis 1: grad[0] = W[0][0] d_1 n (orthorhombic);
//     general cells, where it runs after the others: grad n = sum_c W[c] d_c n
//     from d_1 n and the stored d_2 n, d_3 n, all three Cartesian components
//     written.  MODE 1: v -= d_c q_c (q_c in grad[axis - 1]).
template <typename T, typename C, int RMAX, int MODE>
__global__ void __launch_bounds__(kMaxThreads, 2) k_deriv(const InstDev *insts, const Tile *tiles, const void *twv) {
    extern __shared__ __align__(16) unsigned char smem[];
    C2<C> *buf = reinterpret_cast<C2<C> *>(smem);
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    const int axis = t.slot, ax = axis - 1;
    const FftPlan &pl = axis == 3 ? I.p3 : axis == 2 ? I.p2 : I.p1;
    const int L = pl.n, R1 = pl.r1, R2 = pl.r2, N3 = I.n3, lanes = tile_lanes(R2);
    const size_t N = (size_t)I.n1 * I.n2 * N3;
    const bool rows = axis == 3;
    if (MODE == 0 && rows && t.a == 0 && threadIdx.x == 0) gst(I.bad)[0] = 0;
    // element e of line l (its real part; the imaginary part pst further on)
    // at base + l lst + e est; LDS slot (k1, j) of line l at l ls + k1 ks + j js
    const int W = rows ? t.b : t.c, nl = (W + 1) / 2;
    const int est = rows ? 1 : axis == 2 ? N3 : I.n2 * N3;         // (32-bit offsets: 3 N < 2^31)
    const int lst = rows ? 2 * N3 : 2, pst = rows ? N3 : 1;
    const size_t base = rows ? (size_t)t.a * N3 : (axis == 2 ? (size_t)t.a * I.n2 * N3 : (size_t)t.a * N3) + t.b;
    const int js = rows ? 1 : 1 << lanes, ks = rows ? R2 | 1 : R2 << lanes, ls = rows ? R1 * ks : 1;
    const C2<C> *tw = reinterpret_cast<const C2<C> *>(twv) + pl.tw;
    // items: lanes run along the contiguous direction (residues of a row, or
    // lines of a column tile)
    const FastDiv by1{pl.d1}, by2{pl.d2};
    const int q1 = rows ? by2(threadIdx.x) : (int)threadIdx.x & ((1 << lanes) - 1);
    const int p1 = rows ? (int)threadIdx.x - q1 * R2 : (int)threadIdx.x >> lanes;
    const int q2 = rows ? by1(threadIdx.x) : q1, p2 = rows ? (int)threadIdx.x - q2 * R1 : p1;
    const bool on1 = q1 < nl && p1 < R2, on2 = q2 < nl && p2 < R1;
    const int gofs = q1 * lst + p1 * est, po = 2 * q1 + 1 < W ? pst : 0;
    typedef T pair_t __attribute__((ext_vector_type(2)));
    // pairs as one access where the row length and the pointer allow it
    auto pairable = [&](const void *ptr) { return !rows && ((N3 | W) & 1) == 0 && (reinterpret_cast<uintptr_t>(ptr) & (2 * sizeof(T) - 1)) == 0; };
    const T *src = MODE == 0 ? reinterpret_cast<const T *>(I.n) + base : reinterpret_cast<const T *>(I.grad) + ax * N + base;
    const bool vec = pairable(src);
    if (on1)
        with_radix<RMAX>(R1, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<C> w[R], x[R];
            T re[R], im[R];
            const gptr<const T> f = gld(src + gofs);
            if (vec) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const pair_t v = *(gptr<const pair_t>)(f + (size_t)(r * R2) * est);
                    re[r] = v.x;
                    im[r] = v.y;
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    re[r] = f[(size_t)(r * R2) * est];
                    im[r] = f[(size_t)(r * R2) * est + po];
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) x[r] = mk<C>((C)re[r], (C)im[r]);
            Dft<C, R, -1>::run(x);
            // (the factors after the transform: fetched before it they would
            // hold as many registers again)
            __builtin_amdgcn_sched_barrier(0);
            split_twiddles<C, -1, R>(w, tw, p1);
            C2<C> *o = buf + q1 * ls + p1 * js;
#pragma unroll
            for (int k = 0; k < R; ++k) o[k * ks] = k == 0 ? x[0] : cmul(x[k], w[k - 1]);
        });
    __syncthreads();
    if (on2)
        with_radix<RMAX>(R2, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<C> w[R], x[R];
            C2<C> *o = buf + q2 * ls + p2 * ks;
#pragma unroll
            for (int j = 0; j < R; ++j) x[j] = o[j * js];
            Dft<C, R, -1>::run(x);
            // frequency k = k1 + R1 k2 times i s 2 pi m / L^2
            const double k0 = 2.0 * 3.14159265358979323846 / ((double)L * (double)L) *
                              ((MODE == 0 && !I.general) ? I.fdW[ax][ax] : 1.0);
#pragma unroll
            for (int k2 = 0; k2 < R; ++k2) {
                const int k = p2 + R1 * k2;
                const int m = 2 * k == L ? 0 : (2 * k < L ? k : k - L);
                const C kap = (C)(k0 * (double)m);
                x[k2] = mk<C>(-kap * x[k2].y, kap * x[k2].x);
            }
            Dft<C, R, 1>::run(x);
            __builtin_amdgcn_sched_barrier(0);
            split_twiddles<C, 1, R>(w, tw, p2);
#pragma unroll
            for (int j = 0; j < R; ++j) o[j * js] = j == 0 ? x[0] : cmul(x[j], w[j - 1]);
        });
    // (the divergence's potential so far is fetched across the barrier)
    T *gout = reinterpret_cast<T *>(I.grad) + base + gofs;
    T *vout = reinterpret_cast<T *>(I.v) + base + gofs;
    const T *vin = rows ? reinterpret_cast<const T *>(I.vloc) + base + gofs : vout;
    const bool vvec = MODE == 1 && pairable(vout) && pairable(vin), gvec = MODE == 0 && pairable(gout - gofs + ax * N);
    __syncthreads();
    if (on1)
        with_radix<RMAX>(R1, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<C> x[R];
            T re[R], im[R];
            if constexpr (MODE == 1) {
                const gptr<const T> f = gld(vin);
                if (vvec) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const pair_t v = *(gptr<const pair_t>)(f + (size_t)(r * R2) * est);
                        re[r] = v.x;
                        im[r] = v.y;
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        re[r] = f[(size_t)(r * R2) * est];
                        im[r] = f[(size_t)(r * R2) * est + po];
                    }
                }
            }
            const C2<C> *o = buf + q1 * ls + p1 * js;
#pragma unroll
            for (int k = 0; k < R; ++k) x[k] = o[k * ks];
            Dft<C, R, 1>::run(x);
            if (MODE == 0 && axis == 1 && I.general) {
                // grad n = sum_c W[c] d_c n (the second value of a pair, then the first)
                for (int h = po ? 1 : 0; h >= 0; --h) {
                    const gptr<T> g = gst(gout + h * pst);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const size_t ofs = (size_t)(r * R2) * est;
                        const double d1 = (double)(h ? x[r].y : x[r].x), d2 = (double)g[N + ofs], d3 = (double)g[2 * N + ofs];
#pragma unroll
                        for (int c = 0; c < 3; ++c) g[c * N + ofs] = (T)(I.fdW[0][c] * d1 + I.fdW[1][c] * d2 + I.fdW[2][c] * d3);
                    }
                }
                return;
            }
            const gptr<T> out = gst(MODE == 0 ? gout + ax * N : vout);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                re[r] = MODE == 0 ? (T)x[r].x : re[r] - (T)x[r].x;
                im[r] = MODE == 0 ? (T)x[r].y : im[r] - (T)x[r].y;
            }
            if (MODE == 0 ? gvec : vvec) {
#pragma unroll
                for (int r = 0; r < R; ++r) *(gptr<pair_t>)(out + (size_t)(r * R2) * est) = pair_t{re[r], im[r]};
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    out[(size_t)(r * R2) * est] = re[r];
                    if (po) out[(size_t)(r * R2) * est + po] = im[r];
                }
            }
        });
}

// The same derivatives as direct sums, for grids whose edges are all at most
// kDenseMax: d f_i = sum_s w_s (f_{i+s} - f_{i-s}), s = 1 .. (N - 1)/2, the
// periodic sinc weights w_s = (pi/N) (-1)^(s+1) cot(pi s/N) (N even, its Nyquist
// term zero) or ... / sin(pi s/N) (N odd), the matrix of the spectral
// derivative row by row.  A point then needs its neighbours only, so all three
// axes are one launch: the gradient in any cell, and v = v_loc - sum_c d_c q_c,
// whose three passes each update v.  Small grids are bound by the number of
// dependent launches, not by these sums (24^3 in FP64: one pass of 10 us for
// three of 7, event-timed, 74 -> 69 us per evaluation).
// tile: a = first row (i1 N2 + i2), b = rows.
template <typename T, typename C>
__device__ __forceinline__ C dense_sum(gptr<const T> f, int i, int n, int st, const C *w) {
    constexpr int U = kDenseMax / 2;                           // (all terms' loads in flight)
    const int h = (n - 1) / 2;
    T up[U], dn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int s = min(u + 1, h);                           // (a step past the last repeats it, weight zero)
        up[u] = f[fd_up(i, s, n, st)];
        dn[u] = f[fd_dn(i, s, n, st)];
    }
    C acc = (C)0;
#pragma unroll
    for (int u = 0; u < U; ++u) acc += w[u + 1] * ((C)up[u] - (C)dn[u]);
    return acc;
}

template <typename T, typename C, int MODE>
__global__ void __launch_bounds__(kThreads) k_deriv_dense(const InstDev *insts, const Tile *tiles, const void *twv) {
    constexpr int H = 18;                                      // weights 1 .. h, then zeros
    __shared__ C w[3][H];
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    if (MODE == 0 && t.a == 0 && threadIdx.x == 0) gst(I.bad)[0] = 0;
    const C *tab = reinterpret_cast<const C *>(twv);
    if (threadIdx.x < 3 * H) {
        const int c = threadIdx.x / H, s = threadIdx.x - c * H;
        const FftPlan &pl = c == 0 ? I.p1 : c == 1 ? I.p2 : I.p3;
        const int h = (pl.n - 1) / 2;
        const C v = gld(tab)[pl.dw + min(max(s, 1), h) - 1];
        w[c][s] = s >= 1 && s <= h ? v : (C)0;
    }
    __syncthreads();
    const int N1 = I.n1, N2 = I.n2, N3 = I.n3, plane = N2 * N3, N = N1 * plane;
    const FastDiv by3{I.p3.dn}, by2{I.p2.dn};
    for (int idx = threadIdx.x; idx < t.b * N3; idx += blockDim.x) {
        const int rb = by3(idx), i3 = idx - rb * N3, row = t.a + rb;
        const int i1 = by2(row), i2 = row - i1 * N2, p = row * N3 + i3;
        const T *f = (MODE == 0 ? reinterpret_cast<const T *>(I.n) : reinterpret_cast<const T *>(I.grad)) + p;
        const C d1 = dense_sum<T, C>(gld(f), i1, N1, plane, w[0]);
        const C d2 = dense_sum<T, C>(gld(f + (MODE == 0 ? 0 : N)), i2, N2, N3, w[1]);
        const C d3 = dense_sum<T, C>(gld(f + (MODE == 0 ? 0 : 2 * N)), i3, N3, 1, w[2]);
        if constexpr (MODE == 0) {
            const gptr<T> g = gst(reinterpret_cast<T *>(I.grad) + p);
#pragma unroll
            for (int x = 0; x < 3; ++x) g[x * N] = (T)(I.fdW[0][x] * d1 + I.fdW[1][x] * d2 + I.fdW[2][x] * d3);
        } else {
            gst(reinterpret_cast<T *>(I.v))[p] = gld(reinterpret_cast<const T *>(I.vloc))[p] - (T)(d1 + d2 + d3);
        }
    }
}

// spectra of nl lines (length L, pitch ls) times i s 2 pi m / L^2
template <typename C>
__device__ __forceinline__ void deriv_multiply(C2<C> *buf, int nl, int L, int ls, double s) {
    const double k0 = 2.0 * 3.14159265358979323846 / ((double)L * (double)L) * s;
    for (int idx = threadIdx.x; idx < nl * L; idx += kThreads) {
        const int l = idx / L, m0 = idx - l * L;
        const int m = 2 * m0 == L ? 0 : (2 * m0 < L ? m0 : m0 - L);
        const C kap = (C)(k0 * (double)m);
        C2<C> &z = buf[l * ls + m0];
        z = mk<C>(-kap * z.y, kap * z.x);
    }
    __syncthreads();
}

// Axis 2 at a length without a split (the run-time radix passes).  tile: a =
// i1, b = first i3, c = number W of consecutive i3 (pairs form one complex
// line; an odd W's last line has a zero imaginary part).
template <typename T, typename C, int MODE>
__global__ void __launch_bounds__(kThreads) k_deriv_any(const InstDev *insts, const Tile *tiles, const void *twv) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    constexpr int c = 1;                                       // lattice axis (0-based)
    const int L = I.n2, lp = L | 1, Wc = t.c, np = (Wc + 1) / 2;
    const size_t N = (size_t)I.n1 * I.n2 * I.n3;
    const int stride = I.n3;                                   // (32-bit offsets: 3 N < 2^31)
    const size_t base = (size_t)t.a * I.n2 * I.n3 + t.b;
    C2<C> *tw = reinterpret_cast<C2<C> *>(smem);
    C2<C> *buf = tw + L;
    C *bc = reinterpret_cast<C *>(buf);                        // (re, im) of element e of line j / 2 at 2 ((j/2) lp + e) + j % 2
    const gptr<const T> f = gld(MODE == 0 ? reinterpret_cast<const T *>(I.n) + base
                                          : reinterpret_cast<const T *>(I.grad) + c * N + base);
    // element e of tile column j at f[e stride + j], flat index e Wc + j
    // (positions advanced without divisions: Wc is a runtime width); eight
    // unconditional loads in flight per lane
    const int total = L * Wc;
    {
        RowCursor cur(threadIdx.x, Wc);
        for (int base = threadIdx.x; base < total; base += 8 * kThreads) {
            C r[8];
            int o[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool on = base + u * kThreads < total;
                r[u] = (C)f[on ? cur.l * stride + cur.w : 0];
                o[u] = on ? 2 * ((cur.w >> 1) * lp + cur.l) + (cur.w & 1) : -1;
                cur.step();
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (o[u] >= 0) bc[o[u]] = r[u];
        }
    }
    if (Wc & 1)
        for (int e = threadIdx.x; e < L; e += kThreads) bc[2 * ((np - 1) * lp + e) + 1] = (C)0;
    load_twiddles<C>(tw, I.p2, reinterpret_cast<const C2<C> *>(twv));
    __syncthreads();
    fft_lines<C>(buf, I.p2, np, 1, lp, tw, -1);
    deriv_multiply<C>(buf, np, L, lp, (MODE == 0 && !I.general) ? I.fdW[c][c] : 1.0);
    fft_lines<C>(buf, I.p2, np, 1, lp, tw, 1);
    T *gbase = reinterpret_cast<T *>(I.grad) + base;
    if constexpr (MODE == 0) {
        RowCursor cur(threadIdx.x, Wc);
        for (int idx = threadIdx.x; idx < total; idx += kThreads, cur.step())
            gst(gbase)[c * N + (size_t)cur.l * stride + cur.w] = (T)bc[2 * ((cur.w >> 1) * lp + cur.l) + (cur.w & 1)];
    } else {
        const gptr<T> v = gst(reinterpret_cast<T *>(I.v) + base);
        RowCursor cur(threadIdx.x, Wc);
        for (int b0 = threadIdx.x; b0 < total; b0 += 4 * kThreads) {
            T r[4];
            int go[4], lo[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool on = b0 + u * kThreads < total;
                go[u] = on ? cur.l * stride + cur.w : -1;
                lo[u] = 2 * ((cur.w >> 1) * lp + cur.l) + (cur.w & 1);
                r[u] = v[on ? go[u] : 0];
                cur.step();
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (go[u] >= 0) v[go[u]] = r[u] - (T)bc[lo[u]];
        }
    }
}

// ---------------------------------------------------------------- axis-2 pass

// E_k = (Omega/2) sum of the axis-1 partials; Delta E = dOmega sum of the
// theta partials; E_x, E_c^LDA = dOmega sums of the semilocal partials (zero
// unless the semilocal terms are on), into I.E[0..3]: NaN for a density the
// theta pass flagged.  One workgroup, 256 running sums whatever its size (so
// the summation order is the grid's own), eight loads in flight each.  These
// are the first workgroups of the inverse axis-2 pass, beside its tiles: as a
// launch of its own at the end, one workgroup a grid with one load in flight
// per lane, the reduction took 3 us on 24^3, 18 us on 128^3 and 70 us on
// 160 x 160 x 320.
__device__ __forceinline__ void reduce_energies(const InstDev &I, double *acc) {
    constexpr int V = 256, U = 8;
    const int nt = blockDim.x, nq = I.semilocal ? 4 : 2;
    for (int q = 0; q < nq; ++q) {
        const int n = q == 0 ? I.n_ek : I.n_de, st = q < 2 ? 1 : 2;
        const gptr<const double> p = gld(q == 0 ? I.part_ek : q == 1 ? I.part_de : I.part_sl + (q - 2));
        for (int v = threadIdx.x; v < V; v += nt) {
            double a = 0.0;
            for (int i = v; i < n; i += U * V) {
                double r[U];
#pragma unroll
                for (int u = 0; u < U; ++u) r[u] = p[(size_t)min(i + u * V, n - 1) * st];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (i + u * V < n) a += r[u];
            }
            acc[q * V + v] = a;
        }
    }
    for (int h = V / 2; h > 0; h >>= 1) {
        __syncthreads();
        for (int i = threadIdx.x; i < h * nq; i += nt) {
            const int q = i / h, v = i - q * h;
            acc[q * V + v] += acc[q * V + v + h];
        }
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        const double w = q == 0 ? 0.5 * I.omega : I.dvol;
        gst(I.E)[q] = gld(I.bad)[0] != 0 ? __builtin_nan("") : q < nq ? w * acc[q * V] : 0.0;
    }
}

// The 20 spectra along axis 2, lengths that split into two radices.  A tile is
// kYC (16 or 8) 16-byte chunks of every row i2 of one plane:
// step one loads its rows straight into registers (R1 16-byte loads in
// flight per lane), step two stores its rows straight from them, and the
// lines cross LDS once, conflict-free (lanes on consecutive chunks).  The
// pass is bound by memory; crossing LDS at both ends and between the radix
// passes, with divisions by run-time lengths outside eight lengths, had held
// it below (the forward pass, traced: 96^3 in FP32 46 -> 24 us, in FP64 73 -> 44,
// 90 x 100 x 108 60 -> 27, 160 x 160 x 320 327 -> 253).
// tile: a = i1, b = first chunk of the row, c = chunks (<= kYC; the lanes
// past them repeat the last one and store nothing); a < 0 (inverse pass only):
// the grid's energies.
template <typename T, int S, int RMAX>
__global__ void __launch_bounds__(kMaxThreads) k_y(const InstDev *insts, const Tile *tiles,
                                                                    const void *twv) {
    extern __shared__ __align__(16) unsigned char smem[];
    using K = Chunk<T>;
    using V = typename K::V;
    constexpr int kYC = 1 << tile_lanes(RMAX);
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    if (S > 0 && t.a < 0) {
        reduce_energies(I, reinterpret_cast<double *>(smem));
        return;
    }
    const int R1 = I.p2.r1, R2 = I.p2.r2;
    const size_t rowc = (size_t)I.n3h * (kNQ / K::N);          // chunks per row
    const int c = threadIdx.x % kYC, p = threadIdx.x / kYC;
    V *g = reinterpret_cast<V *>(I.spec) + (size_t)t.a * I.n2 * rowc + t.b + min(c, t.c - 1);
    V *lds = reinterpret_cast<V *>(smem) + c;
    const C2<T> *tw = reinterpret_cast<const C2<T> *>(twv) + I.p2.tw;
    if (p < R2)
        with_radix<RMAX>(R1, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<T> w[R], x[K::N][R];
            V in[R];
            split_twiddles<T, S, R>(w, tw, p);
#pragma unroll
            for (int r = 0; r < R; ++r) in[r] = gld(g + (size_t)(p + r * R2) * rowc)[0];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                C2<T> a[K::N];
                K::split(in[r], a);
#pragma unroll
                for (int q = 0; q < K::N; ++q) x[q][r] = a[q];
            }
#pragma unroll
            for (int q = 0; q < K::N; ++q) Dft<T, R, S>::run(x[q]);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                C2<T> a[K::N];
#pragma unroll
                for (int q = 0; q < K::N; ++q) a[q] = k == 0 ? x[q][0] : cmul(x[q][k], w[k - 1]);
                lds[(k * R2 + p) * kYC] = K::join(a);
            }
        });
    __syncthreads();
    if (p < R1)
        with_radix<RMAX>(R2, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<T> x[K::N][R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                C2<T> a[K::N];
                K::split(lds[(p * R + j) * kYC], a);
#pragma unroll
                for (int q = 0; q < K::N; ++q) x[q][j] = a[q];
            }
#pragma unroll
            for (int q = 0; q < K::N; ++q) Dft<T, R, S>::run(x[q]);
            if (c < t.c) {
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    C2<T> a[K::N];
#pragma unroll
                    for (int q = 0; q < K::N; ++q) a[q] = x[q][k];
                    gst(g + (size_t)(p + k * R1) * rowc)[0] = K::join(a);
                }
            }
        });
}

// The same for any other length (the run-time radix passes).  tile: a = i1,
// b = first flattened (k3, component) index, c = width
template <typename T, int S>
__global__ void __launch_bounds__(kThreads) k_y_any(const InstDev *insts, const Tile *tiles, const void *twv) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    if (S > 0 && t.a < 0) {
        reduce_energies(I, reinterpret_cast<double *>(smem));
        return;
    }
    const int N2 = I.n2, W = t.c, lp = N2 | 1;                 // lines contiguous, odd pitch
    C2<T> *tw = reinterpret_cast<C2<T> *>(smem);
    C2<T> *buf = tw + N2;
    const size_t rowlen = (size_t)I.n3h * kNQ;
    C2<T> *g = reinterpret_cast<C2<T> *>(I.spec) + (size_t)t.a * N2 * rowlen + t.b;
    rows_in_t(buf, lp, g, rowlen, N2, W);
    load_twiddles<T>(tw, I.p2, reinterpret_cast<const C2<T> *>(twv));
    __syncthreads();
    fft_lines<T>(buf, I.p2, W, 1, lp, tw, S);
    rows_out_t(g, rowlen, buf, lp, N2, W);
}

// ---------------------------------------------------------------- axis-1 passes

// How the fused axis-1 pass forms u = phi c: on the vector ALU or the matrix
// cores (FP32) in orthorhombic cells, where the points +-m1 of the columns k2
// and N2 - k2 share a kernel matrix; in general cells a matrix per k point,
// as full rows or packed upper triangles, on the vector ALU.
enum Contraction { CT_VEC = 0, CT_MFMA = 1, CT_GEN = 2, CT_GEN_PACKED = 3 };

// Waves per SIMD the fused pass is compiled for: what the LDS of its common
// tiles lets stand on a CU.  With packed rows the 20 offsets per lane do not
// fit the 128 registers of four waves beside a DFT of 16: 16 values went to
// scratch, and a lone triclinic FP32 grid's pass took 421 us at 128^3 and 522 at
// 160 x 128 x 128 instead of 396 and 499 with three.
template <typename T, int CT, int RMAX>
constexpr int zmain_waves() {
    if (sizeof(T) == 8) return 1;
    if (RMAX <= 16) return CT == CT_GEN_PACKED && RMAX > 10 ? 3 : 4;
    return RMAX <= 20 ? 3 : 2;
}

// Forward axis-1 FFT of the 20 theta spectra, u_a(G) = sum_b phi_ab(|G|) c_b(G)
// with c = Theta / N (Eq. Eoffk, Eq. epsofk), the energy sum
// sum_G w_G sum_a Re(c_a^* u_a), inverse axis-1 FFT.
// tile: a = first entry in the column list, b = items per |m1| (P: 1 or 2
// consecutive k3), c = columns per item (CP: 2 = k2 and N2 - k2, which meet the
// same |G| shell at every (|m1|, k3), then P = 1; else 1).  The list holds
// the tile's P CP <= 2 columns.
//
// The transforms are split ones (fft_split.hpp): the tile's rows (plane i1,
// 160 bytes per column in FP32) go between global memory and registers in
// 16-byte chunks, and LDS holds slot k1 R2 + j (later k1 R2 + k2, the
// frequency k1 + R1 k2) with the tile's components contiguous, so every step
// moves whole chunks, 16 bytes a lane, and works in place: four barriers in
// all.  A padding after each R2 slots keeps the lanes of neighbouring items on
// different banks.  The contraction reads the 20 components of a point as
// contiguous chunks too.  (The radix passes it replaces crossed LDS in words
// of 8 bytes, at both ends and in every pass: the fused pass, traced, went from
// 92 to 55 us at 96^3 in FP32 and from 158 to 127 in FP64, from 162 to 70 at
// 90 x 100 x 108, from 160 to 122 at 128^3, and from 20 to 10 at 24^3 in FP64; with
// packed kernel rows a lone 128^3 triclinic grid stands where it did, at 405.)
//
// Contraction layout (vector ALU): lanes form groups of kNQ (three per wave).
// A group takes one item, a |m1| and a column or pair; lane a loads row a of
// that shell's kernel matrix (kNQ contiguous values, 16-byte loads) into
// registers and forms u_a at the item's points (+-m1 of each column).  The
// rows of the group's next item are loaded meanwhile (two register sets in
// turn).  CT_GEN: every item is one k point with its own shell; lane a loads
// row a of its full matrix, or (packed) gathers the row through offsets fixed
// per lane.
// probe (parity probes of the stages, never in an evaluation): 1 writes the
// forward spectra c = FFT(theta)/N back in place of the tile (no contraction,
// no inverse); 2 writes u = phi c (no inverse); 0 is the evaluation.
template <typename T, int CT, int RMAX>
__global__ void __launch_bounds__(kMaxThreads, (zmain_waves<T, CT, RMAX>()))
k_z_main(const InstDev *insts, const Tile *tiles, const int2 *cols, const void *twv, int probe) {
    extern __shared__ __align__(16) unsigned char smem[];
    using Ch = Chunk<T>;
    using V = typename Ch::V;
    constexpr bool GEN = CT == CT_GEN || CT == CT_GEN_PACKED, PK = CT == CT_GEN_PACKED, MF = CT == CT_MFMA;
    static_assert(!MF || sizeof(T) == 4, "matrix-core contraction: FP32");
    constexpr int kCpc = kNQ / Ch::N;                          // chunks per column
    constexpr int kColB = kNQ * (int)sizeof(C2<T>);            // bytes per column of a slot
    const Tile t = tiles[blockIdx.x];
    const InstDev &I = insts[t.inst];
    const int N1 = I.n1, N2 = I.n2, N3 = I.n3, N3h = I.n3h, P = t.b, CP = t.c, K = P * CP;
    const int R1 = I.p1.r1, R2 = I.p1.r2;
    // the grid's own thread count (a launch has the largest of its grids'): the
    // items of a thread, so the order of the energy sum, do not depend on the
    // other grids of a batch; threads past it take no items
    const int nt = I.zthreads, tid = (int)threadIdx.x < nt ? (int)threadIdx.x : 1 << 28;
    const int C = K * kCpc;                                    // chunks per slot
    const int sb = K * kColB;                                  // bytes per slot
    const int s1 = R2 * sb + (((1 - R2) * sb) & 255);          // bytes per R2 slots: lanes C apart go on where C stop
    unsigned char *buf = smem;
    int *soff = reinterpret_cast<int *>(smem + R1 * s1);       // slot offset of frequency k
    int *sidx = soff + N1;                                     // shell of every item
    const int2 c0 = cols[t.a], c1 = cols[t.a + K - 1];
    const C2<T> *tw = reinterpret_cast<const C2<T> *>(twv) + I.p1.tw;
    const size_t plane = (size_t)N2 * N3h * kNQ;               // complex values
    C2<T> *spec = reinterpret_cast<C2<T> *>(I.spec);
    C2<T> *col0 = spec + (size_t)(c0.x * N3h + c0.y) * kNQ, *col1 = spec + (size_t)(c1.x * N3h + c1.y) * kNQ;
    // orthorhombic cell: item = |m1| P + pr, the +-m1 points share a shell;
    // general cell: item = k1 P + pr over the whole axis, a shell each
    const int k30 = c0.y, m2 = GEN ? c0.x : freq_abs(c0.x, N2);
    const int nitems = (GEN ? N1 : N1 / 2 + 1) * P;
    const gptr<const int> smap = gld(I.shellmap + (size_t)m2 * N3h + k30);
    const size_t smap_m1 = (size_t)(GEN ? N2 : I.h2) * N3h;
    // the thread's first shell index is loaded before the tile (clamped,
    // unconditional) and stored after it
    auto smap_at = [&](int i) { return smap[(size_t)(i >> (P - 1)) * smap_m1 + (i & (P - 1))]; };
    const int sh_first = smap_at(min(tid, nitems - 1));

    const FastDiv byC{K == 2 ? div_magic(2 * kCpc) : div_magic(kCpc)}, byR1{I.p1.d1};
    // step one of the forward transform: rows -> registers -> slots
    for (int it = tid; it < C * R2; it += nt) {
        const int p = byC(it), c = it - __mul24(p, C), w = c / kCpc, e = c - w * kCpc;
        const V *g = reinterpret_cast<const V *>((w ? col1 : col0) + (size_t)p * plane) + e;
        unsigned char *lb = buf + __mul24(p, sb) + c * 16;
        const size_t step = (size_t)R2 * plane * sizeof(C2<T>);
        with_radix<RMAX>(R1, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<T> tf[R], x[Ch::N][R];
            V in[R];
            split_twiddles<T, -1, R>(tf, tw, p);
#pragma unroll
            for (int r = 0; r < R; ++r) in[r] = gld(reinterpret_cast<const V *>(reinterpret_cast<const char *>(g) + r * step))[0];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                C2<T> a[Ch::N];
                Ch::split(in[r], a);
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) x[q][r] = a[q];
            }
#pragma unroll
            for (int q = 0; q < Ch::N; ++q) Dft<T, R, -1>::run(x[q]);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                C2<T> a[Ch::N];
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) a[q] = k == 0 ? x[q][0] : cmul(x[q][k], tf[k - 1]);
                *reinterpret_cast<V *>(lb + k * s1) = Ch::join(a);
            }
        });
    }
    for (int k = tid; k < N1; k += nt) {
        const int q = byR1(k);
        soff[k] = (k - q * R1) * s1 + q * sb;
    }
    if (tid < nitems) sidx[tid] = sh_first;
    for (int i = tid + nt; i < nitems; i += nt) sidx[i] = smap_at(i);

    const int lane = threadIdx.x & 63, wave = tid >> 6, ngroups = (nt >> 6) * (64 / kNQ);
    const int grp = lane / kNQ, al = lane - grp * kNQ;
    const bool lane_on = grp < 64 / kNQ;
    const int gid = wave * (64 / kNQ) + grp;
    // (packed rows: entry (r, q), r <= q, at r kNQ - r (r - 1)/2 + q - r)
    int poff[PK ? kNQ : 1];
    if constexpr (PK) {
#pragma unroll
        for (int b = 0; b < kNQ; ++b) {
            const int r = min(al, b), q = max(al, b);
            poff[b] = r * kNQ - ((r * (r - 1)) >> 1) + q - r;
        }
    }
    // the kernel-matrix row this lane holds: a of its group (vector ALU), or
    // 4 rb + (lane % 4) of its block (matrix cores, below)
    const int mf_blk = lane >> 2, mf_q = lane & 3;
    const bool mf_on = mf_blk < 15;
    const int mf_g = mf_on ? mf_blk / 5 : 2;
    const int mf_rb = mf_on ? mf_blk - (mf_blk / 5) * 5 : 0;
    const int row = MF ? 4 * mf_rb + mf_q : al;
    const T *tab = reinterpret_cast<const T *>(I.shelltab);
    // row `row` of the shell matrix of an item (index clamped to the last
    // item: the loads stay unconditional)
    auto fetch = [&](int item, T *f) {
        const int sh = sidx[min(item, nitems - 1)];
        if constexpr (PK) {
            const gptr<const T> src = gld(tab + (size_t)sh * kTabPacked);
#pragma unroll
            for (int b = 0; b < kNQ; ++b) f[b] = src[poff[b]];
        } else {
            const gptr<const V> src = gld(reinterpret_cast<const V *>(tab + (size_t)sh * kTabRow + row * kNQ));
            constexpr int E = 16 / (int)sizeof(T);
#pragma unroll
            for (int q = 0; q < kNQ / E; ++q) {
                const V v = src[q];
                if constexpr (sizeof(T) == 4) { f[4 * q] = v.x; f[4 * q + 1] = v.y; f[4 * q + 2] = v.z; f[4 * q + 3] = v.w; }
                else { f[2 * q] = v.x; f[2 * q + 1] = v.y; }
            }
        }
    };
    __syncthreads();
    // kernel rows in flight: one item (vector ALU) or round (matrix cores)
    // ahead, the first before step two
    T fa[kNQ], fb[kNQ];
    const int it0 = MF ? wave * (64 / kNQ) + mf_g : gid;
    if (MF || lane_on) fetch(it0, fa);
    // step two: the slots of (chunk, k1), in place
    for (int it = tid; it < C * R1; it += nt) {
        const int p = byC(it), c = it - __mul24(p, C);
        unsigned char *lb = buf + __mul24(p, s1) + c * 16;
        with_radix<RMAX>(R2, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<T> x[Ch::N][R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                C2<T> a[Ch::N];
                Ch::split(*reinterpret_cast<const V *>(lb + j * sb), a);
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) x[q][j] = a[q];
            }
#pragma unroll
            for (int q = 0; q < Ch::N; ++q) Dft<T, R, -1>::run(x[q]);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                C2<T> a[Ch::N];
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) a[q] = x[q][k];
                *reinterpret_cast<V *>(lb + k * sb) = Ch::join(a);
            }
        });
    }
    __syncthreads();

    // (probes) the tile's spectrum to its rows
    auto store_spectrum = [&](T scale) {
        for (int it = tid; it < C * N1; it += nt) {
            const int k = byC(it), c = it - __mul24(k, C), w = c / kCpc, e = c - w * kCpc;
            C2<T> a[Ch::N];
            Ch::split(*reinterpret_cast<const V *>(buf + soff[k] + c * 16), a);
            for (int q = 0; q < Ch::N; ++q) a[q] = cscale(a[q], scale);
            gst(reinterpret_cast<V *>((w ? col1 : col0) + (size_t)k * plane) + e)[0] = Ch::join(a);
        }
    };
    const T inv_n = (T)I.inv_n;
    if (probe == 1) {
        store_spectrum(inv_n);
        if (threadIdx.x == 0) I.part_ek[t.slot] = 0.0;
        return;
    }
    const double wn = (double)inv_n * (double)inv_n;
    double e = 0.0;
    auto weight = [&](int k3) { return (k3 == 0 || ((N3 & 1) == 0 && 2 * k3 == N3)) ? wn : 2.0 * wn; };
    if constexpr (MF) {
        // Matrix cores: v_mfma_f32_4x4x1_16b_f32 forms 16 independent 4 x 4
        // outer products per instruction (A 4 x 1 and B 1 x 4 per block,
        // accumulated over K).  A wave takes the three items its three lane
        // groups take on the vector path.  Block k = lane / 4 (15 of the 16
        // in use): item g = k / 5 of the three, rows 4 rb .. 4 rb + 3 of its
        // kernel matrix (rb = k % 5).  Lane 4 k + i feeds A = row 4 rb + i of
        // the matrix (20 values in registers, one per K step b) and B =
        // theta_b at column i % 2 of the item's pair and point i / 2 (+m1 or
        // -m1), real and imaginary parts in two chains (the kernel is real);
        // it receives in its four accumulators u_{4 rb + r}, r = 0..3, at that
        // column and point.  An item of one column (k2 = 0 and N2/2) gives
        // both lanes of a point the same column (the same values written
        // twice).  The lanes of a wave read theta before any of them writes u
        // (wave-level ordering), as on the vector path.
        typedef float v4f __attribute__((ext_vector_type(4)));
        const int g0 = wave * (64 / kNQ);
        int it = g0 + mf_g;
        const float fin = (float)I.inv_n;
        auto process_mf = [&](const T *f) {
            const bool valid = mf_on && it < nitems;
            const int l = valid ? it >> (P - 1) : 0, pg = it & (P - 1);   // (an item past the end reads point 0)
            int lq = N1 - l;
            const bool two = !(l == 0 || lq == l);
            if (!two) lq = l;
            const double wgt = (valid && (mf_q < 2 || two) && (CP == 2 || !(mf_q & 1))) ? weight(k30 + pg) : 0.0;
            it += ngroups;
            unsigned char *xc = buf + soff[mf_q < 2 ? l : lq] + (CP == 2 ? mf_q & 1 : pg) * kColB;
            float4 *oc = reinterpret_cast<float4 *>(xc + 4 * mf_rb * (int)sizeof(C2<T>));
            // every LDS read of the round before the first product (one
            // wait instead of one per K step)
            float4 th[kNQ / 2];
#pragma unroll
            for (int b = 0; b < kNQ / 2; ++b) th[b] = reinterpret_cast<const float4 *>(xc)[b];
            const float4 o0 = oc[0], o1 = oc[1];
            __builtin_amdgcn_sched_barrier(0);
            v4f are = {0.f, 0.f, 0.f, 0.f}, aim = are;
#pragma unroll
            for (int b = 0; b < kNQ / 2; ++b) {
                are = __builtin_amdgcn_mfma_f32_4x4x1f32(f[2 * b], th[b].x, are, 0, 0, 0);
                aim = __builtin_amdgcn_mfma_f32_4x4x1f32(f[2 * b], th[b].y, aim, 0, 0, 0);
                are = __builtin_amdgcn_mfma_f32_4x4x1f32(f[2 * b + 1], th[b].z, are, 0, 0, 0);
                aim = __builtin_amdgcn_mfma_f32_4x4x1f32(f[2 * b + 1], th[b].w, aim, 0, 0, 0);
            }
            const float es = o0.x * are[0] + o0.y * aim[0] + o0.z * are[1] + o0.w * aim[1] +
                             o1.x * are[2] + o1.y * aim[2] + o1.z * are[3] + o1.w * aim[3];
            e += wgt * (double)es;
            wave_sync();
            if (valid) {
                oc[0] = make_float4(are[0] * fin, aim[0] * fin, are[1] * fin, aim[1] * fin);
                oc[1] = make_float4(are[2] * fin, aim[2] * fin, are[3] * fin, aim[3] * fin);
            }
        };
        // rounds of three items per wave, the loop bound uniform over the wave
        for (int base = g0; base < nitems; base += 2 * ngroups) {
            fetch(it + ngroups, fb);               // the next round's row (clamped past the end)
            process_mf(fa);
            if (base + ngroups >= nitems) break;
            fetch(it + ngroups, fa);
            process_mf(fb);
        }
    } else {
        // u at the points of item `it` with the kernel row f; a group's lanes
        // share one wave, so reads of theta and writes of u need wave-level
        // ordering only
        auto process = [&](int it, const T *f) {
            // the points +-m1 of each column of the item (lq = l for k1 = 0 and
            // the Nyquist plane: the second point is the first again, its
            // energy masked and its u the same value written twice); one
            // point in general cells
            const int l = it >> (P - 1), pr = it & (P - 1);
            int lq = N1 - l;
            const bool two = !(GEN || l == 0 || lq == l);
            if (!two) lq = l;
            const T mask2 = two ? (T)1 : (T)0;
            const double wgt = weight(k30 + pr);
            const int o1 = soff[l], o2 = soff[lq];
            auto column = [&](int w) {
                C2<T> u1 = mk<T>((T)0, (T)0), u2 = u1;
                C2<T> *x1 = reinterpret_cast<C2<T> *>(buf + o1 + w * kColB), *x2 = reinterpret_cast<C2<T> *>(buf + o2 + w * kColB);
#pragma unroll
                for (int b = 0; b < kCpc; ++b) {
                    C2<T> t1[Ch::N], t2[Ch::N];
                    Ch::split(reinterpret_cast<const V *>(x1)[b], t1);
                    if (!GEN) Ch::split(reinterpret_cast<const V *>(x2)[b], t2);
#pragma unroll
                    for (int q = 0; q < Ch::N; ++q) {
                        u1.x += f[Ch::N * b + q] * t1[q].x;
                        u1.y += f[Ch::N * b + q] * t1[q].y;
                        if (!GEN) {
                            u2.x += f[Ch::N * b + q] * t2[q].x;
                            u2.y += f[Ch::N * b + q] * t2[q].y;
                        }
                    }
                }
                const C2<T> own1 = x1[al];
                T es = own1.x * u1.x + own1.y * u1.y;
                if (!GEN) {
                    const C2<T> own2 = x2[al];
                    es += mask2 * (own2.x * u2.x + own2.y * u2.y);
                }
                e += wgt * (double)es;
                // every lane of the group has read theta at these points before
                // any lane overwrites its component with u; the next column or
                // item reads other points (each k point belongs to one item),
                // so no ordering is needed after the writes
                wave_sync();
                x1[al] = cscale(u1, inv_n);
                if (!GEN) x2[al] = cscale(u2, inv_n);
            };
            column(CP == 2 ? 0 : pr);
            if (CP == 2) column(1);
        };
        for (int it = gid; lane_on && it < nitems;) {
            fetch(it + ngroups, fb);               // the next item's row (clamped past the end)
            process(it, fa);
            it += ngroups;
            if (it >= nitems) break;
            fetch(it + ngroups, fa);
            process(it, fb);
            it += ngroups;
        }
    }
    __syncthreads();
    if (probe == 2) {
        store_spectrum((T)1);
        return;
    }
    // the inverse transform: step two backwards, in place
    for (int it = tid; it < C * R1; it += nt) {
        const int p = byC(it), c = it - __mul24(p, C);
        unsigned char *lb = buf + __mul24(p, s1) + c * 16;
        with_radix<RMAX>(R2, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<T> tf[R], x[Ch::N][R];
            split_twiddles<T, 1, R>(tf, tw, p);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                C2<T> a[Ch::N];
                Ch::split(*reinterpret_cast<const V *>(lb + k * sb), a);
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) x[q][k] = a[q];
            }
#pragma unroll
            for (int q = 0; q < Ch::N; ++q) Dft<T, R, 1>::run(x[q]);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                C2<T> a[Ch::N];
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) a[q] = j == 0 ? x[q][0] : cmul(x[q][j], tf[j - 1]);
                *reinterpret_cast<V *>(lb + j * sb) = Ch::join(a);
            }
        });
    }
    __syncthreads();
    // and step one: slots -> registers -> rows
    for (int it = tid; it < C * R2; it += nt) {
        const int p = byC(it), c = it - __mul24(p, C), w = c / kCpc, q0 = c - w * kCpc;
        V *g = reinterpret_cast<V *>((w ? col1 : col0) + (size_t)p * plane) + q0;
        const unsigned char *lb = buf + __mul24(p, sb) + c * 16;
        const size_t step = (size_t)R2 * plane * sizeof(C2<T>);
        with_radix<RMAX>(R1, [&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            C2<T> x[Ch::N][R];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                C2<T> a[Ch::N];
                Ch::split(*reinterpret_cast<const V *>(lb + k * s1), a);
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) x[q][k] = a[q];
            }
#pragma unroll
            for (int q = 0; q < Ch::N; ++q) Dft<T, R, 1>::run(x[q]);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                C2<T> a[Ch::N];
#pragma unroll
                for (int q = 0; q < Ch::N; ++q) a[q] = x[q][r];
                gst(reinterpret_cast<V *>(reinterpret_cast<char *>(g) + r * step))[0] = Ch::join(a);
            }
        });
    }
    const double sum = block_sum(e);
    if (threadIdx.x == 0) I.part_ek[t.slot] = sum;
}

// ---------------------------------------------------------------- stage probes

// Parity probes (never part of an evaluation): the launches cover the tiles of
// a whole pass, and every workgroup whose tile belongs to another grid than
// `target` returns at once (uniformly).

// theta_a(r_i) = n_i p_a(q0_i) (the text after Eq. (Eoffk)) of the tile's
// points into dst [kNQ][N] (working precision), from n and the stored grad n,
// as the theta pass forms them.  tile: a = first row, b = rows.
template <typename T>
__global__ void __launch_bounds__(kMaxThreads) k_probe_theta(const InstDev *insts, const Tile *tiles,
                                                          const Consts *cst, void *dstv, int target) {
    __shared__ T qm[kNQ], Mm[kNQ * kNQ], invm[kMaxMc + 1];
    const Tile t = tiles[blockIdx.x];
    if (t.inst != target) return;
    const InstDev &I = insts[t.inst];
    load_consts<T>(cst, qm, Mm, invm);
    __syncthreads();
    const int N3 = I.n3;
    const size_t N = (size_t)I.n1 * I.n2 * I.n3, p0 = (size_t)t.a * N3;
    const T *nin = reinterpret_cast<const T *>(I.n) + p0;
    const T *gin = reinterpret_cast<const T *>(I.grad) + p0;
    T *dst = reinterpret_cast<T *>(dstv) + p0;
    for (int idx = threadIdx.x; idx < t.b * N3; idx += blockDim.x) {
        const T nv = nin[idx];
        T th[kNQ];
#pragma unroll
        for (int a = 0; a < kNQ; ++a) th[a] = (T)0;
        if (nv >= (T)cst->nmin) {
            const T gx = gin[idx], gy = gin[N + idx], gz = gin[2 * N + idx];
            LocalQ<T, false> lq;
            lq.eval(nv, gx * gx + gy * gy + gz * gz, cst->qc, cst->iqc, cst->mc, invm);
            SplineW<T> sw;
            sw.locate(lq.q0, qm, kNQ);
            const T *Mj = Mm + sw.j * kNQ;
#pragma unroll
            for (int a = 0; a < kNQ; ++a) {
                T v = nv * sw.C0 * Mj[a] + nv * sw.C1 * Mj[kNQ + a];
                if (a == sw.j) v += nv * sw.A0;
                if (a == sw.j + 1) v += nv * sw.A1;
                th[a] = v;
            }
        }
#pragma unroll
        for (int a = 0; a < kNQ; ++a) dst[a * N + idx] = th[a];
    }
}

// u_a(r_i) = sum_G u_a(G) exp(i G.r_i) (Eq. (epsilon)): the inverse axis-3
// transform of the u spectra, as the assembly pass forms it, into dst
// [kNQ][N] (working precision).  tile: a = first row, b = rows.
template <typename T, int RMAX>
__global__ void __launch_bounds__(kMaxThreads) k_probe_u(const InstDev *insts, const Tile *tiles, const void *twv,
                                                        void *dstv, int target) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Tile t = tiles[blockIdx.x];
    if (t.inst != target) return;
    const InstDev &I = insts[t.inst];
    const XTile<T, 0, 0> X(I.p3);
    const int N3 = X.len(), N3h = N3 / 2 + 1, row0 = t.a, B = t.b, nt = blockDim.x;
    const size_t N = (size_t)I.n1 * I.n2 * I.n3;
    C2<T> *tw = reinterpret_cast<C2<T> *>(smem + B * X.rs());
    load_twiddles<T>(tw, I.p3, reinterpret_cast<const C2<T> *>(twv));
    u_lines_in(smem, X, reinterpret_cast<const C2<T> *>(I.spec) + (size_t)row0 * N3h * kNQ, B, I.dn3h);
    __syncthreads();
    xtile_fft<T, 1, RMAX, 0, 0>(smem, X, B, tw);
    T *dst = reinterpret_cast<T *>(dstv) + (size_t)row0 * N3;
    for (int idx = threadIdx.x; idx < (kNQ / 2) * B * N3; idx += nt) {
        const int m = idx / (B * N3), rest = idx - m * B * N3, rb = rest / N3, k = rest - rb * N3;
        const C2<T> z = reinterpret_cast<const C2<T> *>(smem + __mul24(rb, X.rs()) + X.elem(k))[m];
        dst[(size_t)(2 * m) * N + rest] = z.x;
        dst[(size_t)(2 * m + 1) * N + rest] = z.y;
    }
}

// ---------------------------------------------------------------- launchers

// The passes launch by family (the axis they transform): axis 3 (x), axis 2
// (y), axis 1 (z); each family's launcher is compiled in a translation unit
// of its own per precision (kernels_f32_x.hip ...), so the build runs them in
// parallel.  A launch with ntiles == 0 only raises the kernel's LDS limit
// (done once when the launches are planned, never while a stream is being
// captured).

// Kernels that take more than 64 KB of LDS opt in to the device's limit.
template <typename K>
static void allow_lds(K kernel, size_t bytes) {
    if (bytes > 65536) (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

#define VDWNL_LAUNCH(kern, ...)                                                                      \
    do {                                                                                             \
        if (a.ntiles == 0) allow_lds(kern, a.lds);                                                   \
        else hipLaunchKernelGGL(kern, dim3(a.ntiles), dim3(a.threads), a.lds, a.stream, a.insts, a.tiles, \
                                __VA_ARGS__);                                                        \
    } while (0)

// the axis-3 passes: by split class, or as a compile-time length.  These two
// passes do more index work a point than the others, and constants pay at every
// one of the common lengths (compile-time against run-time radices, us an
// evaluation: 24^3 60 and 64, 48^3 93 and 96, 64^3 110 and 112, 96^3 212 and 224,
// 128^3 399 and 427, 160 x 160 x 320 1743 and 1941, where the theta pass alone takes
// 276 and 406; FP64 the same way, 96^3 378 and 400).
template <typename T, int RMAX, int CR1, int CR2>
hipError_t launch_x_pass(int kind, const LaunchArgs &a) {
    switch (kind) {
        case KX_THETA: VDWNL_LAUNCH((k_x_theta<T, RMAX, CR1, CR2>), a.cst, a.tw); break;
        case KX_ASSEMBLE: VDWNL_LAUNCH((k_x_assemble<T, RMAX, CR1, CR2>), a.cst, a.tw); break;
        case KP_U: VDWNL_LAUNCH((k_probe_u<T, RMAX>), a.tw, a.dst, a.target); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <typename T>
hipError_t launch_x(int kind, int cls, const LaunchArgs &a) {
    switch (a.len) {
        case 24: return launch_x_pass<T, 10, 4, 6>(kind, a);
        case 32: return launch_x_pass<T, 10, 4, 8>(kind, a);
        case 48: return launch_x_pass<T, 10, 6, 8>(kind, a);
        case 64: return launch_x_pass<T, 10, 8, 8>(kind, a);
        case 96: return launch_x_pass<T, 16, 8, 12>(kind, a);
        case 128: return launch_x_pass<T, 16, 8, 16>(kind, a);
        case 160: return launch_x_pass<T, 16, 10, 16>(kind, a);
        case 320: return launch_x_pass<T, 20, 16, 20>(kind, a);
        default: break;
    }
    switch (cls) {
        case 0: return launch_x_pass<T, kSplitClassMax[0], 0, 0>(kind, a);
        case 1: return launch_x_pass<T, kSplitClassMax[1], 0, 0>(kind, a);
        case 2: return launch_x_pass<T, kSplitClassMax[2], 0, 0>(kind, a);
        case 3: return launch_x_pass<T, kSplitClassMax[3], 0, 0>(kind, a);
        default: return hipErrorInvalidValue;
    }
}

// the one-axis derivatives: by split class (the gradient's transforms in FP64,
// the divergence's in T); kLenGeneric: axis 2 without a split
template <typename T, typename C, int MODE>
hipError_t launch_deriv(int cls, const LaunchArgs &a) {
    const void *tw = MODE == 0 ? a.twd : a.tw;
    switch (cls) {
        case 0: VDWNL_LAUNCH((k_deriv<T, C, kSplitClassMax[0], MODE>), tw); break;
        case 1: VDWNL_LAUNCH((k_deriv<T, C, kSplitClassMax[1], MODE>), tw); break;
        case 2: VDWNL_LAUNCH((k_deriv<T, C, kSplitClassMax[2], MODE>), tw); break;
        case 3: VDWNL_LAUNCH((k_deriv<T, C, kSplitClassMax[3], MODE>), tw); break;
        case kDenseClass: VDWNL_LAUNCH((k_deriv_dense<T, C, MODE>), tw); break;
        default: VDWNL_LAUNCH((k_deriv_any<T, C, MODE>), tw); break;
    }
    return hipGetLastError();
}
template <typename T>
hipError_t launch_deriv(int kind, int cls, const LaunchArgs &a) {
    const bool grad = kind == KG_X || kind == KG_Y || kind == KG_Z;
    return grad ? launch_deriv<T, double, 0>(cls, a) : launch_deriv<T, T, 1>(cls, a);
}

// the axis-2 passes of the 20 spectra: by split class
template <typename T, int S>
hipError_t launch_y20(int cls, const LaunchArgs &a) {
    switch (cls) {
        case 0: VDWNL_LAUNCH((k_y<T, S, kSplitClassMax[0]>), a.tw); break;
        case 1: VDWNL_LAUNCH((k_y<T, S, kSplitClassMax[1]>), a.tw); break;
        case 2: VDWNL_LAUNCH((k_y<T, S, kSplitClassMax[2]>), a.tw); break;
        case 3: VDWNL_LAUNCH((k_y<T, S, kSplitClassMax[3]>), a.tw); break;
        default: VDWNL_LAUNCH((k_y_any<T, S>), a.tw); break;
    }
    return hipGetLastError();
}

// the fused axis-1 pass and its probes: by split class (N1 <= 204: radices to 25)
template <typename T, int CT>
hipError_t launch_zmain(int cls, int probe, const LaunchArgs &a) {
    switch (cls) {
        case 0: VDWNL_LAUNCH((k_z_main<T, CT, kZClassMax[0]>), a.cols, a.tw, probe); break;
        case 1: VDWNL_LAUNCH((k_z_main<T, CT, kZClassMax[1]>), a.cols, a.tw, probe); break;
        case 2: VDWNL_LAUNCH((k_z_main<T, CT, kZClassMax[2]>), a.cols, a.tw, probe); break;
        case 3: VDWNL_LAUNCH((k_z_main<T, CT, kZClassMax[3]>), a.cols, a.tw, probe); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <typename T>
hipError_t launch_zmain(int cls, int probe, const LaunchArgs &a) {
    if (a.general) return a.packed ? launch_zmain<T, CT_GEN_PACKED>(cls, probe, a) : launch_zmain<T, CT_GEN>(cls, probe, a);
    if constexpr (sizeof(T) == 4)
        if (a.mfma) return launch_zmain<T, CT_MFMA>(cls, probe, a);
    return launch_zmain<T, CT_VEC>(cls, probe, a);
}

#undef VDWNL_LAUNCH

}  // namespace vdwnl
