// Forward-mode dual numbers with N tangent directions, used by the adjoint
// kernels to contract flux and source Jacobians (dPhi/dQ, dS/dQ) without
// hand-written derivative code.  Arithmetic is the ordinary chain rule.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#ifndef LBM_FAST_CONTRACT
#pragma clang fp contract(on)
#endif

template <class R, int N>
struct Dual {
    R v;
    R d[N];

    __host__ __device__ Dual() {}
    __host__ __device__ Dual(R x) : v(x)
    {
#pragma unroll
        for (int j = 0; j < N; ++j) d[j] = R(0);
    }
};

template <class T> struct ScalarOf { using type = T; };
template <class R, int N> struct ScalarOf<Dual<R, N>> { using type = R; };

#define DUAL_BINOP(OP, VAL, DER)                                                        \
    template <class R, int N>                                                           \
    __host__ __device__ inline Dual<R, N> operator OP(const Dual<R, N> &a, const Dual<R, N> &b) \
    {                                                                                   \
        Dual<R, N> r;                                                                   \
        r.v = VAL;                                                                      \
        _Pragma("unroll") for (int j = 0; j < N; ++j) r.d[j] = DER;                     \
        return r;                                                                       \
    }
DUAL_BINOP(+, a.v + b.v, a.d[j] + b.d[j])
DUAL_BINOP(-, a.v - b.v, a.d[j] - b.d[j])
DUAL_BINOP(*, a.v * b.v, a.d[j] * b.v + a.v * b.d[j])
#undef DUAL_BINOP

template <class R, int N>
__host__ __device__ inline Dual<R, N> operator/(const Dual<R, N> &a, const Dual<R, N> &b)
{
    Dual<R, N> r;
    const R inv = R(1) / b.v;
    r.v = a.v * inv;
#pragma unroll
    for (int j = 0; j < N; ++j) r.d[j] = (a.d[j] - r.v * b.d[j]) * inv;
    return r;
}

template <class R, int N>
__host__ __device__ inline Dual<R, N> operator-(const Dual<R, N> &a)
{
    Dual<R, N> r;
    r.v = -a.v;
#pragma unroll
    for (int j = 0; j < N; ++j) r.d[j] = -a.d[j];
    return r;
}

// mixed scalar/dual arithmetic
template <class R, int N> __host__ __device__ inline Dual<R, N> operator+(const Dual<R, N> &a, R b) { return a + Dual<R, N>(b); }
template <class R, int N> __host__ __device__ inline Dual<R, N> operator+(R a, const Dual<R, N> &b) { return Dual<R, N>(a) + b; }
template <class R, int N> __host__ __device__ inline Dual<R, N> operator-(const Dual<R, N> &a, R b) { return a - Dual<R, N>(b); }
template <class R, int N> __host__ __device__ inline Dual<R, N> operator-(R a, const Dual<R, N> &b) { return Dual<R, N>(a) - b; }
template <class R, int N>
__host__ __device__ inline Dual<R, N> operator*(const Dual<R, N> &a, R b)
{
    Dual<R, N> r;
    r.v = a.v * b;
#pragma unroll
    for (int j = 0; j < N; ++j) r.d[j] = a.d[j] * b;
    return r;
}
template <class R, int N> __host__ __device__ inline Dual<R, N> operator*(R a, const Dual<R, N> &b) { return b * a; }
template <class R, int N> __host__ __device__ inline Dual<R, N> operator/(const Dual<R, N> &a, R b) { return a * (R(1) / b); }
template <class R, int N> __host__ __device__ inline Dual<R, N> operator/(R a, const Dual<R, N> &b) { return Dual<R, N>(a) / b; }

// log(1 + x) and its derivative 1 / (1 + x).
// Single precision on the device, for |x| <= 1/4, through the series
// log(1 + x) = 2 atanh(s) = 2 (s + s^3/3 + s^5/5 + ...), s = x / (2 + x)
// (|s| <= 1/7: five terms leave a truncation below 2^-27 of the result),
// with s carried as a float-float pair: 2 + x = t + e exactly (|x| < 2),
// s_hi = x / t by reciprocal and one Newton step, and the remainder
// x - s_hi t (exact by fma) gives s_lo = (x - s_hi t - s_hi e) / t.  The
// leading 2 s_hi is exact, so the result rounds once more than its
// correction.  About a sixth of the instructions of the library's log1pf,
// which serves larger arguments and the host.
__host__ __device__ inline float lbm_log1p(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if (!(fabsf(x) <= 0.25f)) return log1pf(x);
    const float t = 2.0f + x, e = x - (t - 2.0f);
    const float rt = __builtin_amdgcn_rcpf(t);
    float sh = x * rt;
    sh = fmaf(fmaf(-sh, t, x), rt, sh);
    const float sl = (fmaf(-sh, t, x) - sh * e) * rt;
    const float s2 = sh * sh;
    const float p = fmaf(s2, fmaf(s2, fmaf(s2, fmaf(s2, 1.0f / 11, 1.0f / 9), 1.0f / 7), 1.0f / 5), 1.0f / 3);
    return fmaf(2.0f, sh, 2.0f * fmaf(sh * s2, p, sl));
#else
    return log1pf(x);
#endif
}
__host__ __device__ inline double lbm_log1p(double x) { return log1p(x); }
template <class R, int N>
__host__ __device__ inline Dual<R, N> lbm_log1p(const Dual<R, N> &a)
{
    Dual<R, N> r;
    r.v = lbm_log1p(a.v);
    const R s = R(1) / (R(1) + a.v);
#pragma unroll
    for (int j = 0; j < N; ++j) r.d[j] = a.d[j] * s;
    return r;
}

// sqrt(x) and its derivative 1 / (2 sqrt(x))
__host__ __device__ inline float lbm_sqrt(float x) { return sqrtf(x); }
__host__ __device__ inline double lbm_sqrt(double x) { return sqrt(x); }
template <class R, int N>
__host__ __device__ inline Dual<R, N> lbm_sqrt(const Dual<R, N> &a)
{
    Dual<R, N> r;
    r.v = lbm_sqrt(a.v);
    const R s = R(0.5) / r.v;
#pragma unroll
    for (int j = 0; j < N; ++j) r.d[j] = a.d[j] * s;
    return r;
}

// Parameter type of kernels that keep populations in float and compute in
// double (an expression of Wd and double values is plain double arithmetic).
// Their quotients, roots and logarithms need relative errors far below the
// 2^-24 of the store they end in, not correct rounding: lbm_div, lbm_sqrt_of
// and lbm_log1p_of take the parameter type R and use, for Wd, the double
// instruction's estimate (about 2^-24) and one Newton step, and series of that
// accuracy: five instructions against about 16 of the IEEE division.  The float
// instruction's estimate costs the same with its two conversions, but has the
// float range: its results beyond 2^126 and those of products below 2^-126 are
// lost (a relativistic fluid of energy 2^-66: not a number).
struct Wd {
    double v;
    Wd() = default;
    __host__ __device__ constexpr Wd(double x) : v(x) {}
    __host__ __device__ constexpr operator double() const { return v; }
};

// 1 / x.  Where the estimate is infinite or zero its error is not a number,
// and the minimum takes the other operand: 1 / 0 and 1 / inf are inf and 0.
__host__ __device__ inline double lbm_rcp_wide(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const double r = __builtin_amdgcn_rcp(x);
    return fma(r, fmin(fma(-x, r, 1.0), 0.5), r);
#else
    return 1.0 / x;
#endif
}

template <class R, class S>
__host__ __device__ inline S lbm_div(const S &a, const S &b)
{
    if constexpr (std::is_same<R, Wd>::value)
        return a * lbm_rcp_wide(b);
    else
        return a / b;
}

template <class R, class S>
__host__ __device__ inline S lbm_sqrt_of(const S &x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (std::is_same<R, Wd>::value) {
        // y = x rsqrt(x) and one Newton step; zeros and infinity (class bits)
        // are their own roots
        const double r = __builtin_amdgcn_rsq(x), y = x * r;
        return __builtin_amdgcn_class(x, 0x260) ? x : fma(fma(-y, y, x), 0.5 * r, y);
    } else
#endif
        return lbm_sqrt(x);
}

// log(1 + x): for |x| <= 1/4 the series 2 atanh(s), s = x / (2 + x), |s| <=
// 1/7, seven terms (truncation below 2^-43 of the result)
template <class R, class S>
__host__ __device__ inline S lbm_log1p_of(const S &x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (std::is_same<R, Wd>::value) {
        if (!(fabs(x) <= 0.25)) return log1p(x);
        const double s = x * lbm_rcp_wide(2.0 + x), s2 = s * s;
        double t = fma(s2, 1.0 / 15, 1.0 / 13);
        t = fma(s2, t, 1.0 / 11);
        t = fma(s2, t, 1.0 / 9);
        t = fma(s2, t, 1.0 / 7);
        t = fma(s2, t, 1.0 / 5);
        t = fma(s2, t, 1.0 / 3);
        return 2.0 * fma(s * s2, t, s);
    } else
#endif
        return lbm_log1p(x);
}
