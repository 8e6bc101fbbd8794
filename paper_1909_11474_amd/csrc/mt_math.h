// Device math of the site routine's arguments.  Needs nothing but the HIP keywords
// and the compiler's builtins.
#pragma once

namespace mt {

// ---------------------------------------------------------------------------
// float: the hardware transcendental instructions (v_exp_f32,
// v_log_f32, v_rcp_f32); arguments on the hot path stay in the normal range.
//
// double: 2^x, log2 x (x > 0) and 1/x for the arguments the site routine has.
// They are most of a float64 bond's instructions, and the device library's
// (special cases) take about twice as many: a bond 250
// instructions with those, 150 with these (64 candidates x 60 structures 176 ->
// 152 us).  The polynomials interpolate at Chebyshev nodes (computed in 60
// digits); errors below 0.9 ulp (2^x), 0.6 ulp (log2) and 0.6 ulp (1/x).  The
// float64 kernels' errors against 64-bit sums in another order stay where they
// were (2e-15 of a force).  A candidate inside the domain may overflow zeta^n or
// zeta, so infinite arguments have the device library's outcome.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float dexp2(float x) { return __builtin_amdgcn_exp2f(x); }
template <bool Inf = false>
__device__ __forceinline__ float dlog2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float drcp(float x) { return __builtin_amdgcn_rcpf(x); }

constexpr double kMaxDouble = 1.7976931348623157e308;

// 1/x, x and 1/x finite and not 0: the hardware's estimate (about 2^-24) and two
// Newton steps.
__device__ __forceinline__ double drcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// 1/x with 0 for infinite x, as the float instruction has it.  The comparison lies
// beside the Newton steps' chain.
__device__ __forceinline__ float drcp_inf(float x) { return drcp(x); }
__device__ __forceinline__ double drcp_inf(double x) {
    const double r = drcp(x);
    return x > kMaxDouble ? 0.0 : r;
}

// x = k + f with k = rint(x), |f| <= 1/2; 2^f = 1 + f q(f), q of degree 10
// (relative error of 2^f 2e-17 before rounding).  The conversion of k saturates,
// so infinite x need f = 0 only.
__device__ __forceinline__ double dexp2(double x) {
    const double k = __builtin_rint(x);
    const double f = x == k ? 0.0 : x - k;
    double q = 4.4549605981865186e-10;
    q = __builtin_fma(q, f, 7.072585949269223e-09);
    q = __builtin_fma(q, f, 1.0178062445845774e-07);
    q = __builtin_fma(q, f, 1.321544258792169e-06);
    q = __builtin_fma(q, f, 1.525273382983612e-05);
    q = __builtin_fma(q, f, 0.0001540353044173605);
    q = __builtin_fma(q, f, 0.0013333558146416936);
    q = __builtin_fma(q, f, 0.009618129107606888);
    q = __builtin_fma(q, f, 0.0555041086648216);
    q = __builtin_fma(q, f, 0.24022650695910097);
    q = __builtin_fma(q, f, 0.6931471805599453);
    return __builtin_amdgcn_ldexp(__builtin_fma(q, f, 1.0), (int)k);
}

// x = 2^e m, m in [sqrt(1/2), sqrt(2)); with s = (m - 1)/(m + 1),
// log2 m = s L(s^2), L of degree 7 (relative error 1.4e-17 before rounding); s and
// the leading product 2/ln 2 s carry their rounding errors to the last sum (without
// them 2.0 ulp).  Float64 Tersoff-form gradients against 64-bit sums: 2.1e-15 on 64-atom
// cells and 2.9e-16 on uneven sets; with the device library 2.1e-15 and 2.6e-16.
// Infinite x counts as the largest finite value, or, with Inf, comes out as it is.
template <bool Inf = false>
__device__ __forceinline__ double dlog2(double x) {
    if (!Inf) x = __builtin_fmin(x, kMaxDouble);
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.7071067811865476;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double num = m - 1.0, den = m + 1.0, dlo = m - (den - 1.0);
    double r = __builtin_amdgcn_rcp(den);
    r = __builtin_fma(r, __builtin_fma(-den, r, 1.0), r);
    const double s0 = num * r;
    const double slo = __builtin_fma(-dlo, s0, __builtin_fma(-den, s0, num)) * r;
    const double s = s0 + slo;
    const double w = s * s;
    double l = 0.21366122502798326;
    l = __builtin_fma(l, w, 0.22091286734180157);
    l = __builtin_fma(l, w, 0.26233436060329546);
    l = __builtin_fma(l, w, 0.3205985347650481);
    l = __builtin_fma(l, w, 0.4121985858422942);
    l = __builtin_fma(l, w, 0.577078016345514);
    l = __builtin_fma(l, w, 0.9617966939259898);
    constexpr double kHi = 2.8853900817779268, kLo = 4.0710547481862066e-17;   // 2 / ln 2
    const double t = s0 * kHi;
    double lo = __builtin_fma(s0, kLo, __builtin_fma(slo, kHi, __builtin_fma(s0, kHi, -t)));
    lo = __builtin_fma(s * w, l, lo);
    const double ed = (double)e, hi = ed + t;
    lo += (ed - hi) + t;
    return Inf && x > kMaxDouble ? x : hi + lo;
}

// float64 2^y for the energy terms of the float path, finite arguments only:
// as dexp2 with q of degree 6 (relative error 1.1e-10, under 2e-9 eV on a 15 eV
// energy term; the Taylor series to degree 8 has 2.7e-10 and one operation more).
__device__ __forceinline__ double exp2_acc(double y) {
    const double k = __builtin_rint(y);
    const double f = y - k;
    double q = 1.5297323760701075e-05;
    q = __builtin_fma(q, f, 0.0001546144469856913);
    q = __builtin_fma(q, f, 0.001333350238616277);
    q = __builtin_fma(q, f, 0.009618056678524637);
    q = __builtin_fma(q, f, 0.055504108839096185);
    q = __builtin_fma(q, f, 0.24022650922288757);
    q = __builtin_fma(q, f, 0.6931471805599453);
    return __builtin_amdgcn_ldexp(__builtin_fma(q, f, 1.0), (int)k);
}

}  // namespace mt
