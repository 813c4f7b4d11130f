// Double-double arithmetic for the exact path and the model build.
//
// A value is hi + lo with |lo| <= ulp(hi)/2, ~106 significant bits.  Built from
// two error-free transformations: Knuth's TwoSum (s + e = a + b exactly) and
// the product with its rounding error recovered by one fused multiply-add
// (Dekker 1971 with an FMA in place of the splitting).  The square roots take
// an fp64 estimate and one correction.  exp uses argument reduction by ln 2, a
// further division by 1024, a Taylor series and repeated squaring.  Every
// function turns floating-point contraction off: a product fused into a later
// addition would break the error-free steps.
#pragma once
#include <hip/hip_runtime.h>

struct dd {
    double hi, lo;
};

__host__ __device__ __forceinline__ dd dd_make(double a)
{
#pragma clang fp contract(off)
    return dd{a, 0.0};
}

__host__ __device__ __forceinline__ dd two_sum(double a, double b)
{
#pragma clang fp contract(off)
    double s = a + b;
    double bb = s - a;
    double e = (a - (s - bb)) + (b - bb);
    return dd{s, e};
}

__host__ __device__ __forceinline__ dd quick_two_sum(double a, double b)
{
#pragma clang fp contract(off)
    double s = a + b;
    return dd{s, b - (s - a)};
}

__host__ __device__ __forceinline__ dd two_prod(double a, double b)
{
#pragma clang fp contract(off)
    double p = a * b;
    return dd{p, fma(a, b, -p)};
}

__host__ __device__ __forceinline__ dd dd_add(dd x, dd y)
{
#pragma clang fp contract(off)
    dd s = two_sum(x.hi, y.hi);
    dd t = two_sum(x.lo, y.lo);
    s.lo += t.hi;
    s = quick_two_sum(s.hi, s.lo);
    s.lo += t.lo;
    return quick_two_sum(s.hi, s.lo);
}

__host__ __device__ __forceinline__ dd dd_neg(dd x)
{
#pragma clang fp contract(off)
    return dd{-x.hi, -x.lo};
}
__host__ __device__ __forceinline__ dd dd_sub(dd x, dd y)
{
#pragma clang fp contract(off)
    return dd_add(x, dd_neg(y));
}

__host__ __device__ __forceinline__ dd dd_add_d(dd x, double b)
{
#pragma clang fp contract(off)
    dd s = two_sum(x.hi, b);
    s.lo += x.lo;
    return quick_two_sum(s.hi, s.lo);
}

__host__ __device__ __forceinline__ dd dd_mul(dd x, dd y)
{
#pragma clang fp contract(off)
    dd p = two_prod(x.hi, y.hi);
    p.lo = fma(x.hi, y.lo, p.lo);
    p.lo = fma(x.lo, y.hi, p.lo);
    return quick_two_sum(p.hi, p.lo);
}

__host__ __device__ __forceinline__ dd dd_mul_d(dd x, double b)
{
#pragma clang fp contract(off)
    dd p = two_prod(x.hi, b);
    p.lo = fma(x.lo, b, p.lo);
    return quick_two_sum(p.hi, p.lo);
}

// sqrt for x > 0: s = sqrt(hi), then s + (x - s^2) / (2 s).
__host__ __device__ __forceinline__ dd dd_sqrt(dd x)
{
#pragma clang fp contract(off)
    double s = sqrt(x.hi);
    dd s2 = two_prod(s, s);
    dd r = dd_sub(x, s2);
    return quick_two_sum(s, r.hi / (2.0 * s));
}

// 1/sqrt(x) for x > 0: the fp64 value y and the next terms of its series in
// e = 1 - x y^2 (|e| of the order of 1e-16): y + y (e/2 + 3 e^2 / 8).  1 - x.hi y^2
// cancels exactly but for the products' low parts s; e is below that difference's
// own grid, so the rounding r of e is kept too.
__device__ __forceinline__ dd dd_rsqrt(dd x)
{
#pragma clang fp contract(off)
    const double y = rsqrt(x.hi);
    const dd h = two_prod(y, y);
    const dd q = two_prod(x.hi, h.hi);
    const double a = 1.0 - q.hi;
    const double s = fma(x.lo, h.hi, fma(x.hi, h.lo, q.lo));
    const double e = a - s, r = (a - e) - s;
    const double w = 0.5 * y;
    return quick_two_sum(y, fma(w, e, w * fma(0.75 * e, e, r)));
}

// a - p q and a - p q - r s: error-free leading products and sums, what is
// below them in fp64 sums (about five roundings of up to 2^-106 of the largest
// term, where dd_mul and dd_sub leave six).  The first adds its low parts as a
// short tree: it forms the pivots, whose errors reach every later entry.
__device__ __forceinline__ dd dd_fms(dd a, dd p, dd q)
{
#pragma clang fp contract(off)
    const dd t = two_prod(p.hi, q.hi);
    const dd u = two_sum(a.hi, -t.hi);
    const double c = fma(p.hi, q.lo, p.lo * q.hi);
    return quick_two_sum(u.hi, (a.lo - t.lo) + (u.lo - c));
}
__device__ __forceinline__ dd dd_fms2(dd a, dd p, dd q, dd r, dd s)
{
#pragma clang fp contract(off)
    const dd f = two_prod(p.hi, q.hi), g = two_prod(r.hi, s.hi);
    const dd t = two_sum(f.hi, g.hi);
    const dd u = two_sum(a.hi, -t.hi);
    double lo = fma(-p.hi, q.lo, a.lo);
    lo = fma(-p.lo, q.hi, lo);
    lo = fma(-r.hi, s.lo, lo);
    lo = fma(-r.lo, s.hi, lo);
    lo += u.lo - ((f.lo + g.lo) + t.lo);
    return quick_two_sum(u.hi, lo);
}

// exp(x) for |x| < 700.  x = k ln2 + r; r' = r / 1024 (at most 3.4e-4); expm1 by
// Taylor to degree 9 (the next term is below 2e-41), coefficients 1/i! as
// double-doubles; ten steps expm1(2y) = 2 expm1(y) + expm1(y)^2 (squarings of exp
// itself would multiply its rounding by 1024); scale by 2^k.
__host__ __device__ inline dd dd_exp(dd x)
{
#pragma clang fp contract(off)
    const dd ln2 = dd{6.93147180559945286227e-01, 2.31904681384629955842e-17};
    const dd cf[10] = {{1.0, 0.0}, {1.0, 0.0},
                       {0.5, 0.0}, {0.16666666666666666, 9.25185853854297e-18},
                       {0.041666666666666664, 2.3129646346357427e-18}, {0.008333333333333333, 1.1564823173178714e-19},
                       {0.001388888888888889, -5.300543954373577e-20}, {0.0001984126984126984, 1.7209558293420705e-22},
                       {2.48015873015873e-05, 2.1511947866775882e-23}, {2.7557319223985893e-06, -1.858393274046472e-22}};
    double k = rint(x.hi / ln2.hi);
    dd r = dd_sub(x, dd_mul_d(ln2, k));
    r = dd_mul_d(r, 1.0 / 1024.0);
    dd s = cf[9];
#pragma unroll
    for (int i = 8; i >= 1; --i) s = dd_add(dd_mul(s, r), cf[i]);
    s = dd_mul(s, r);
    for (int i = 0; i < 10; ++i) s = dd_add(dd{2.0 * s.hi, 2.0 * s.lo}, dd_mul(s, s));
    s = dd_add_d(s, 1.0);
    double sc = ldexp(1.0, (int)k);
    return dd{s.hi * sc, s.lo * sc};
}
