// Modular arithmetic on the FP64 vector ALU.
//
// Why floating point: a 64-bit Shoup/Barrett product needs about ten 32-bit integer
// multiplies and their additions, and v_fma_f64 issues as fast as one of those (36 - 38 T
// lane-instructions/s, both).  For moduli p < 2^51 a modular product can be made
// EXACT with six FP64 instructions: the product is split error-free into
// h = RN(a*b) and l = fma(a,b,-h); the quotient estimate q = rint(a * (b/p)) is
// within one unit of the true quotient; fma(-q,p,h) + l then equals a*b - q*p
// exactly because that integer is below 2^53.  Every quantity below is an integer
// held in a double; "exact" means no rounding ever happens on the value path.
//
// Ranges (p < 2^51, so 4p <= 2^53):
//   mulmod_w(y, w)  : |y| <= 2^53, |w| <= p/2 prepared as (w, RN(w/p))
//                     result r = y*w - q*p with |r| <= (1/2 + |y|*2^-53) p  (< 1.5 p)
//   mulmod(a, b)    : |a|,|b| <= p, result |r| <= 1.25 p; in general |a| <= 2^53, |b| <= p/2: |r| <= (1/2 + 1.5 |a|*2^-53) p
//   reduce_balanced : |x| <= 2^53 -> |r| <= p/2 + 1
//   canon           : |x| <= 2^53 -> [0, p)
#pragma once

struct WMulD { double w, wp; };

__device__ __forceinline__ double u2d(unsigned long long x) {  // x < 2^52, exact
    return __longlong_as_double((long long)(x | 0x4330000000000000ull)) - 4503599627370496.0;
}
__device__ __forceinline__ unsigned long long d2u(double d) {  // integer 0 <= d < 2^52
    return (unsigned long long)__double_as_longlong(d + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull;
}

__device__ __forceinline__ double mulmod_w(double y, double w, double wp, double p) {
    double h = y * w;
    double l = fma(y, w, -h);
    double q = rint(y * wp);
    double c = fma(-q, p, h);
    return c + l;
}

__device__ __forceinline__ double mulmod(double a, double b, double p, double pinv) {
    double h = a * b;
    double l = fma(a, b, -h);
    double q = rint(h * pinv);
    double c = fma(-q, p, h);
    return c + l;
}

// Sum of K = 2 .. 4 products y_k * w_k (0 <= y < 2^51, |w| <= p/2) with ONE reduction, p < 2^50: the sum runs in s, which starts
// at M = 3*2^51*p (a multiple of p, so large that s never leaves [2^51 p, 2.5*2^52 p] and h = s' - s is exact); what the
// rounding of s drops, y*w - h, is an integer below 2^50.3 and is collected in l.  4K + 3 instructions against 7K.
// Three sources in ModUp and in a product's tail at N = 2^16, 64 items of 24 primes: 7216 -> 7046 us for the whole product.
// |value| <= (0.875 + 1.0 + 1.125 + 1.25)p (the first K of them) + (2 + K/4)p + |addend|, see chain_bound
struct ProductChain { double s, l; };
__device__ __forceinline__ double chain_origin(double p) { return 6755399441055744.0 * p; }
__device__ __forceinline__ ProductChain chain_first(double M, double y, double w) {
    const double s = fma(y, w, M), h = s - M;
    return ProductChain{s, fma(y, w, -h)};
}
__device__ __forceinline__ void chain_add(ProductChain &c, double y, double w) {
    const double s = fma(y, w, c.s), h = s - c.s;
    c.l += fma(y, w, -h);
    c.s = s;
}
__device__ __forceinline__ double chain_value(const ProductChain &c, double p, double pinv) {
    const double q = rint(c.s * pinv);
    return fma(-q, p, c.s) + c.l;
}
constexpr double chain_bound(int K) {
    double b = 2.0 + 0.25 * K;
    for (int k = 1; k <= K; k++) b += 0.5 * (1.5 + 0.25 * k);
    return b;
}

__device__ __forceinline__ double reduce_balanced(double x, double p, double pinv) {
    return fma(-rint(x * pinv), p, x);
}

__device__ __forceinline__ double canon(double x, double p, double pinv) {
    double r = reduce_balanced(x, p, pinv);
    return r < 0.0 ? r + p : r;
}

// |x| <= 2.9 p -> [0, p).  p < 2^50: the quotient is taken half a unit of x above x / p, so that floor is the exact one: for |x| < 3p
// the two roundings of t move it by less than 2 * 2^-53 + 2^-52 <= 2^-51 where floor changes (at -2 .. 2), and x / p + 0.5 / p is
// 0.5 / p > 2^-51 away from there.  Three instructions instead of seven.  p < 2^51: the distance would not do.
template <bool P51>
__device__ __forceinline__ double canon_near(double x, double p, double pinv) {
    if (P51) return canon(x, p, pinv);
    return fma(-floor(fma(x, pinv, 0.5 * pinv)), p, x);
}

// value known to lie in (-p, p)
__device__ __forceinline__ double canon_small(double r, double p) { return r < 0.0 ? r + p : r; }

__device__ __forceinline__ bool is_p51(const P51Mask &m, int t) { return (m.w[t >> 6] >> (t & 63)) & 1ull; }

// Intermediate between the two passes of a transform (never visible outside the library): the value as the pass leaves it
// (within the bounds of LazyRange, ntt_v2.h), stored as the bits of the double itself.  Saves the canonical form, both integer
// conversions and the reduction.
__device__ __forceinline__ unsigned long long mid_store(double x) { return (unsigned long long)__double_as_longlong(x); }
__device__ __forceinline__ double mid_load(unsigned long long bits) { return __longlong_as_double((long long)bits); }
