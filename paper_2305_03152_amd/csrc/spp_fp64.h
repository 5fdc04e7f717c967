// fp64 functions of the passes that finish vertices: 1 - e^s for s <= 0 and log(1 - x) for 0 <= x <= 1.
//
// The library's routines and a division take some 300 instructions, which set the pace of those passes.  These take
// less than half of that and are more accurate: the parts that decide the last place (the reduced argument, the
// first two terms of the series, the quotient, the multiple of ln 2) are carried with their rounding errors
// (sums and products whose error is recovered exactly: Dekker, Numer. Math. 18, 1971), so that little more than the
// final rounding is left.  Largest errors over 4M points against 113-bit arithmetic on gfx950, in units in the last place:
// 0.71 and 0.56, the library's expm1 and log1p 1.13 and 0.65.  The passes that finish the vertices of a 14M-vertex
// graph after its first two hops: 106 and 181 us with the library's, 84 and 131 with these, 70 and 131 with the same series
// summed plainly (1.2 and 2.9 units).
#ifndef SPP_FP64_H
#define SPP_FP64_H

namespace spp {

// ln 2 in two parts; the upper one has 32 trailing zeros, so its small integer multiples are exact.
constexpr double kLn2Hi = 0x1.62e42feep-1, kLn2Lo = 0x1.a39ef35793c76p-33;

// 1 - e^s, s <= 0.  e^s = 2^k e^r, |r| <= ln2 / 2: 1 - 2^k - 2^k (r + r^2/2 + r^3 P(r)), P from the Taylor series up to
// r^13.  -inf gives 1, NaN stays NaN.
__device__ __forceinline__ double one_minus_exp(double s) {
    s = s < -64.0 ? -64.0 : s;                   // 1 - e^-64 rounds to 1
    const double k = rint(s * 1.4426950408889634);
    const double t = fma(-k, kLn2Hi, s);         // exact
    const double r = fma(-k, kLn2Lo, t), rl = fma(-k, kLn2Lo, t - r);
    double p = 1.0 / 6227020800.0;
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    const double h = 0.5 * r, q = h * r, ql = fma(h, r, -q);             // r^2 / 2
    const double low = fma(q * (r + r), p, ql) + fma(rl, r, rl);         // the rest of the series, and what r lacks
    const double e = ldexp(1.0, (int)k);
    const double one_e = 1.0 - e, er = e * r, eq = e * q;                // exact
    const double a = one_e - er, al = (one_e - a) - er;
    const double b = a - eq, bl = (a - b) - eq;
    return b + fma(-e, low, al + bl);
}

// f / d for integers 0 < f <= 64, 0 < d < 2^31: the IEEE quotient, in a third of its instructions.  A reciprocal refined
// twice, the quotient once: what that leaves before the last rounding is below 2^-50 of a unit in the last place, and f / d
// is 1 / (2 d) of one, 2^-32 at least, away from where the rounding turns.
__device__ __forceinline__ double small_quotient(double f, double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double q = f * r;
    return fma(fma(-d, q, f), r, q);
}

// log(1 - x), 0 <= x <= 1: log(2^e m) = e ln2 + 2 atanh(f / (2 + f)), m = 1 + f between sqrt(1/2) and sqrt(2), the
// series of atanh up to the 21st power; f = -x itself where e = 0.  1 gives -inf, NaN stays NaN.
__device__ __forceinline__ double log1p_neg(double x) {
    const double w = 1.0 - x, wl = (1.0 - w) - x;
    const bool near_one = w >= 0.70710678;       // e = 0
    double m = __builtin_amdgcn_frexp_mant(w);
    int ex = __builtin_amdgcn_frexp_exp(w);
    const bool low = m < 0.70710678;
    m = low ? 2.0 * m : m;
    ex -= low ? 1 : 0;
    const double f = near_one ? -x : m - 1.0, e = near_one ? 0.0 : (double)ex;
    // what 1 - x lost, in the scale of m: nothing above 1/2, and below it m is 2 w
    const double fl = near_one ? 0.0 : wl + wl;
    const double den = 2.0 + f, dl = (2.0 - den) + f;
    double r = __builtin_amdgcn_rcp(den);
    r = fma(fma(-den, r, 1.0), r, r);
    r = fma(fma(-den, r, 1.0), r, r);
    const double s = f * r;
    const double sl = fma(-s, dl + fl, fma(-den, s, f) + fl) * r;        // (f + fl) / (2 + f + fl) = s + sl
    const double z = s * s;
    double p = 1.0 / 21.0;
    p = fma(p, z, 1.0 / 19.0);
    p = fma(p, z, 1.0 / 17.0);
    p = fma(p, z, 1.0 / 15.0);
    p = fma(p, z, 1.0 / 13.0);
    p = fma(p, z, 1.0 / 11.0);
    p = fma(p, z, 1.0 / 9.0);
    p = fma(p, z, 1.0 / 7.0);
    p = fma(p, z, 1.0 / 5.0);
    p = fma(p, z, 1.0 / 3.0);
    const double t = s + s, tl = fma(t * z, p, sl + sl);
    const double c = e * kLn2Hi;                 // exact; 0 or larger than t
    const double a = c + t, al = (c - a) + t;
    const double l = a + (al + fma(e, kLn2Lo, tl));
    return x >= 1.0 ? -__builtin_inf() : l;
}

}  // namespace spp
#endif
