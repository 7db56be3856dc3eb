// Exact modular arithmetic for primes t < 2^50 on gfx950, done in FP64 with FMA.
//
// Residues live in HBM as uint64 and are moved into doubles in registers (every
// integer below 2^53 is exact in a double).  A product a*b (|a|,|b| < 2^50) is
// split exactly as h + l with h = fl(a*b) and l = fma(a, b, -h) (Dekker/Kahan
// two-product); a quotient estimate c = rint(h * (1/t)) is off by at most a
// few units, so h - c*t is an integer below 2^52 that one fma computes exactly,
// and adding l gives the exact a*b - c*t.  On gfx950 this costs ~8 full-rate
// FP64 operations, about 1.8x the throughput of a 64-bit Shoup product built from
// 32-bit integer multiplies (measured: 3.2 vs 1.8 T products/s).
//
// Bounds used below (u = 2^-53, every modulus t < 2^50; contexts take primes from 2^30 on):
//   mul_canon:  a, b in [0, t)              -> |ab/t - c| < 7/8, result in [0, t)
//   mul_lazy:   |a| <= B 2^50, b in [0, t)  -> exact representative within (1/2 + 3B/8) t, B <= 8
//               (7/8 t at B = 1; corr may follow directly only for B < 4/3, else reduce)
//   corr:       integer s in (-t, 2t)       -> [0, t)
//   reduce:     integer |x| < 2^53          -> [0, t)
//   reduce_c:   integer |x| < 2^53          -> centred, |r| <= t/2 + 2 (half of reduce's cost)
// Centred words are what transforms keep between their rounds and passes: 3 operations
// instead of 6 per word and round, and headroom for one more doubling.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define NJ_HD __host__ __device__ __forceinline__

namespace nj {

constexpr double kTwo52 = 4503599627370496.0;  // 2^52

// uint64 x < 2^52  <->  double, by placing x in the mantissa of 2^52 + x
NJ_HD double u2d(uint64_t x)
{
    union { uint64_t u; double d; } v;
    v.u = x | 0x4330000000000000ull;
    return v.d - kTwo52;
}
NJ_HD uint64_t d2u(double x)  // x an integer in [0, 2^52)
{
    union { uint64_t u; double d; } v;
    v.d = x + kTwo52;
    return v.u & 0x000FFFFFFFFFFFFFull;
}

struct Mod {
    double t;   // the prime
    double ti;  // fl(1 / t)
};

// An integer s in (-t, 2t)  ->  s mod t in [0, t), with no compare or select:
// floor(s/t) = rint((s + 1/2)/t - 1/2), evaluated as rint(fma(s, ti, ti/2 - 1/2)).  The
// exact value lies at least 0.5/t >= 2^-51 from a half-integer; the computed one is
// within 2^-52 (ti's relative error 2^-53 on |s/t| < 2) + 2^-53 (the fma's rounding) +
// 2^-55 (the offset's rounding) of it, so rint returns floor(s/t) exactly.
NJ_HD double corr(double s, Mod m)
{
    const double c = rint(fma(s, m.ti, fma(0.5, m.ti, -0.5)));
    return fma(-c, m.t, s);
}

// a, b in [0, t)  ->  a*b mod t in [0, t)
NJ_HD double mul_canon(double a, double b, Mod m)
{
    double h = a * b;
    double l = fma(a, b, -h);
    double c = rint(h * m.ti);
    return corr(fma(-c, m.t, h) + l, m);
}

// Shoup-style product with a fixed canonical factor w and its companion wq = fl(w/t):
// b in [0, t) -> b*w mod t in [0, t).  |b wq - b w/t| <= 2u b w/t < 1/4.
NJ_HD double mul_shoup(double b, double w, double wq, Mod m)
{
    double h = b * w;
    double l = fma(b, w, -h);
    double c = rint(b * wq);
    return corr(fma(-c, m.t, h) + l, m);
}

// Lazy product for signed operands |a| <= B 2^50, |b| < t, B <= 8: returns an exact
// representative of a*b mod t.  |ab/t| <= B 2^50 is estimated to within 3u B 2^50 = 3B/8 and
// rounded, so |ab - ct| <= (1/2 + 3B/8) t; c is at most 2^53, |l| at most 2^49, and h - ct and
// the sum stay integers below 2^53.
NJ_HD double mul_lazy(double a, double b, Mod m)
{
    double h = a * b;
    double l = fma(a, b, -h);
    double c = rint(h * m.ti);
    return fma(-c, m.t, h) + l;
}

// any exact integer |x| < 2^53  ->  x mod t in [0, t)
NJ_HD double reduce(double x, Mod m)
{
    double c = rint(x * m.ti);
    return corr(fma(-c, m.t, x), m);
}

// any exact integer |x| < 2^53  ->  the representative next to 0, |r| <= t/2 + 2 (the
// quotient's error is below |x/t| 2^-52, times t at most 2)
NJ_HD double reduce_c(double x, Mod m)
{
    double c = rint(x * m.ti);
    return fma(-c, m.t, x);
}

// mul_shoup without its last correction: |b| <= 1.5 t, w in [0, t), wq = fl(w/t) -> exact
// representative within (-t, t): |b wq - b w/t| <= 2u 1.5 2^50 = 3/8, so |r| <= 7/8 t
NJ_HD double mul_shoup_lazy(double b, double w, double wq, Mod m)
{
    double h = b * w;
    double l = fma(b, w, -h);
    double c = rint(b * wq);
    return fma(-c, m.t, h) + l;
}

NJ_HD double add_mod(double a, double b, Mod m) { return corr(a + b, m); }
NJ_HD double sub_mod(double a, double b, Mod m) { return corr(a - b, m); }

}  // namespace nj
