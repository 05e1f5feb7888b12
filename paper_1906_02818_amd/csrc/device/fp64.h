// Double-precision elementary functions of the FP64 paths, for exactly the
// arguments the paths have: Box-Muller from two 23-bit uniforms, and exp of
// a log-price. A library log / sincos / exp / sqrt accepts every double, and
// its argument reduction and special cases were most of an FP64 path's time.
// log and exp are table-driven after P. T. P. Tang (ACM Transactions on
// Mathematical Software 15 (1989) 144 for exp, 16 (1990) 378 for log): the
// argument is reduced by the nearest of a table's points, a short polynomial
// takes the rest.
//
//  - log u: u = m 2^-24 with an odd m below 2^24. z = m scaled to [1, 2)
//    falls in one of 128 intervals with a centre c; 1/c is held to 24 bits,
//    so r = z/c - 1 is exact and |r| <= 2^-8, and
//        -2 ln u = k (-2 ln 2) + (-2 ln c) + (-2 r + r^2 Q(r)),
//    Q of degree 4 (relative error 3e-17). The constants are held as a high
//    part, whose products and sums are exact, and a low part that joins the
//    small terms, so that one rounding of the size of the result is left
//    (0.51 ulp). From the 64th interval on z is halved, and the last centre
//    is 2: near u = 1 only r is left, with its relative accuracy.
//  - cos, sin of 2 pi u: modulo half a turn u is a 22-bit fraction of
//    (-1/4, 1/4) turn, exactly; minimax polynomials there (cosine of degree
//    8 in the square, error 4e-18; sine of degree 8, relative error 3e-19)
//    and the sign of the half turn on the radius. ROUND_ANGLE turns the
//    result by the rounding error of the product 2 pi u, so that it is the
//    sine and cosine of the rounded angle: the Heston derivatives near v = 0
//    magnify a change of 4e-16 in a normal a hundred thousand times, and a
//    64-bit reference takes the functions of the rounded product.
//  - sqrt by Goldschmidt's iteration from v_rsq_f64 with a final correction;
//    the argument is -2 ln u in [1.1e-7, 33.3].
//  - exp z for |z| < 700: z = n ln2/64 + r, a table of 2^(i/64) and a
//    polynomial of degree 5; the library's exp elsewhere.
// Coefficients: interpolation at Chebyshev nodes in 60-digit arithmetic.
// The tables (3.5 KB) are computed by the workgroup into LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fp64_tables.h"

namespace mcp {

struct F64Tables {
  double2 lg[128];   // 1/c to 24 bits, high part of -2 ln c (of c/2 from entry 64)
  double lo[128];    // its low part
  double ex[64];     // 2^(i/64)
};

// Every thread of the workgroup; __syncthreads() before the first use.
__device__ __forceinline__ void f64_tables_fill(F64Tables& t) {
  for (uint32_t i = threadIdx.x; i < 128u; i += blockDim.x) {
    t.lg[i] = make_double2(kLogHi[i][0], kLogHi[i][1]);
    t.lo[i] = kLogLo[i];
    if (i < 64u) t.ex[i] = kExp[i];
  }
}

// -2 ln u(w), u(w) = (2 (w >> 9) + 1) 2^-24.
__device__ __forceinline__ double neg2_log_f64(uint32_t w, const F64Tables& t) {
  const double m = (double)((w & 0xFFFFFE00u) | 0x100u);       // u 2^32
  const uint32_t hi = (uint32_t)__double2hiint(m), lo = (uint32_t)__double2loint(m);
  const uint32_t i = (hi >> 13) & 127u;
  const double2 e = t.lg[i];
  const double z = __hiloint2double((int)((hi & 0xFFFFFu) | 0x3FF00000u), (int)lo);
  const double k = (double)((int)((hi + 0x80000u) >> 20) - (1023 + 32));
  const double r = fma(z, e.x, -1.0);
  double q = 0x1.5556988b99fbap-2;
  q = fma(q, r, -0x1.999b0afc28e8ap-2);
  q = fma(q, r, 0x1.ffffffffae630p-2);
  q = fma(q, r, -0x1.5555555526b28p-1);
  q = fma(q, r, 1.0);
  const double small = fma(r * r, q, fma(r, -2.0, fma(k, -0x1.ef35793c7673p-44, t.lo[i])));
  return fma(k, -0x1.62e42fefa38p+0, e.y) + small;
}

// sqrt(x) of a positive x well inside the normal range.
__device__ __forceinline__ double sqrt_pos_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  return fma(fma(-g, g, x), h, g);
}

template <bool ROUND_ANGLE>
__device__ __forceinline__ void box_muller_f64(uint32_t w_rad, uint32_t w_ang,
                                               const F64Tables& t, double& z0, double& z1) {
  const double rad = sqrt_pos_f64(neg2_log_f64(w_rad, t));
  // The angle modulo half a turn: x pi / 2^32, |x| < 2^31.
  const double x = (double)(int)(((w_ang << 1) & 0xFFFFFC00u) | 0x200u);
  const double y = x * x;
  double c = 0x1.1678f9078a9b3p-530;
  c = fma(c, y, -0x1.b6957b54dd389p-462);
  c = fma(c, y, 0x1.f9d254582ac30p-394);
  c = fma(c, y, -0x1.a6d1efc8c38bep-326);
  c = fma(c, y, 0x1.e1f506813a321p-259);
  c = fma(c, y, -0x1.55d3c7e3bfbf5p-192);
  c = fma(c, y, 0x1.03c1f081b5992p-126);
  c = fma(c, y, -0x1.3bd3cc9be45dbp-62);
  c = fma(c, y, 1.0);
  double s = 0x1.9d462020fcc78p-565;
  s = fma(s, y, -0x1.6f7acdb8f6580p-496);
  s = fma(s, y, 0x1.e8f3675ee37ddp-428);
  s = fma(s, y, -0x1.e3074dfaf87afp-360);
  s = fma(s, y, 0x1.5078348551854p-292);
  s = fma(s, y, -0x1.32d2cce627c86p-225);
  s = fma(s, y, 0x1.466bc6775aa7dp-159);
  s = fma(s, y, -0x1.4abbce625be52p-94);
  s = fma(s, y, 0x1.921fb54442d18p-31);
  // Half turns taken off: 0, 1 or 2; an odd number flips both signs.
  const uint32_t flip = (w_ang ^ (w_ang << 1)) & 0x80000000u;
  const double rs = __hiloint2double(__double2hiint(rad) ^ (int)flip, __double2loint(rad));
  s *= x;
  if constexpr (ROUND_ANGLE) {
    // 2 pi = C + 0x1.1a62633145c07p-52; u 2^32 = m; the product C m rounds by
    // fma(C, m, -round(C m)).
    const double m = (double)((w_ang & 0xFFFFFE00u) | 0x100u), C = 0x1.921fb54442d18p+2;
    const double e = fma(-0x1.1a62633145c07p-52, m, -fma(C, m, -(C * m))) * 0x1p-32;
    const double c0 = c;
    c = fma(-e, s, c);
    s = fma(e, c0, s);
  }
  z0 = rs * c;
  z1 = rs * s;
}

__device__ __forceinline__ double exp_f64(double z, const F64Tables& t) {
  if (!(fabs(z) < 700.0)) return exp(z);
  const double magic = 0x1.8p+52;                  // rounds to a multiple of 1/64 in log2
  const double tn = fma(z, 0x1.71547652b82fep+6, magic);
  const int n = __double2loint(tn);
  const double nd = tn - magic;
  const double r = fma(nd, -0x1.f473de6af278fp-36, fma(nd, -0x1.62e42fe000000p-7, z));
  double q = 0x1.11111d9625013p-7;
  q = fma(q, r, 0x1.55556b3e385f1p-5);
  q = fma(q, r, 0x1.5555555555252p-3);
  q = fma(q, r, 0x1.ffffffffff574p-2);
  const double p = fma(r * r, q, r);               // e^r - 1
  const double T = t.ex[n & 63];
  const double v = fma(T, p, T);
  return __hiloint2double(__double2hiint(v) + (int)((uint32_t)(n & ~63) << 14),
                          __double2loint(v));
}

}  // namespace mcp
