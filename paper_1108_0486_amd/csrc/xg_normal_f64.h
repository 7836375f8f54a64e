// FP64 normal variates of the 64-bit member (gfx950): the Box-Muller map on a
// pair of 64-bit generator outputs.
//
// u1 = ((e >> 11) + 1) 2^-53 in (0, 1] and u2 = (o >> 11) 2^-53 in [0, 1) are
// exact; z0 = rho cos(2 pi u2), z1 = rho sin(2 pi u2), rho = sqrt(-2 ln u1).
//
// The logarithm, root, sine and cosine are written for these arguments alone
// (u1 normal and at most 1, an angle already reduced to an eighth turn), which
// leaves out the special cases, the second angle reduction and the extended
// precision of general library functions: 133 VALU instructions per pair with
// the two generator words, where a pair through the device library's log,
// sqrt and sincospi took about 390.  VALU issue bounds the kernel: 2048 streams
// x 2^17 normals went from 1389 us to 590 us (1.55 to 3.6 TB/s).  Against a
// 113-bit reference over 2^18 normals the results are nearer than the
// library's functions gave: at most 1.93 ulp off (before 2.33), a root mean
// square relative error of 6.7e-17 (before 8.1e-17).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace xg {
namespace dev {

// Coefficients (constant term first) and their errors: normal_f64_fit.py.
constexpr double kLog[7] = {0x1.5555555555558p-1, 0x1.99999999952e2p-2, 0x1.2492492df148dp-2, 0x1.c71c62e5800a1p-3,
                            0x1.7462b4ab2ef6bp-3, 0x1.39fe606542ddep-3, 0x1.2b584aae78a57p-3};
constexpr double kSin[6] = {-0x1.4abbce625be52p+2, 0x1.466bc6775a476p+1, -0x1.32d2cce500387p-1,
                            0x1.50783208843ebp-4,  -0x1.e3027dea82bd7p-8, 0x1.e4a9d9166f052p-12};
constexpr double kCos[7] = {-0x1.3bd3cc9be45dep+2, 0x1.03c1f081b5ac0p+2,  -0x1.55d3c7e3cb241p+0, 0x1.e1f5068688d5bp-3,
                            -0x1.a6d1eef479be1p-6, 0x1.f9ce245cada0bp-10, -0x1.b2f3eb054afcdp-14};
constexpr double kLn2Hi64 = 0x1.62e42fefa39efp-1, kLn2Lo64 = 0x1.abc9e3b39803fp-56;
constexpr double kPiHi64 = 0x1.921fb54442d18p+1, kPiLo64 = 0x1.1a62633145c07p-53;

// The constants in scalar registers, set up once before a loop.  (Left to
// itself the compiler copies each coefficient to the destination of an adding
// form of the FMA first, 18 further instructions per pair.)
struct ConstsF64 {
  double log[7], sin[6], cos[7], ln2_hi, ln2_lo, pi_hi, pi_lo;
};

__device__ __forceinline__ double scalar_const(double c) {
  asm volatile("" : "+s"(c));
  return c;
}

__device__ __forceinline__ ConstsF64 consts_f64() {
  ConstsF64 k;
#pragma unroll
  for (int i = 0; i < 7; ++i) k.log[i] = scalar_const(kLog[i]);
#pragma unroll
  for (int i = 0; i < 6; ++i) k.sin[i] = scalar_const(kSin[i]);
#pragma unroll
  for (int i = 0; i < 7; ++i) k.cos[i] = scalar_const(kCos[i]);
  k.ln2_hi = scalar_const(kLn2Hi64);
  k.ln2_lo = scalar_const(kLn2Lo64);
  k.pi_hi = scalar_const(kPiHi64);
  k.pi_lo = scalar_const(kPiLo64);
  return k;
}

// The functions below work on P independent arguments at once, step by step,
// so that a wavefront alone on its SIMD has P chains in flight.
template <int P, int N>
__device__ __forceinline__ void horner(const double (&c)[N], const double (&x)[P], double (&p)[P]) {
#pragma unroll
  for (int u = 0; u < P; ++u) p[u] = fma(c[N - 1], x[u], c[N - 2]);
#pragma unroll
  for (int i = N - 3; i >= 0; --i) {
#pragma unroll
    for (int u = 0; u < P; ++u) p[u] = fma(p[u], x[u], c[i]);
  }
}

// The reduction and the form of the sum are those of the published logarithm of
// Sun's fdlibm (e_log.c); the polynomial and the quotient are this file's own.
// ln u1 = k ln 2 + ln m with m = u1 2^-k in [0.7071, 1.4142) (the exponent is
// taken after adding 1 - 0.7071 to u1's high word, so that u1 just below 1 has
// k = 0 and f = m - 1 is exact).  With s = f / (2 + f), ln m = 2 s + s z Q(z),
// z = s^2, and 2 s = f - s f, so ln m = f - s (f - z Q(z)): only the small
// second term carries s's rounding.  The quotient is the hardware reciprocal
// (24 bits) with one Newton step and one correction by the exact remainder.
template <int P>
__device__ __forceinline__ void ln_u1(const ConstsF64 &K, const uint64_t (&e)[P], double (&ln)[P]) {
  double k[P], f[P], s[P], z[P], q[P];
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const uint32_t ehi = (uint32_t)(e[u] >> 32), elo = (uint32_t)e[u] >> 11;
    const double u1 = fma((double)ehi, 0x1p-32, fma((double)elo, 0x1p-53, 0x1p-53));  // exact
    const uint64_t b = (uint64_t)__double_as_longlong(u1);
    const uint32_t hx = (uint32_t)(b >> 32) + (0x3FF00000u - 0x3FE6A09Eu);
    k[u] = (double)((int32_t)(hx >> 20) - 0x3FF);
    const uint32_t mh = (hx & 0xFFFFFu) + 0x3FE6A09Eu;
    const double m = __longlong_as_double((long long)(((uint64_t)mh << 32) | (uint32_t)b));
    f[u] = m - 1.0;
    s[u] = m + 1.0;
  }
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const double d = s[u];
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    const double t = f[u] * r;
    s[u] = fma(r, fma(-d, t, f[u]), t);
    z[u] = s[u] * s[u];
  }
  horner(K.log, z, q);
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const double g = fma(-z[u], q[u], f[u]);
    ln[u] = fma(k[u], K.ln2_hi, fma(k[u], K.ln2_lo, fma(-s[u], g, f[u])));
  }
}

// sqrt(x) as g + t, |t| tiny, for x = 0 or a normal number above 2^-54: the
// hardware reciprocal square root (24 bits), one Newton step (46 bits), and
// the correction t by the exact remainder, left unadded.
template <int P>
__device__ __forceinline__ void sqrt_parts(const double (&x)[P], double (&g)[P], double (&t)[P]) {
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const double y = __builtin_amdgcn_rsq(__builtin_fmax(x[u], 0x1p-100));  // x = 0 gives g = t = 0
    const double h = 0.5 * y;
    g[u] = x[u] * y;
    g[u] = fma(g[u], fma(-h, g[u], 0.5), g[u]);
    t[u] = h * fma(-g[u], g[u], x[u]);
  }
}

// cos and sin of 2 pi u2.  The angle is reduced exactly on the word as in
// dev::sincos_turn: adding 2^61 to o leaves the quadrant q in bits 63:62 and
// (o's low 11 bits cleared) 2^61 + f 2^63 in bits 61:0, |f| <= 1/4.  Odd q
// swaps the two; the signs come from the sum.  ORDERED = false leaves out the
// swap: (c, s) are the two values in an order that depends on q.
template <bool ORDERED, int P>
__device__ __forceinline__ void sincos_turn_f64(const ConstsF64 &K, const uint64_t (&o)[P], double (&c)[P],
                                                double (&s)[P]) {
  uint32_t hi[P];
  double f[P], t[P], sp[P], cp[P];
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const uint64_t qf = o[u] + (1ull << 61);
    hi[u] = (uint32_t)(qf >> 32);
    const uint32_t lo = (uint32_t)qf & 0xFFFFF800u;
    f[u] = fma((double)(hi[u] & 0x3FFFFFFFu), 0x1p-31, fma((double)lo, 0x1p-63, -0.25));  // exact
    t[u] = f[u] * f[u];
  }
  horner(K.sin, t, sp);
  horner(K.cos, t, cp);
#pragma unroll
  for (int u = 0; u < P; ++u) {
    sp[u] = fma(f[u], K.pi_hi, f[u] * fma(sp[u], t[u], K.pi_lo));  // sin(pi f)
    cp[u] = fma(cp[u], t[u], 1.0);                             // cos(pi f)
    const bool odd = ORDERED && ((hi[u] >> 30) & 1u) != 0u;
    const double c0 = odd ? sp[u] : cp[u], s0 = odd ? cp[u] : sp[u];
    // Ordered: the cosine is negative in quadrants 1 and 2, the sine in 2 and
    // 3.  Unordered: cos(pi f) turns negative where the sine does, and the
    // other way round (see sincos_turn_unordered).
    const uint64_t sign_s = (uint64_t)(hi[u] & 0x80000000u) << 32;
    const uint64_t sign_c = (uint64_t)((hi[u] + 0x40000000u) & 0x80000000u) << 32;
    c[u] = __longlong_as_double((long long)((uint64_t)__double_as_longlong(c0) ^ (ORDERED ? sign_c : sign_s)));
    s[u] = __longlong_as_double((long long)((uint64_t)__double_as_longlong(s0) ^ (ORDERED ? sign_s : sign_c)));
  }
}

// P pairs.  The products take rho as the unrounded sum of its two parts.
template <bool ORDERED, int P>
__device__ __forceinline__ void box_muller_f64(const ConstsF64 &K, const uint64_t (&e)[P], const uint64_t (&o)[P],
                                               double (&z0)[P], double (&z1)[P]) {
  double x[P], g[P], t[P], c[P], s[P];
  ln_u1(K, e, x);
#pragma unroll
  for (int u = 0; u < P; ++u) x[u] *= -2.0;
  sqrt_parts(x, g, t);
  sincos_turn_f64<ORDERED>(K, o, c, s);
#pragma unroll
  for (int u = 0; u < P; ++u) {
    z0[u] = fma(g[u], c[u], t[u] * c[u]);
    z1[u] = fma(g[u], s[u], t[u] * s[u]);
  }
}

}  // namespace dev
}  // namespace xg
