// Device building blocks: counter-based Philox4x32-10, uniform lattices and
// Box-Muller, coefficient-function evaluation, domain test / projection and
// wavefront reductions.  Everything is a header so the compiler can inline it
// into each kernel instantiation.
#pragma once
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#include <stdint.h>
#endif

#include "pdd_internal.hpp"

namespace pdd {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 products
// and xors.  The key (the seed) is uniform across a wavefront, so the key
// schedule stays in scalar registers.  The three-way xors are single
// three-input bitwise operations (truth table 0x96 = a ^ b ^ c).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ void philox4x32_10(uint32_t& c0, uint32_t& c1, uint32_t& c2, uint32_t& c3,
                                              uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// ---------------------------------------------------------------------------
// Uniforms on open lattices and Gaussians.
//   QUAD24: u = (2 (w >> 9) + 1) 2^-24 (exact in FP32)
//   PAIR52: u = (2 k + 1) 2^-53, k = (w_hi << 20) | (w_lo >> 12) (exact in FP64)
// Box-Muller: z0 = r cos(2 pi u_b), z1 = r sin(2 pi u_b), r = sqrt(-2 ln u_a).
__device__ __forceinline__ float u24f(uint32_t w) {
  // 0x3F800000 | (w >> 9) is the float 1 + (w >> 9) 2^-23 in [1, 2) (one
  // funnel shift of 0x7F:w); subtracting 1 - 2^-24 is exact and leaves
  // (2 (w >> 9) + 1) 2^-24.
  const uint32_t bits = __builtin_amdgcn_alignbit(0x7Fu, w, 9);
  return __builtin_bit_cast(float, bits) - 0x1.fffffep-1f;
}
__device__ __forceinline__ double u24d(uint32_t w) {
  return (double)(w >> 9) * 0x1p-23 + 0x1p-24;
}
__device__ __forceinline__ double u52d(uint32_t whi, uint32_t wlo) {
  const uint64_t k = ((uint64_t)whi << 20) | (uint64_t)(wlo >> 12);
  return (double)k * 0x1p-52 + 0x1p-53;
}

// FP32 Box-Muller on the hardware transcendental units: v_log_f32 is log2,
// v_sin/v_cos_f32 take their argument in revolutions, so 2 pi u needs no
// multiply.  -2 ln u = -2 ln2 log2 u.
__device__ __forceinline__ void box_muller_f(float ua, float ub, float& z0, float& z1) {
  const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(ua));
  z0 = r * __builtin_amdgcn_cosf(ub);
  z1 = r * __builtin_amdgcn_sinf(ub);
}
// FP64 Box-Muller from the library functions: for walk on spheres, whose jumps
// amplify rounding differences (a path of 35 jumps turned two ulps of a
// Gaussian into 8e-12 of its value), so that its paths follow the plain
// formula's rounding.
__device__ __forceinline__ void box_muller_libm(double ua, double ub, double& z0, double& z1) {
  const double r = sqrt(-2.0 * log(ua));
  double s, c;
  sincos(2.0 * 3.14159265358979323846 * ub, &s, &c);
  z0 = r * c;
  z1 = r * s;
}

// FP64 Box-Muller.  The FP64 walks spend most of their time here, and most of
// that in what general log / sqrt / sincos do for arguments that a uniform on
// an open lattice cannot be: zero, subnormals, infinities, large angles.
// Here u_a is in [2^-53, 1 - 2^-53], so -2 ln u_a in [2^-52, 74], and the
// angle is reduced in units of a quarter turn, which is exact for u_b in
// (0, 1) (2 pi u_b itself would be rounded first).  About 75 FP64 operations
// instead of about 250; the Gaussians are as close to their exact values as
// before or closer (against 113-bit values, in ulps of r, over 3 10^6 pairs of
// both lattices and their ends: largest error 2.0 against 6.2 of log, sqrt
// and sincos of the rounded angle, mean 0.42 against 1.08).
//
// -2 ln u (u normal): u = m 2^e with m in [sqrt(1/2), sqrt 2), ln m =
// 2 atanh(s), s = (m - 1) / (m + 1) carried as s + sl; the polynomial is
// (2 atanh(s) - 2 s) / s^3 in s^2, interpolated at Chebyshev points (relative
// error of ln m below 2^-57).
__device__ __forceinline__ double neg2_log_unit(double u) {
  double m = __builtin_amdgcn_frexp_mant(u);        // [1/2, 1)
  int e = __builtin_amdgcn_frexp_exp(u);
  const bool low = m < 0x1.6a09e667f3bcdp-1;        // sqrt(1/2)
  m = low ? m + m : m;
  e -= low ? 1 : 0;
  const double f = m - 1.0;                         // exact
  const double d = m + 1.0;
  const double dl = m - (d - 1.0);                  // d + dl = m + 1
  double r = __builtin_amdgcn_rcp(d);               // about 2^-24; two Newton steps
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  const double s = f * r;
  const double sl = fma(-s, dl, fma(-s, d, f)) * r;
  const double z = s * s;
  double p = 0x1.2b5bd9a316a24p-3;
  p = fma(p, z, 0x1.39fe16ad885a7p-3);
  p = fma(p, z, 0x1.7462b6e311a89p-3);
  p = fma(p, z, 0x1.c71c62ddb431bp-3);
  p = fma(p, z, 0x1.2492492df7663p-2);
  p = fma(p, z, 0x1.99999999952abp-2);
  p = fma(p, z, 0x1.5555555555558p-1);
  const double ed = (double)e;
  // low-order part: 2 sl + s^3 p + e (ln 2 - its double)
  const double lo = fma(s * z, p, fma(2.0, sl, ed * 0x1.abc9e3b39803fp-56));
  return -2.0 * (fma(ed, 0x1.62e42fefa39efp-1, 2.0 * s) + lo);
}

// sqrt of a normal x: Goldschmidt iterations from the hardware reciprocal
// square root, the last two corrected by the exact residual x - g^2.
__device__ __forceinline__ double sqrt_normal(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, x), h, g);
  return fma(fma(-g, g, x), h, g);
}

__device__ __forceinline__ void box_muller_d(double ua, double ub, double& z0, double& z1) {
  const double r = sqrt_normal(neg2_log_unit(ua));
  // 4 u_b = q + f, |f| <= 1/2 (adding 1.5 2^52 rounds to a whole number and
  // leaves it in the low bits); f is exact
  const double t = 4.0 * ub;
  const double qm = t + 0x1.8p52;
  const uint32_t q = (uint32_t)__builtin_bit_cast(uint64_t, qm);
  const double f = t - (qm - 0x1.8p52);
  const double f2 = f * f;
  // sin and cos of f pi / 2
  double ps = 0x1.e4a9d9166f052p-25;
  ps = fma(ps, f2, -0x1.e3027dea82bd7p-19);
  ps = fma(ps, f2, 0x1.50783208843ebp-13);
  ps = fma(ps, f2, -0x1.32d2cce500387p-8);
  ps = fma(ps, f2, 0x1.466bc6775a476p-4);
  ps = fma(ps, f2, -0x1.4abbce625be52p-1);
  const double sf = fma(f, 0x1.921fb54442d18p+0, f * fma(ps, f2, 0x1.1a62633145c07p-54));
  double pc = -0x1.b2f3eb054afcdp-28;
  pc = fma(pc, f2, 0x1.f9ce245cada0bp-22);
  pc = fma(pc, f2, -0x1.a6d1eef479be1p-16);
  pc = fma(pc, f2, 0x1.e1f5068688d5bp-11);
  pc = fma(pc, f2, -0x1.55d3c7e3cb241p-6);
  pc = fma(pc, f2, 0x1.03c1f081b5ac0p-2);
  pc = fma(pc, f2, -0x1.3bd3cc9be45dep+0);
  const double cf = fma(pc, f2, 1.0);
  const bool odd = (q & 1u) != 0u;
  const double c = odd ? sf : cf, s = odd ? cf : sf;
  // cos is negative in the second and third quarter turn, sin in the last two
  const double rc = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, r) ^ ((uint64_t)((q + 1u) & 2u) << 62));
  const double rs = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, r) ^ ((uint64_t)(q & 2u) << 62));
  z0 = rc * c;
  z1 = rs * s;
}

// The Gaussians of one Philox block.  LIBM: box_muller_libm in FP64.
template <typename R, int LAYOUT, bool LIBM = false>
struct Normals {
  static constexpr int kPerBlock = LAYOUT == RNG_QUAD24 ? 4 : 2;
  __device__ __forceinline__ static void pair(R ua, R ub, R* z) {
    if constexpr (sizeof(R) == 4) box_muller_f(ua, ub, z[0], z[1]);
    else if constexpr (LIBM) box_muller_libm(ua, ub, z[0], z[1]);
    else box_muller_d(ua, ub, z[0], z[1]);
  }
  __device__ __forceinline__ static void from_words(const uint32_t* w, R* z) {
    if constexpr (sizeof(R) == 4) {
      pair(u24f(w[0]), u24f(w[1]), z);
      pair(u24f(w[2]), u24f(w[3]), z + 2);
    } else if constexpr (LAYOUT == RNG_QUAD24) {
      pair(u24d(w[0]), u24d(w[1]), z);
      pair(u24d(w[2]), u24d(w[3]), z + 2);
    } else {
      pair(u52d(w[0], w[1]), u52d(w[2], w[3]), z);
    }
  }
  __device__ __forceinline__ static void gen(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                             uint32_t k1, R* z) {
    uint32_t w[4] = {c0, c1, c2, c3};
    philox4x32_10(w[0], w[1], w[2], w[3], k0, k1);
    from_words(w, z);
  }
};

// ---------------------------------------------------------------------------
// Elementary functions per precision.  FP32 uses the hardware exp2 / sin / cos
// units (inputs here stay far inside their valid ranges); FP64 uses the
// accurate library routines.
__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ __forceinline__ double fexp(double x) { return exp(x); }
__device__ __forceinline__ float fsin(float x) { return __builtin_amdgcn_sinf(x * 0.15915494309189535f); }
__device__ __forceinline__ double fsin(double x) { return sin(x); }
__device__ __forceinline__ float fcos(float x) { return __builtin_amdgcn_cosf(x * 0.15915494309189535f); }
__device__ __forceinline__ double fcos(double x) { return cos(x); }
__device__ __forceinline__ float ftanh(float x) {
  // tanh x = 1 - 2 / (e^{2x} + 1); saturates correctly at both ends.
  const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}
__device__ __forceinline__ double ftanh(double x) { return tanh(x); }

// Read-only tables (factor records, coefficients) are read through the
// constant address space, which compiles to scalar loads: the records are
// wave-uniform, so their fields land in scalar registers and the switch over
// the factor's function becomes a uniform branch.  The empty asm statement
// hides the table address from the optimiser, so the loads stay next to
// their use instead of being hoisted out of the stepping loop into scalar
// registers that would then spill.
#define PDD_CONST_AS __attribute__((address_space(4)))

template <typename T>
__device__ __forceinline__ const T PDD_CONST_AS* const_table(const T* p) {
  uint64_t a = reinterpret_cast<uint64_t>(p);
  asm volatile("" : "+s"(a));
  return (const T PDD_CONST_AS*)a;
}

template <typename R>
__device__ __forceinline__ R fac_a(const DevFactor& f);
template <>
__device__ __forceinline__ float fac_a<float>(const DevFactor& f) { return f.af; }
template <>
__device__ __forceinline__ double fac_a<double>(const DevFactor& f) { return f.ad; }
template <typename R>
__device__ __forceinline__ R fac_b(const DevFactor& f);
template <>
__device__ __forceinline__ float fac_b<float>(const DevFactor& f) { return f.bf; }
template <>
__device__ __forceinline__ double fac_b<double>(const DevFactor& f) { return f.bd; }

template <typename R>
__device__ __forceinline__ R coef_at(const double* __restrict__ cd, const float* __restrict__ cf, int i);
template <>
__device__ __forceinline__ float coef_at<float>(const double* __restrict__, const float* __restrict__ cf, int i) {
  return cf[i];
}
template <>
__device__ __forceinline__ double coef_at<double>(const double* __restrict__ cd, const float* __restrict__, int i) {
  return cd[i];
}

// Coordinate d of x (DIM coordinates; DIM = 4 when a time argument follows
// three space coordinates).
template <typename R, int DIM>
__device__ __forceinline__ R pick(const R* x, int d) {
  if (DIM == 1) return x[0];
  if (DIM == 2) return d == 0 ? x[0] : x[1];
  if (DIM == 3) return d == 0 ? x[0] : (d == 1 ? x[1] : x[2]);
  return d == 0 ? x[0] : (d == 1 ? x[1] : (d == 2 ? x[2] : x[3]));
}

// One factor.  The factor record is wave-uniform (scalar loads), so the switch
// is a uniform branch.
template <typename R, int DIM>
__device__ __forceinline__ R factor_value(const DevFactor& fa, const R* x) {
  const R s = fac_a<R>(fa) * pick<R, DIM>(x, fa.dim) + fac_b<R>(fa);
  R v;
  switch (fa.fn) {
    case FN_EXP: v = fexp(s); break;
    case FN_SIN: v = fsin(s); break;
    case FN_COS: v = fcos(s); break;
    case FN_TANH: v = ftanh(s); break;
    default: v = s; break;
  }
  R r = (R)1;
  for (int k = 0; k < fa.power; ++k) r *= v;
  return r;
}

// factor_value with the function and the power fixed at compile time (the
// form used by problem-specialised kernels): the same operations in the same
// order, so it returns the same bits.
template <typename R, int DIM, int FN, int POW>
__device__ __forceinline__ R factor_fixed(const R* x, int d, R a, R b) {
  const R s = a * pick<R, DIM>(x, d) + b;
  R v;
  if constexpr (FN == FN_EXP) v = fexp(s);
  else if constexpr (FN == FN_SIN) v = fsin(s);
  else if constexpr (FN == FN_COS) v = fcos(s);
  else if constexpr (FN == FN_TANH) v = ftanh(s);
  else v = s;
  R r = (R)1;
#pragma unroll
  for (int k = 0; k < POW; ++k) r *= v;
  return r;
}

// Product of the factors of term t (without its coefficient).
template <typename R, int DIM>
__device__ __forceinline__ R term_value(const DevFactor* __restrict__ fac, const DevFun& F, int t, const R* x) {
  R v = (R)1;
  const DevFactor PDD_CONST_AS* tf = const_table(fac) + F.fac_off + t * F.n_factors;
  for (int j = 0; j < F.n_factors; ++j) {
    DevFactor fa;
    fa.fn = tf[j].fn;
    fa.dim = tf[j].dim;
    fa.power = tf[j].power;
    fa.af = tf[j].af;
    fa.bf = tf[j].bf;
    fa.ad = tf[j].ad;
    fa.bd = tf[j].bd;
    v *= factor_value<R, DIM>(fa, x);
  }
  return v;
}

template <typename R>
__device__ __forceinline__ R coef_const(const double* __restrict__ cd, const float* __restrict__ cf, int i);
template <>
__device__ __forceinline__ float coef_const<float>(const double* __restrict__, const float* __restrict__ cf, int i) {
  return const_table(cf)[i];
}
template <>
__device__ __forceinline__ double coef_const<double>(const double* __restrict__ cd, const float* __restrict__, int i) {
  return const_table(cd)[i];
}

template <typename R, int DIM>
__device__ __forceinline__ R terms_sum(const DevFactor* __restrict__ fac, const double* __restrict__ cd,
                                       const float* __restrict__ cf, const DevFun& F, const R* x) {
  R s = (R)0;
  for (int t = 0; t < F.n_terms; ++t) s += coef_const<R>(cd, cf, F.coef_off + t) * term_value<R, DIM>(fac, F, t, x);
  return s;
}

// Dense polynomial of runtime degree, coefficients in nested order
// (a outer, b middle, c inner), evaluated with running products.
template <typename R, int DIM>
__device__ __forceinline__ R poly_nested(const double* __restrict__ cd, const float* __restrict__ cf, int deg,
                                         int off, const R* x) {
  R s = (R)0;
  int idx = off;
  R xa = (R)1;
  for (int a = 0; a <= deg; ++a) {
    if (DIM == 1) {
      s += coef_at<R>(cd, cf, idx++) * xa;
    } else {
      R xb = xa;
      for (int b = 0; b <= deg - a; ++b) {
        if (DIM == 2) {
          s += coef_at<R>(cd, cf, idx++) * xb;
        } else {
          R xc = xb;
          for (int c = 0; c <= deg - a - b; ++c) {
            s += coef_at<R>(cd, cf, idx++) * xc;
            xc *= x[2];
          }
        }
        xb *= x[1];
      }
    }
    xa *= x[0];
  }
  return s;
}

// s + the N coefficients from idx on times xp, xp x, xp x^2, ..
template <typename R, int N>
__device__ __forceinline__ R poly_row(const double* __restrict__ cd, const float* __restrict__ cf, int idx, R s, R xp,
                                      R x) {
  R c[N];
#pragma unroll
  for (int k = 0; k < N; ++k) c[k] = coef_at<R>(cd, cf, idx + k);
#pragma unroll
  for (int k = 0; k < N; ++k) {
    s += c[k] * xp;
    xp *= x;
  }
  return s;
}

// poly_nested with straight code for each length of a row of the innermost
// variable, its coefficients read together, in place of a load, a wait and a
// branch for each (the same operations in the same order).  For the forward
// walks: 4096 nodes x 10000 paths on a ball, g of 120 monomials, 25.3 -> 24.5
// ms; the adjoint walk lost 1 to 2% with it (84.5 -> 85.2 ms at 4096 x 20000).
template <typename R, int DIM>
__device__ __forceinline__ R poly_rows(const double* __restrict__ cd, const float* __restrict__ cf, int deg,
                                         int off, const R* x) {
  R s = (R)0;
  int idx = off;
  auto row = [&](int n, R xp) {
    switch (n) {
      case 1: s = poly_row<R, 1>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      case 2: s = poly_row<R, 2>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      case 3: s = poly_row<R, 3>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      case 4: s = poly_row<R, 4>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      case 5: s = poly_row<R, 5>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      case 6: s = poly_row<R, 6>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      case 7: s = poly_row<R, 7>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      case 8: s = poly_row<R, 8>(cd, cf, idx, s, xp, x[DIM - 1]); break;
      default:
        for (int k = 0; k < n; ++k) {
          s += coef_at<R>(cd, cf, idx + k) * xp;
          xp *= x[DIM - 1];
        }
    }
    idx += n;
  };
  if constexpr (DIM == 1) {
    row(deg + 1, (R)1);
  } else {
    R xa = (R)1;
    for (int a = 0; a <= deg; ++a) {
      if constexpr (DIM == 2) {
        row(deg - a + 1, xa);
      } else {
        R xb = xa;
        for (int b = 0; b <= deg - a; ++b) {
          row(deg - a - b + 1, xb);
          xb *= x[1];
        }
      }
      xa *= x[0];
    }
  }
  return s;
}

// Graded-lexicographic monomial table of total degree <= D in DIM variables,
// built at compile time so that fully unrolled loops index registers only.
constexpr int binom(int n, int k) {
  int r = 1;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}
template <int DIM, int D>
struct GradedLex {
  static constexpr int N = D < 0 ? 0 : binom(D + DIM, DIM);
  int e[N > 0 ? N : 1][3];
  constexpr GradedLex() : e{} {
    int m = 0;
    for (int k = 0; k <= D; ++k) {
      if (DIM == 1) {
        e[m][0] = k; e[m][1] = 0; e[m][2] = 0; ++m;
      } else if (DIM == 2) {
        for (int a = k; a >= 0; --a) { e[m][0] = a; e[m][1] = k - a; e[m][2] = 0; ++m; }
      } else {
        for (int a = k; a >= 0; --a)
          for (int b = k - a; b >= 0; --b) { e[m][0] = a; e[m][1] = b; e[m][2] = k - a - b; ++m; }
      }
    }
  }
};

// All monomials of degree <= D at x, graded-lex order.  Powers of unused
// coordinates are the constant 1, which the compiler folds away.
template <typename R, int DIM, int D>
__device__ __forceinline__ void monomials(const R* x, R* mono) {
  constexpr GradedLex<DIM, D> T{};
  R p[3][D + 1];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    p[k][0] = (R)1;
#pragma unroll
    for (int j = 1; j <= D; ++j) p[k][j] = (k < DIM) ? p[k][j - 1] * x[k < DIM ? k : 0] : (R)1;
  }
#pragma unroll
  for (int m = 0; m < GradedLex<DIM, D>::N; ++m) mono[m] = p[0][T.e[m][0]] * p[1][T.e[m][1]] * p[2][T.e[m][2]];
}

// ---------------------------------------------------------------------------
// Domain: open box or ball; a boundary point counts as outside.
template <typename R>
struct Dom {
  int kind;
  R lo[3], hi[3], ctr[3], rad, rad2;
};

template <typename R>
__device__ __forceinline__ Dom<R> make_dom(const LinearParams& P);
template <>
__device__ __forceinline__ Dom<float> make_dom<float>(const LinearParams& P) {
  Dom<float> D;
  D.kind = P.dom_kind;
  for (int k = 0; k < 3; ++k) { D.lo[k] = P.lof[k]; D.hi[k] = P.hif[k]; D.ctr[k] = P.ctrf[k]; }
  D.rad = P.radf;
  D.rad2 = P.rad2f;
  return D;
}
template <>
__device__ __forceinline__ Dom<double> make_dom<double>(const LinearParams& P) {
  Dom<double> D;
  D.kind = P.dom_kind;
  for (int k = 0; k < 3; ++k) { D.lo[k] = P.lo[k]; D.hi[k] = P.hi[k]; D.ctr[k] = P.ctr[k]; }
  D.rad = P.rad;
  D.rad2 = P.rad2;
  return D;
}

// Domain of the exit test: D, or D shrunk for the boundary-corrected scheme
// (only the fields the test reads: kind, lo, hi, ctr, rad2).
template <typename R>
__device__ __forceinline__ Dom<R> make_test_dom(const LinearParams& P);
template <>
__device__ __forceinline__ Dom<float> make_test_dom<float>(const LinearParams& P) {
  Dom<float> D;
  D.kind = P.dom_kind;
  for (int k = 0; k < 3; ++k) { D.lo[k] = P.tlof[k]; D.hi[k] = P.thif[k]; D.ctr[k] = P.ctrf[k]; }
  D.rad = P.radf;
  D.rad2 = P.trad2f;
  return D;
}
template <>
__device__ __forceinline__ Dom<double> make_test_dom<double>(const LinearParams& P) {
  Dom<double> D;
  D.kind = P.dom_kind;
  for (int k = 0; k < 3; ++k) { D.lo[k] = P.tlo[k]; D.hi[k] = P.thi[k]; D.ctr[k] = P.ctr[k]; }
  D.rad = P.rad;
  D.rad2 = P.trad2;
  return D;
}

// |d|^2.  In FP32 the fused products are written out: left to the compiler,
// which of the first two products is rounded on its own would depend on the
// code around it, and a path's exit step with it.
template <typename R, int DIM>
__device__ __forceinline__ R norm2(const R* d) {
  if constexpr (sizeof(R) == 4) {
    if constexpr (DIM == 1) return d[0] * d[0];
    R s = __builtin_fmaf(d[0], d[0], d[1] * d[1]);
    if constexpr (DIM == 3) s = __builtin_fmaf(d[2], d[2], s);
    return s;
  } else {
    R s = (R)0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) s += d[k] * d[k];
    return s;
  }
}

template <typename R, int DIM>
__device__ __forceinline__ bool inside(const Dom<R>& D, const R* x) {
  if (D.kind == DOM_BOX) {
    bool in = true;
#pragma unroll
    for (int k = 0; k < DIM; ++k) in = in && (x[k] > D.lo[k]) && (x[k] < D.hi[k]);
    return in;
  }
  R d[DIM];
#pragma unroll
  for (int k = 0; k < DIM; ++k) d[k] = x[k] - D.ctr[k];
  return norm2<R, DIM>(d) < D.rad2;
}

// Distance from x to the boundary of D (negative outside): ball R - |x - c|,
// box min_k min(x_k - lo_k, hi_k - x_k).  FP64: every product and sum rounded
// on its own (no fused multiply-add), so that walk-on-spheres paths, whose
// jumps amplify rounding differences, follow the oracle's arithmetic exactly.
template <typename R, int DIM>
__device__ __forceinline__ R boundary_distance(const Dom<R>& D, const R* x) {
  if constexpr (sizeof(R) == 8) {
#pragma clang fp contract(off)
    if (D.kind == DOM_BOX) {
      R m = x[0] - D.lo[0];
      m = fmin(m, D.hi[0] - x[0]);
#pragma unroll
      for (int k = 1; k < DIM; ++k) {
        m = fmin(m, x[k] - D.lo[k]);
        m = fmin(m, D.hi[k] - x[k]);
      }
      return m;
    }
    R r2 = (R)0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      const R d = x[k] - D.ctr[k];
      r2 += d * d;
    }
    return D.rad - sqrt(r2);
  }
  if (D.kind == DOM_BOX) {
    R m = x[0] - D.lo[0];
    m = fmin(m, D.hi[0] - x[0]);
#pragma unroll
    for (int k = 1; k < DIM; ++k) {
      m = fmin(m, x[k] - D.lo[k]);
      m = fmin(m, D.hi[k] - x[k]);
    }
    return m;
  }
  R d[DIM];
#pragma unroll
  for (int k = 0; k < DIM; ++k) d[k] = x[k] - D.ctr[k];
  return D.rad - sqrt(norm2<R, DIM>(d));
}

// |z|^2 of one jump's Gaussians (FP64 without fused multiply-add, as above).
template <typename R, int DIM>
__device__ __forceinline__ R sum_squares(const R* z) {
  if constexpr (sizeof(R) == 8) {
#pragma clang fp contract(off)
    R s = (R)0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) s += z[k] * z[k];
    return s;
  }
  return norm2<R, DIM>(z);
}

// x += r z / |z| (z2 = |z|^2): FP64 in the order r (z_k / |z|) with every
// operation rounded on its own (IEEE square root and division, no fused
// multiply-add); FP32 with the hardware reciprocal square root.
template <typename R, int DIM>
__device__ __forceinline__ void jump_sphere(R* x, R r, R z2, const R* z);
template <>
__device__ __forceinline__ void jump_sphere<double, 1>(double* x, double r, double z2, const double* z) {
#pragma clang fp contract(off)
  const double zn = sqrt(z2);
  x[0] = x[0] + r * (z[0] / zn);
}
template <>
__device__ __forceinline__ void jump_sphere<double, 2>(double* x, double r, double z2, const double* z) {
#pragma clang fp contract(off)
  const double zn = sqrt(z2);
  for (int k = 0; k < 2; ++k) x[k] = x[k] + r * (z[k] / zn);
}
template <>
__device__ __forceinline__ void jump_sphere<double, 3>(double* x, double r, double z2, const double* z) {
#pragma clang fp contract(off)
  const double zn = sqrt(z2);
  for (int k = 0; k < 3; ++k) x[k] = x[k] + r * (z[k] / zn);
}
template <int DIM>
__device__ __forceinline__ void jump_sphere_f(float* x, float r, float z2, const float* z) {
  const float s = r * __builtin_amdgcn_rsqf(z2);
#pragma unroll
  for (int k = 0; k < DIM; ++k) x[k] = x[k] + s * z[k];
}
template <>
__device__ __forceinline__ void jump_sphere<float, 1>(float* x, float r, float z2, const float* z) {
  jump_sphere_f<1>(x, r, z2, z);
}
template <>
__device__ __forceinline__ void jump_sphere<float, 2>(float* x, float r, float z2, const float* z) {
  jump_sphere_f<2>(x, r, z2, z);
}
template <>
__device__ __forceinline__ void jump_sphere<float, 3>(float* x, float r, float z2, const float* z) {
  jump_sphere_f<3>(x, r, z2, z);
}

// Nearest boundary point.  Outside a box: clamp; inside a box (censored path):
// the nearest face; ball: c + R (x - c)/|x - c| (c + R e_0 at the centre).
template <typename R, int DIM>
__device__ __forceinline__ void project(const Dom<R>& D, const R* x, R* out) {
#pragma unroll
  for (int k = 0; k < 3; ++k) out[k] = (k < DIM) ? x[k] : (R)0;
  if (D.kind == DOM_BOX) {
    if (!inside<R, DIM>(D, x)) {
#pragma unroll
      for (int k = 0; k < DIM; ++k) out[k] = fmin(fmax(x[k], D.lo[k]), D.hi[k]);
    } else {
      int best = 0;
      R bestd = (R)1e30, target = (R)0;
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
        const R dl = x[k] - D.lo[k], dh = D.hi[k] - x[k];
        if (dl < bestd) { bestd = dl; best = k; target = D.lo[k]; }
        if (dh < bestd) { bestd = dh; best = k; target = D.hi[k]; }
      }
#pragma unroll
      for (int k = 0; k < DIM; ++k) if (k == best) out[k] = target;
    }
  } else {
    R d[DIM];
#pragma unroll
    for (int k = 0; k < DIM; ++k) d[k] = x[k] - D.ctr[k];
    const R r = sqrt(norm2<R, DIM>(d));
    if (r == (R)0) {
#pragma unroll
      for (int k = 0; k < DIM; ++k) out[k] = D.ctr[k] + (k == 0 ? D.rad : (R)0);
    } else {
      const R s = D.rad / r;
#pragma unroll
      for (int k = 0; k < DIM; ++k) out[k] = D.ctr[k] + s * (x[k] - D.ctr[k]);
    }
  }
}

// ---------------------------------------------------------------------------
// Wavefront reductions (64 lanes) with butterfly shuffles.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ __forceinline__ int64_t wave_sum(int64_t v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Chan et al. merge of Welford triples (n, mean, m2), written without
// branches (an empty side has n = 0 and mean = 0, which the formulas absorb:
// f = 0 keeps the left triple, f = 1 with n = 0 returns the right one).
__device__ __forceinline__ void chan_merge(double& n, double& mean, double& m2, double nb, double meanb,
                                           double m2b) {
  const double nn = n + nb;
  const double d = meanb - mean;
  const double f = nb / (nn > 0.0 ? nn : 1.0);
  mean = mean + d * f;
  m2 = m2 + m2b + d * d * n * f;
  n = nn;
}

// Butterfly merge; both partners merge (lower lane, upper lane) in that order,
// so every lane ends with the same bits.  Operand order is picked with
// selects, not branches, so the reduction adds no divergent control flow.
__device__ __forceinline__ void wave_welford(double& n, double& mean, double& m2) {
  const int lane = (int)(threadIdx.x & (kWave - 1));
#pragma unroll
  for (int o = 1; o <= 32; o <<= 1) {
    const double nb = __shfl_xor(n, o, kWave);
    const double mb = __shfl_xor(mean, o, kWave);
    const double qb = __shfl_xor(m2, o, kWave);
    const bool up = (lane & o) != 0;
    double an = up ? nb : n, am = up ? mb : mean, aq = up ? qb : m2;
    const double bn = up ? n : nb, bm = up ? mean : mb, bq = up ? m2 : qb;
    chan_merge(an, am, aq, bn, bm, bq);
    n = an;
    mean = am;
    m2 = aq;
  }
}

// Pops the next work-item index for the whole wavefront (call with all lanes
// active).  readfirstlane puts the index in a scalar register, so the
// compiler sees it as wave-uniform and the caller's "queue empty" exit is a
// uniform branch; a per-lane copy (e.g. a shuffle) makes that exit look
// divergent and can leave lanes without a fresh index.
// The atomic is issued by every lane (increment 1 from lane 0, 0 from the
// rest) rather than under `if (lane == 0)`: a lane-divergent branch here, ahead
// of the loop exit that tests the popped index, has been compiled into a
// nested loop whose exit mask was the lane-0 mask, sending lanes 1..63 back
// through the body with a stale index (a wave that never finishes).
__device__ __forceinline__ uint32_t pop_item(uint32_t* qhead) {
  const uint32_t inc = (threadIdx.x & (kWave - 1)) == 0 ? 1u : 0u;
  const uint32_t v = atomicAdd(qhead, inc);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// The wavefronts of a branching launch start on the items of their own numbers
// and pop the rest of the queue: all starting on the queue's one atomic cost 12 ns a
// wavefront (75 us of a 190 us launch of 6000 small items), and with one item
// per wavefront or less the queue is not touched.  The launch's grid is what
// the chip holds at a time, so no item waits for a wavefront yet to start.
__device__ __forceinline__ uint32_t first_item() {
  return blockIdx.x * (kBlock / kWave) + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
}
__device__ __forceinline__ uint32_t next_item(uint32_t* qhead, int n_items) {
  const uint32_t n_waves = gridDim.x * (kBlock / kWave);
  return n_waves < (uint32_t)n_items ? n_waves + pop_item(qhead) : n_waves;
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ int lane_rank(uint64_t mask) {
  // number of set bits of `mask` below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

}  // namespace pdd
