// Device helpers shared by the block kernels: MFMA operand conventions,
// covariance functions, cross-lane moves and reciprocal square roots.
#pragma once
#include <hip/hip_runtime.h>

#include "sbv_internal.h"

namespace sbv {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// MFMA 16x16x4 operand conventions (checked on the device):
//   A (16x4): lane l holds A[l%16][l/16];  B (4x16): lane l holds B[l/16][l%16];
//   C/D:      lane l, register t holds C[row(l/16, t)][l%16] with
//             row = g + 4t for FP64 and 4g + t for FP32.
// The K index of chunk q seen by lane group g is kap(q, g) = row(g, q), so that
// register q of a tile is the A operand of chunk q of its transpose.
template <typename T>
struct MF;
template <>
struct MF<double> {
  typedef d4 acc;
  __device__ static acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static constexpr int row(int g, int t) { return g + 4 * t; }
};
template <>
struct MF<float> {
  typedef f4 acc;
  __device__ static acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static constexpr int row(int g, int t) { return 4 * g + t; }
};

// e^x of the dense covariance matrix (x = -r <= 0): Cody and Waite's reduction
// x = k ln 2 + f, k = rint(x / ln 2), |f| <= ln(2) / 2, with ln 2 split into a
// 42-bit leading part (k ln2_hi is exact for |k| < 2^11) and the rest; then
// e^f = 1 + (f + f^2 P(f)), P the Taylor series of (e^f - 1 - f) / f^2 to
// degree 11 (truncation below 1e-17 relative), evaluated by Estrin's scheme:
// the dependent chain is 6 operations deep against Horner's 13, and adding the 1
// last keeps the error within one ulp; finally scaled by 2^k.  x is clamped at -1000, where e^x is 0.
__device__ __forceinline__ double t_exp(double x) {
  x = fmax(x, -1000.0);
  const double k = rint(x * 0x1.71547652b82fep+0);
  double f = fma(-k, 0x1.62e42fefa3800p-1, x);
  f = fma(-k, 0x1.ef35793c76730p-45, f);
  const double f2 = f * f, f4 = f2 * f2, f8 = f4 * f4;
  const double d0 = fma(f, 0x1.5555555555555p-3, 0x1.0000000000000p-1);
  const double d1 = fma(f, 0x1.1111111111111p-7, 0x1.5555555555555p-5);
  const double d2 = fma(f, 0x1.a01a01a01a01ap-13, 0x1.6c16c16c16c17p-10);
  const double d3 = fma(f, 0x1.71de3a556c734p-19, 0x1.a01a01a01a01ap-16);
  const double d4 = fma(f, 0x1.ae64567f544e4p-26, 0x1.27e4fb7789f5cp-22);
  const double d5 = fma(f, 0x1.6124613a86d09p-33, 0x1.1eed8eff8d898p-29);
  const double e0 = fma(d1, f2, d0), e1 = fma(d3, f2, d2), e2 = fma(d5, f2, d4);
  const double p = fma(e2, f8, fma(e1, f4, e0));
  return __builtin_amdgcn_ldexp(1.0 + fma(f2, p, f), (int)k);
}
// Distance from its square in the dense covariance matrix (r2 >= 0): the
// hardware reciprocal square root (about 23 good bits) refined by one coupled
// Newton-Raphson step for sqrt(r2) and 1/(2 sqrt(r2)) and one residual
// correction (Goldschmidt's square-root iteration as in Markstein's IA-64
// elementary functions), which lands within rounding of the library sqrt.
// Squared distances below 2^-1000 give 0: no covariance entry can tell them
// apart.
__device__ __forceinline__ double g_sqrt(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  double g = r2 * y, h = 0.5 * y;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  g = fma(fma(-g, g, r2), h, g);
  return r2 < 0x1p-1000 ? 0.0 : g;
}

// 16-byte vectors: coordinates in LDS, operand tiles.
template <typename T>
struct ZV;
template <>
struct ZV<double> {
  typedef double v __attribute__((ext_vector_type(2)));
  static constexpr int w = 2;
};
template <>
struct ZV<float> {
  typedef float v __attribute__((ext_vector_type(4)));
  static constexpr int w = 4;
};

// Matern correlation, closed forms of Eq. (maternkernel) for half-integer nu:
// p(r) e^{-r} with p = 1, 1 + r, 1 + r + r^2/3, 1 + r + 2 r^2/5 + r^3/15 for
// nu = 1/2, 3/2, 5/2, 7/2, taken as 1 + r (c1 + r (c2 + r c3)) with the
// coefficients selected once from the (uniform) smoothness (dense covariance matrix).
template <typename T>
__device__ __forceinline__ T matern(T r, int two_nu) {
  const T c1 = two_nu >= 3 ? T(1) : T(0);
  const T c2 = two_nu == 5 ? T(1.0 / 3.0) : (two_nu == 7 ? T(0.4) : T(0));
  const T c3 = two_nu == 7 ? T(1.0 / 15.0) : T(0);
  return fma(r, fma(r, fma(r, c3, c2), c1), T(1)) * t_exp(-r);
}

constexpr double kLog2Pi = 1.83787706640934548356065947281123527;

// 1/sqrt(p): hardware reciprocal square root refined by Newton steps
// r <- r (3 - p r^2) / 2 (two for FP64, one for FP32).
__device__ __forceinline__ double rsqrt_nr(double p) {
  double r = __builtin_amdgcn_rsq(p);
  r = r * (1.5 - 0.5 * p * r * r);
  r = r * (1.5 - 0.5 * p * r * r);
  return r;
}
__device__ __forceinline__ float rsqrt_nr(float p) {
  // (1 - p r^2 with the rounding error of p r added back)
  const float r = __builtin_amdgcn_rsqf(p), h = p * r, l = fmaf(p, r, -h);
  return fmaf(0.5f * r, fmaf(-l, r, fmaf(-h, r, 1.0f)), r);
}

// Lane 0 of every 16-lane row broadcast to its row (DPP row_newbcast, checked on the
// device; FP64 as one 64-bit move).
__device__ __forceinline__ double row_first(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, 0x150, 0xf, 0xf, true);
}
__device__ __forceinline__ float row_first(float v) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x150, 0xf, 0xf, true));
}

// Sum of the four rows' values at the same position within the row, left in
// every row: rows (0 1 2 3) -> permlane16_swap pairs (0,1) and (2,3), then
// permlane32_swap pairs the two halves.
__device__ __forceinline__ double rows_sum(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  const double s1 = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
                    __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
  const unsigned long long w = (unsigned long long)__double_as_longlong(s1);
  const auto lo2 = __builtin_amdgcn_permlane32_swap((unsigned)w, (unsigned)w, false, false);
  const auto hi2 = __builtin_amdgcn_permlane32_swap((unsigned)(w >> 32), (unsigned)(w >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)hi2[0] << 32) | lo2[0])) +
         __longlong_as_double((long long)(((unsigned long long)hi2[1] << 32) | lo2[1]));
}
__device__ __forceinline__ float rows_sum(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float s1 = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const unsigned w = __float_as_uint(s1);
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Elements of a 16-byte vector.
template <typename T>
constexpr int kOV = 16 / (int)sizeof(T);

// 2^(i/32), correctly rounded.
static __device__ const double kExp2Table[32] = {
    0x1.0000000000000p+0, 0x1.059b0d3158574p+0, 0x1.0b5586cf9890fp+0, 0x1.11301d0125b51p+0,
    0x1.172b83c7d517bp+0, 0x1.1d4873168b9aap+0, 0x1.2387a6e756238p+0, 0x1.29e9df51fdee1p+0,
    0x1.306fe0a31b715p+0, 0x1.371a7373aa9cbp+0, 0x1.3dea64c123422p+0, 0x1.44e086061892dp+0,
    0x1.4bfdad5362a27p+0, 0x1.5342b569d4f82p+0, 0x1.5ab07dd485429p+0, 0x1.6247eb03a5585p+0,
    0x1.6a09e667f3bcdp+0, 0x1.71f75e8ec5f74p+0, 0x1.7a11473eb0187p+0, 0x1.82589994cce13p+0,
    0x1.8ace5422aa0dbp+0, 0x1.93737b0cdc5e5p+0, 0x1.9c49182a3f090p+0, 0x1.a5503b23e255dp+0,
    0x1.ae89f995ad3adp+0, 0x1.b7f76f2fb5e47p+0, 0x1.c199bdd85529cp+0, 0x1.cb720dcef9069p+0,
    0x1.d5818dcfba487p+0, 0x1.dfc97337b9b5fp+0, 0x1.ea4afa2a490dap+0, 0x1.f50765b6e4540p+0};

// exp of the covariance generation, e^{-r} for 0 <= r <= end; e^{-end} is 0, and the
// callers clamp r there: the polynomials and squared differences that it multiplies
// grow without limit, so that a smallest value other than 0 would not do (v_ldexp
// instead of an addition to the exponent field: n = 1e6, m = 200 9.97 -> 10.07 ms,
// the other paths within 1 %; a select on r > 708 cost the gradient paths 1-3 %).
// Cody and Waite's reduction in both precisions.  FP64: k = rint(-32 r / ln 2)
// from the low bits of a sum with 1.5 2^52, f = -r - k ln(2)/32 with ln(2)/32
// split into a 34-bit leading part and the rest (|f| <= ln(2)/64), then e^f by its
// Taylor series to degree 6 (truncation 4e-18) times 2^((k mod 32)/32) from a table
// in LDS and 2^(k div 32) by v_ldexp, which underflows as the exact value does.
// Within one ulp (mean 0.31) of normal results; the 32 entries lie on 32 different
// bank pairs.
// FP32: k = rint(-r / ln 2) the same way, v_exp_f32 of the rest (1/ln 2 in two
// parts) and 2^k by v_ldexp; within the ulp of v_exp_f32 for normal results (r < 87).
template <typename T>
struct ExpTable;
template <>
struct ExpTable<double> {
  static constexpr int n = 32;
  static constexpr double end = 750.0;  // (e^-745.2 rounds to 0)
  __device__ static double entry(int i) { return kExp2Table[i]; }
  // EXACT: within rounding; otherwise without the two highest terms of the series
  // (|f| <= ln 2 / 64: 2^-39)
  template <bool EXACT = true>
  __device__ __forceinline__ static double exp_neg(double r, const double* tab) {
    const double kd = fma(r, -0x1.71547652b82fep+5, 0x1.8p+52);
    const int k = __double2loint(kd);
    const double kf = kd - 0x1.8p+52;
    double f = fma(-kf, 0x1.62e42fef80000p-6, -r);
    f = fma(-kf, 0x1.1cf79abc9e3b4p-41, f);
    const double t = tab[k & 31];
    double q = 0x1.5555555555555p-5;
    if (EXACT) q = fma(fma(f, 0x1.6c16c16c16c17p-10, 0x1.1111111111111p-7), f, q);
    q = fma(q, f, 0x1.5555555555555p-3);
    q = fma(q, f, 0.5);
    const double p = fma(f * f, q, f);
    const double s = __builtin_amdgcn_ldexp(t, k >> 5);
    return fma(s, p, s);
  }
};
template <>
struct ExpTable<float> {
  static constexpr int n = 1;
  static constexpr float end = 105.0f;  // (e^-104 rounds to 0)
  __device__ static float entry(int) { return 0.f; }
  __device__ __forceinline__ static float exp_neg(float r, const float*) {
    const float kd = fmaf(r, -0x1.715476p+0f, 0x1.8p+23f);
    const float kf = kd - 0x1.8p+23f;
    float f = fmaf(r, -0x1.715476p+0f, -kf);
    f = fmaf(r, -0x1.4ae0c0p-26f, f);
    return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), __float_as_int(kd) - __float_as_int(0x1.8p+23f));
  }
};

// Distance from its square: the hardware reciprocal square root y (2^-23), g =
// x y, e = 1 - g y, and sqrt(x) = g (1 + e/2 + 3 e^2/8): cubic, truncation below
// 2^-66, within one rounding of g.  Sums of squares start at 2^-1000 instead of 0
// (no covariance can tell), so that coinciding points need no test.  FP32 takes
// the one-instruction hardware square root (1 ulp).
template <bool EXACT = true>
__device__ __forceinline__ double c_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double e = fma(-g, y, 1.0);
  return fma(g * e, EXACT ? fma(e, 0.375, 0.5) : 0.5, g);  // (without: 2^-44)
}
__device__ __forceinline__ float c_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
template <typename T>
constexpr T kTinyR2 = sizeof(T) == 8 ? T(0x1p-1000) : T(0);

// Pointers of a set descriptor point to device memory (kept as such, their loads
// need not go through the flat path).
template <typename E>
__device__ __forceinline__ const __attribute__((address_space(1))) E* as_global(const E* p) {
  return (const __attribute__((address_space(1))) E*)p;
}

}  // namespace sbv
