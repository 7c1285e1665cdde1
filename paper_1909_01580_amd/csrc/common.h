// Shared device helpers of the HGKS kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// The per-lane arithmetic (reconstruction, flux) is also instantiated on the
// host by the operation-counting tool, hence host-and-device functions.
#define HGKS_FN __host__ __device__ __forceinline__

namespace hgks {

// A double constant in a scalar register pair.  FP64 vector instructions
// take no 64-bit literal, so a constant whose low word is not zero is
// otherwise rebuilt by two vector moves at every use; from a scalar pair it
// is a plain operand (one scalar operand per instruction: the addend or the
// multiplier of an FMA), built by scalar moves that issue beside the vector
// work.
HGKS_FN double sreg(double c) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r;
  asm volatile("" : "=s"(r) : "0"(c));
  return r;
#else
  return c;
#endif
}
template <typename T> HGKS_FN T kconst(double c) { return T(c); }
template <> HGKS_FN double kconst<double>(double c) { return sreg(c); }

// exp(x) in double: Cody and Waite's reduction x = k ln2 + r, k = rint(x /
// ln2), |r| <= ln2 / 2, with ln2 split as hi + lo (hi has 21 significant
// bits, so k hi is exact for every k that does not overflow), then 1 + r +
// r^2 q(r) by Horner's rule, q interpolating (e^r - 1 - r) / r^2 at the ten
// Chebyshev nodes of that interval (computed in 60 digits; 1.6e-17
// relative, two steps shorter than the Taylor polynomial), scaled by 2^k.
// Arguments below -1000 are raised to -1000 (the result is 0 either way);
// NaN passes through.
constexpr double kExp11[12] = {
    1.0, 1.0, 0.5000000000000001,
    0.16666666666666669, 0.04166666666662416, 0.008333333333330063,
    0.0013888888917199863, 0.00019841269863042963, 2.4801521317484083e-05,
    2.7557268476553695e-06, 2.7620078203806394e-07, 2.5100377619606372e-08};
HGKS_FN double exp_cw(double x) {
  x = x < -1000.0 ? -1000.0 : x;
  const double k = rint(x * kconst<double>(1.4426950408889634));  // 1/ln2
  double r = fma(-k, 0.693146705627441406250, x);                 // ln2 hi
  r = fma(-k, kconst<double>(4.7493250390316727e-07), r);          // ln2 lo
  double p = kconst<double>(kExp11[11]);
#pragma unroll
  for (int n = 10; n >= 0; --n) p = fma(p, r, kconst<double>(kExp11[n]));
  return ldexp(p, (int)k);
}

template <typename T> HGKS_FN T d_exp(T x);
template <> HGKS_FN double d_exp<double>(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return exp_cw(x);
#else
  return exp(x);
#endif
}
template <> HGKS_FN float d_exp<float>(float x) { return expf(x); }
// erf(x) / x for |x| <= 1 as a polynomial in x^2 that interpolates its
// Maclaurin series at the Chebyshev nodes of [0, 1] (computed in 60 digits):
// relative error 1.6e-17 with 13 coefficients (double) and 1.4e-9 with 7
// (float), where the truncated series took 18 and 11.
constexpr double kErf12[13] = {
    1.1283791670955126, -0.3761263890318375, 0.11283791670954879,
    -0.026866170645076792, 0.0052239776248180145, -0.000854832698083379,
    0.0001205533111164271, -1.4925595266831182e-05, 1.6461000484121368e-06,
    -1.6350312701054695e-07, 1.4659775274047436e-08, -1.1372848856791674e-09,
    5.957176147748911e-11};
constexpr double kErf6[7] = {
    1.1283791658483509, -0.37612626666720334, 0.11283594715160218,
    -0.026854212010626412, 0.005189087423433974, -0.000801686428716587,
    7.875875062685488e-05};

template <int N, typename T>
HGKS_FN T erf_small(T x, const double (&c)[N]) {
  const T t = x * x;
  T s = T(c[N - 1]);
#pragma unroll
  for (int n = N - 2; n >= 0; --n) s = s * t + kconst<T>(c[n]);
  return s * x;
}

// (1 + 2 y) exp(y^2) erfc(y) for y >= 1 as a polynomial in t = (y - 5/2) /
// (y + 5/2), which maps y >= 1 to [-3/7, 1] (the form of Shepherd and
// Laframboise, Math. Comp. 36 (1981) 249; the coefficients here interpolate
// it at the Chebyshev nodes of that interval, computed in 60 digits from
// the series and the continued fraction of erfc).  Relative error below
// 8e-17 (double) and 1.2e-8 (float).
constexpr double kErfcx20[21] = {
    1.2648381843668615, -0.12235676308240334, -0.09902453957361883,
    0.15762991902306947, -0.1029670560369499, 0.03276089327449818,
    0.0009318927560479804, -0.004382078407562973, 0.0004918669534855608,
    0.0006321238749692234, -8.849021316160707e-05, -0.00011350557508225432,
    6.314854131183766e-06, 2.2557189087445965e-05, 2.58439735084272e-06,
    -3.736015440011357e-06, -2.0969626664127912e-06, 1.9248433454712853e-07,
    1.6811287081232611e-06, -9.341138827040256e-07, 1.5677373653870477e-07};
constexpr double kErfcx9[10] = {
    1.264838192458751, -0.12235658115265136, -0.09902554193976162,
    0.15762353273444266, -0.10294296676703253, 0.032807473163065384,
    0.00072638705545182, -0.004371426325112118, 0.0010439879858344689,
    3.6121971193970767e-05};

template <typename T> HGKS_FN T d_rcp(T x);

// erfc(y) = e P(t) / (1 + 2 y) for y >= 1, e = exp(-y^2).  Beyond y = 30 e
// is 0 in both precisions.
template <int N, typename T>
HGKS_FN T erfc_tail(T y, T e, const double (&c)[N]) {
  y = y < T(30) ? y : T(30);
  const T a = y + T(2.5), b = T(2) * y + T(1);
  const T r = d_rcp(a * b);
  const T t = (y - T(2.5)) * (b * r);
  T p = T(c[N - 1]);
#pragma unroll
  for (int n = N - 2; n >= 0; --n) p = p * t + kconst<T>(c[n]);
  return e * p * (a * r);
}

// erfc(x) given e = exp(-x^2): 1 - erf by the polynomial where |x| <= 1 (every
// smooth-flow interface state has |sqrt(lambda) U| well below 1), the tail
// form elsewhere.  The library erfc it replaces forms its own exponential
// and kept some 160 instructions and their registers in each side's code.
template <typename T> HGKS_FN T d_erfc(T x, T e);
template <> HGKS_FN double d_erfc<double>(double x, double e) {
  if (fabs(x) <= 1.0) return 1.0 - erf_small(x, kErf12);
  const double t = erfc_tail(fabs(x), e, kErfcx20);
  return x > 0.0 ? t : 2.0 - t;
}
template <> HGKS_FN float d_erfc<float>(float x, float e) {
  if (fabsf(x) <= 1.0f) return 1.0f - erf_small(x, kErf6);
  const float t = erfc_tail(fabsf(x), e, kErfcx9);
  return x > 0.0f ? t : 2.0f - t;
}
template <typename T> HGKS_FN T d_sqrt(T x);
template <> HGKS_FN double d_sqrt<double>(double x) { return sqrt(x); }
template <> HGKS_FN float d_sqrt<float>(float x) { return sqrtf(x); }
// |x|.  For double and float the sign bit is cleared (an abs modifier on
// the instruction that uses it, or one bitwise and), where the comparison
// form costs a compare, a negation and two selects per double.
template <typename T> HGKS_FN T d_abs(T x) { return x < T(0) ? -x : x; }
template <> HGKS_FN double d_abs<double>(double x) { return __builtin_fabs(x); }
template <> HGKS_FN float d_abs<float>(float x) { return __builtin_fabsf(x); }

// The larger of a and b (one max instruction for double and float; the
// same value as the comparison form unless an argument is not a number).
template <typename T> HGKS_FN T d_max(T a, T b) { return a > b ? a : b; }
template <> HGKS_FN double d_max<double>(double a, double b) { return __builtin_fmax(a, b); }
template <> HGKS_FN float d_max<float>(float a, float b) { return __builtin_fmaxf(a, b); }

// Reciprocal of a nonzero finite x: the hardware estimate refined by
// Newton-Raphson steps r <- r + r (1 - x r) (two in double, one in float),
// at a fraction of the cost of a correctly rounded division.  On gfx950 the
// FP64 estimate is within 2^-24.4 of 1/x; one step leaves up to 11 ulp, two
// steps gave the correctly rounded 1/x on 4 million sampled inputs.
template <> HGKS_FN double d_rcp<double>(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
#else
  return 1.0 / x;
#endif
}
template <> HGKS_FN float d_rcp<float>(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
#else
  return 1.0f / x;
#endif
}

// x plus x of lane l ^ MASK (MASK = 1 or 2) within each group of four
// lanes: a quad-permute DPP move per 32-bit half, which the vector unit
// does in the instruction itself (no LDS-unit round trip as for a general
// lane shuffle).
template <int MASK>
__device__ __forceinline__ float quad_xor_add(float x) {
  constexpr int ctrl = MASK == 1 ? 0xB1 : 0x4E;  // quad_perm [1,0,3,2] / [2,3,0,1]
  return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), ctrl, 0xF, 0xF, false));
}

template <int MASK>
__device__ __forceinline__ double quad_xor_add(double x) {
  constexpr int ctrl = MASK == 1 ? 0xB1 : 0x4E;
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)u, ctrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), ctrl, 0xF, 0xF, false);
  return x + __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Workgroups are dispatched round-robin over the eight XCDs (block b runs
// on XCD b % 8).  Remapping gives every XCD one contiguous range of logical
// blocks, so that neighbouring tiles share an L2.  The grid must hold
// 8 * ceil(nb / 8) blocks; logical ids >= nb do nothing.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned nb_padded) {
  const unsigned per = nb_padded >> 3;
  return (b & 7u) * per + (b >> 3);
}

}  // namespace hgks
