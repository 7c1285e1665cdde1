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
// r^2 q(r) by Horner's rule, q interpolating (e^r - 1 - r) / r^2 at the
// eleven Chebyshev nodes of that interval (computed in 60 digits; 3e-19
// relative where the Taylor polynomial, one step longer, has 7e-18; with ten
// nodes, 1.6e-17, the error against 64 bits was larger than that one's),
// scaled by 2^k.  Arguments below -1000 are raised to -1000 (the result is 0
// either way); NaN passes through.
constexpr double kExp12[13] = {
    1.0, 1.0, 0.5,
    0.1666666666666667, 0.04166666666666667, 0.008333333333326141,
    0.0013888888888883752, 0.00019841269874800512, 2.4801587325533377e-05,
    2.7557255425720897e-06, 2.75572736613304e-07, 2.510520638458724e-08,
    2.091467938417506e-09};
HGKS_FN double exp_cw(double x) {
  x = x < -1000.0 ? -1000.0 : x;
  const double k = rint(x * kconst<double>(1.4426950408889634));  // 1/ln2
  double r = fma(-k, 0.693146705627441406250, x);                 // ln2 hi
  r = fma(-k, kconst<double>(4.7493250390316727e-07), r);          // ln2 lo
  double p = kconst<double>(kExp12[12]);
#pragma unroll
  for (int n = 11; n >= 0; --n) p = fma(p, r, kconst<double>(kExp12[n]));
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

// P(t) = (1 + 2 y) exp(y^2) erfc(y) for y >= 1 as a polynomial in t = (y -
// 5/2) / (y + 5/2) (the form of Shepherd and Laframboise, Math. Comp. 36
// (1981) 249; the coefficients here interpolate it at the Chebyshev nodes of
// the interval of t, computed in 60 digits).  Double: 1 <= y <= 30, relative
// error 4e-19 before the coefficients are rounded, the first one in two
// parts; float: 1 <= y <= 10.5, 5e-11.
constexpr double kErfcx21[22] = {
    1.2648381843668615, -0.1223567630824043, -0.09902453957360235,
    0.15762991902321885, -0.10296705603851898, 0.032760893268653696,
    0.000931892815307037, -0.004382078339872744, 0.0004918658536842841,
    0.0006321243168957018, -8.847971929518672e-05, -0.00011352181855272056,
    6.26936202312381e-06, 2.2693527327655664e-05, 2.5971676254965236e-06,
    -4.181932452772929e-06, -1.58008076814213e-06, 4.254768999387085e-07,
    6.243366585283449e-07, 1.0943714025627054e-07, -3.172387991637216e-07,
    8.596810916622534e-08};
constexpr double kErfcx21Low = 2.187269270200059e-17;
constexpr double kErfcx10[11] = {
    1.2648381844224124, -0.12235676258686475, -0.09902455259899415,
    0.15762988884746656, -0.1029665512994253, 0.032761221394023654,
    0.0009248454795583878, -0.004380325802225843, 0.0005328702366322006,
    0.0005971990384327377, -0.00017215213115138133};

template <typename T> HGKS_FN T d_rcp(T x);
template <> HGKS_FN double d_rcp<double>(double x);

// (P(t) - P(0)) / t, and with the first coefficient P(t).
template <int N>
HGKS_FN double erfcx_poly(double t, const double (&c)[N]) {
  double p = kconst<double>(c[N - 1]);
#pragma unroll
  for (int n = N - 2; n >= 1; --n) p = fma(p, t, kconst<double>(c[n]));
  return p;
}

// erfc(y) for y >= 1, given e = exp(-z) for a z within some ulp of y^2.
// Beyond y = 30 the result is 0 (e is).
//
// As exact as the C library's erfc (rms 0.62 units of 2^-53 and at most 2.4
// on samples where that has 0.79 and 3.2): the rounding of z is worth z
// units of e, so e is corrected by e^(z - y^2) = 1 - (y^2 - z), and the sums
// and the quotient P / (1 + 2 y) carry their remainders to the last product.
// e P / (1 + 2 y) as it stands is off by up to 12 units at y = 3, 36 at 5.
HGKS_FN double erfc_tail(double y0, double e, double z) {
  const double y = y0 > 30.0 ? 30.0 : y0;
  const double a = y + 2.5, b = 2.0 * y + 1.0;
  const double r = d_rcp(a * b);
  const double t = (y - 2.5) * (b * r);
  const double q = erfcx_poly(t, kErfcx21);
  const double c0 = kconst<double>(kErfcx21[0]);
  const double p = fma(q, t, c0);
  const double pl = fma(q, t, c0 - p) + kErfcx21Low;
  const double bl = 1.0 - (b - 2.0 * y);
  const double rb = a * r;
  const double s = p * rb;                                // P / (1 + 2 y)
  const double sl = (fma(-s, b, p) + (pl - s * bl)) * rb;  // and its remainder
  const double v = fma(e, s, e * (sl - fma(y, y, -z) * s));
  return y0 >= 30.0 ? 0.0 : v;
}

// In float the tail is formed in double from the argument alone (its own
// exponential), and rounded once.
HGKS_FN float erfc_tail(float y0) {
  const double y = y0 > 10.5f ? 10.5 : (double)y0;
  const double a = y + 2.5, b = 2.0 * y + 1.0;
  const double r = d_rcp(a * b);
  const double t = (y - 2.5) * (b * r);
  return (float)(exp_cw(-(y * y)) * (fma(erfcx_poly(t, kErfcx10), t, kconst<double>(kErfcx10[0])) * (a * r)));
}

// erfc(x) given e = exp(-z), z = x^2 but for rounding: 1 - erf by the
// polynomial where |x| <= 1 (every smooth-flow interface state has
// |sqrt(lambda) U| well below 1), the tail form elsewhere.  The library erfc
// it replaces forms its own exponential and kept some 160 instructions and
// their registers in each side's code.
template <typename T> HGKS_FN T d_erfc(T x, T e, T z);
template <> HGKS_FN double d_erfc<double>(double x, double e, double z) {
  if (fabs(x) <= 1.0) return 1.0 - erf_small(x, kErf12);
  const double t = erfc_tail(fabs(x), e, z);
  return x > 0.0 ? t : 2.0 - t;
}
template <> HGKS_FN float d_erfc<float>(float x, float, float) {
  if (fabsf(x) <= 1.0f) return 1.0f - erf_small(x, kErf6);
  const float t = erfc_tail(fabsf(x));
  return x > 0.0f ? t : 2.0f - t;
}
// e = exp(-x^2), x^2 as it rounds.
template <typename T> HGKS_FN T d_erfc(T x, T e) { return d_erfc<T>(x, e, x * x); }
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
