// Shared device helpers of the lessdec kernels (gfx950, wave64).
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

namespace lessdec {

constexpr int kWave = 64;

// ---- 16-byte vector access to the storage type --------------------------------------
template <typename T> struct Store;
template <> struct Store<float> {
  static constexpr int kPerVec = 4;
  struct Vec { float4 raw; };
  __device__ static inline float get(const Vec &v, int i) { return (&v.raw.x)[i]; }
  __device__ static inline float from_float(float x) { return x; }
  __device__ static inline float to_float(float x) { return x; }
};
template <> struct Store<__half> {
  static constexpr int kPerVec = 8;
  struct Vec { uint4 raw; };
  __device__ static inline float get(const Vec &v, int i)
  {
    const __half *h = reinterpret_cast<const __half *>(&v.raw);
    return __half2float(h[i]);
  }
  __device__ static inline __half from_float(float x) { return __float2half_rn(x); }
  __device__ static inline float to_float(__half x) { return __half2float(x); }
};

template <typename T>
__device__ inline typename Store<T>::Vec load_vec(const T *p)
{
  typename Store<T>::Vec v;
  v.raw = *reinterpret_cast<const decltype(v.raw) *>(p);
  return v;
}

// Eviction candidate: smaller accumulated score first, then the older token.
struct Cand {
  double acc;
  int pos;
  int slot;
};
__device__ inline bool cand_less(const Cand &a, const Cand &b)
{
  return a.acc < b.acc || (a.acc == b.acc && a.pos < b.pos);
}
__device__ inline Cand cand_none() { return Cand{__builtin_inf(), INT_MAX, -1}; }

// e^x in fp64 for the softmax weights of the prompt phase, where x = s - max <= 0 up to
// rounding: x = n ln 2 + r with |r| <= ln 2 / 2, Taylor polynomial of degree 10 in r
// (truncation 2e-13 relative), scaled by 2^n; 0 below the underflow threshold and for -inf.
// Half the instructions of the library routine; its error is far inside the 1e-6 margin by
// which accumulated probabilities may differ before an eviction is called a tie.
__device__ inline double exp_softmax_f64(double x)
{
  const double n = __builtin_rint(x * 1.44269504088896338700e+00);
  double r = fma(n, -6.93147180369123816490e-01, x);
  r = fma(n, -1.90821492927058770002e-10, r);
  double p = 2.75573192239858906526e-07;                   // 1 / 10!
  p = fma(p, r, 2.75573192239858906526e-06);
  p = fma(p, r, 2.48015873015873015873e-05);
  p = fma(p, r, 1.98412698412698412698e-04);
  p = fma(p, r, 1.38888888888888888889e-03);
  p = fma(p, r, 8.33333333333333333333e-03);
  p = fma(p, r, 4.16666666666666666667e-02);
  p = fma(p, r, 1.66666666666666666667e-01);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return x > -708.0 ? __builtin_ldexp(p, (int)n) : 0.0;
}

// e^s for s <= 0 to fp64, as 2^n times the value returned: s = n ln 2 + r with |r| <= ln 2 / 2, 1 + r + r^2/2 + r^3 times a
// polynomial of degree 8 (fit_gelu_f64.py; to 3.3e-17 relatively, with two constants and steps less than the Taylor polynomial).
__device__ inline double exp_parts_f64(double s, double &n)
{
  n = __builtin_rint(s * 1.44269504088896338700e+00);
  double r = fma(n, -6.93147180369123816490e-01, s);
  r = fma(n, -1.90821492927058770002e-10, r);
  double e = 2.50955546771111123e-08;
  e = fma(e, r, 2.76138068615382899e-07);
  e = fma(e, r, 2.75572800670169807e-06);
  e = fma(e, r, 2.48015363886907663e-05);
  e = fma(e, r, 1.98412698543386110e-04);
  e = fma(e, r, 1.38888889058815424e-03);
  e = fma(e, r, 8.33333333333215534e-03);
  e = fma(e, r, 4.16666666666513572e-02);
  e = fma(e, r, 1.66666666666666657e-01);
  e = fma(e, r, 0.5);
  e = fma(e, r, 1.0);
  return fma(e, r, 1.0);
}

// GELU, x * Phi(x) (Sec. 3.2 names GELU as the activation of both feature maps), to fp64: with t = |x| the upper normal tail is
// Q(t) = exp(-t^2/2) F(t), F(t) = 1/2 + c_1 v + ... + c_20 v^20, v = t / (1 + t/5) (constants from fit_gelu_f64.py: F to 2e-17 about
// zero, to 1e-17 t^2 far out), and gelu(x) = max(x, 0) - t Q(t).  Small t have small v, so that next to 1/2 the roundings of v and of the
// sum do not count; in powers of u = 1 - v/5 about a point in the middle such a polynomial loses two bits there.  Measured on gfx950,
// relative root mean square error, and that of 0.5 x erfc(-x / sqrt 2) with the library's erfc: 6.6e-17 and 1.0e-16 on
// [1/10, 1/2], 9.1e-17 and 1.1e-16 on [-1/2, -1/10], 1.5e-16 and 2.8e-16 on [-2, -1], 7.5e-16 and 1.7e-15 on [-5, -4], 3.4e-15 and
// 9.2e-15 on [-12, -9]; in no range larger.  Without branches, and with fewer instructions.
__device__ inline double gelu_f64(double x)
{
  const double t = fabs(x), d = fma(0.2, t, 1.0);
  double u = __builtin_amdgcn_rcp(d);                      // 1 / d by two Newton steps
  u = fma(fma(-d, u, 1.0), u, u);
  u = fma(fma(-d, u, 1.0), u, u);
  const double v = t * u;
  double a = 1.58786077144202701e-17;
  a = fma(a, v, -6.89092555243121660e-16);
  a = fma(a, v, 1.31042258713820988e-14);
  a = fma(a, v, -1.42343597368398350e-13);
  a = fma(a, v, 9.80397908017772762e-13);
  a = fma(a, v, -4.75183761533774438e-12);
  a = fma(a, v, 1.93559579361540074e-11);
  a = fma(a, v, -6.38317779694905220e-11);
  a = fma(a, v, 2.67371916151553225e-11);
  a = fma(a, v, 2.91037901031313963e-10);
  a = fma(a, v, 9.33696418654484656e-09);
  a = fma(a, v, -3.76287761994632628e-08);
  a = fma(a, v, -8.06546275186788731e-07);
  a = fma(a, v, 5.78778320229877026e-06);
  a = fma(a, v, 5.43923726596774734e-05);
  a = fma(a, v, -1.14984213077303334e-03);
  a = fma(a, v, 9.52000568140541799e-03);
  a = fma(a, v, -4.89384513504943219e-02);
  a = fma(a, v, 1.70211543919754654e-01);
  a = fma(a, v, -3.98942280401433647e-01);
  a = fma(a, v, 0.5);
  double n;
  const double e = exp_parts_f64(-0.5 * t * t, n);
  // t takes the power of two: the last multiply-add is then the one rounding behind a e
  const double near = fma(-__builtin_ldexp(t, (int)n), a * e, x >= 0.0 ? x : 0.0);
  // beyond 40 the tail is 0 (the formula's infinities would meet); of -infinity and of what is no number, no number
  return t < 40.0 ? near : x >= 0.0 ? x : x * 0.0;
}

// The fp32 GELU of the matrix-core feature maps' hidden layers, branch-free and with one transcendental: with t = |x| the upper
// normal tail is Q(t) = 2^p(t), log2 Q being smooth enough for a polynomial of degree 10 (fit_gelu_poly.py), and
// gelu(x) = max(x, 0) - t 2^p(t).  p is written about t = 1, where it is small, so that the roundings of Horner's scheme stay below
// those of the other roundings up to t = 4; its leading term is negative, so that p goes to -infinity beyond the fit.
// Measured on gfx950 against erfc, root mean square: 1.6e-9 on [-3, -5/2], 1.1e-8 on [-1, -1/2], 9.2e-9 on [1/4, 1/2]; in every
// range of half a unit from -13/2 to 13 no larger than that of the form e^{-t^2/2} u q(u), u = 1 / (1 + 0.24 t), of
// fit_gelu_poly.py, which takes 16 instructions, two of them transcendental, where this one takes 14 (those errors: 1.6e-9, 2.1e-8,
// 1.9e-8).  Below -13/2, where gelu is above -2.7e-10, to 2e-13.  Degree 8 about t = 0 (11 instructions) errs by 5 to 700 times
// as much as that form below -5/2.
__device__ inline float gelu_exp2_f32(float x)
{
  const float t = fabsf(x), s = t - 1.0f;
  float p = -2.3653170089e-08f;
  p = fmaf(p, s, 4.8210540626e-07f);
  p = fmaf(p, s, -3.9688147808e-06f);
  p = fmaf(p, s, 1.4616596673e-05f);
  p = fmaf(p, s, 1.5595947843e-05f);
  p = fmaf(p, s, -5.8290286688e-04f);
  p = fmaf(p, s, 4.7590648755e-03f);
  p = fmaf(p, s, -2.8118170798e-02f);
  p = fmaf(p, s, -5.7772850990e-01f);
  p = fmaf(p, s, -2.2003047466e+00f);
  p = fmaf(p, s, -2.6560328007e+00f);
  const float e = __builtin_amdgcn_exp2f(p);
  // max(x, 0) on the bits: one instruction, where fmaxf quiets its input in another (a NaN stays one through e)
  const int xi = __builtin_bit_cast(int, x);
  return fmaf(-t, e, __builtin_bit_cast(float, xi > 0 ? xi : 0));
}

// GELU in fp64 with Q(t) = exp(-t^2/2) (c1 u + ... + c7 u^7), u = 1 / (1 + 0.24 t) (absolute error 1e-9; constants from
// fit_gelu_poly.py): for the handful of layer-2 activations per row, whose inputs already carry the fp32 rounding of
// layer 1.  Evaluated to fp64 (within 6e-16 of the same formula with the library's exponential and a division, relatively),
// and much lighter on registers than the library erfc.
__device__ inline double gelu_poly_f64(double x)
{
  const double t = fabs(x), d = fma(0.24, t, 1.0);
  // 1 / d to fp64 by two Newton steps: d >= 1 needs none of the scaling and fixing of a division
  double u = __builtin_amdgcn_rcp(d);
  u = fma(fma(-d, u, 1.0), u, u);
  u = fma(fma(-d, u, 1.0), u, u);
  double a = -1.2459717568e-01;
  a = fma(a, u, 5.5222350684e-01);
  a = fma(a, u, -6.4138824846e-01);
  a = fma(a, u, 6.2064721284e-01);
  a = fma(a, u, -1.5113306584e-01);
  a = fma(a, u, 1.5460257740e-01);
  a = fma(a, u, 8.9645194151e-02);
  a *= u;
  // exp(-t^2/2); 0 below the smallest fp64 number (and where t is infinite, which has no n)
  double n;
  const double s = -0.5 * t * t, e = exp_parts_f64(s, n);
  const double tq = t * (a * (s > -746.0 ? __builtin_ldexp(e, (int)n) : 0.0));
  return x >= 0.0 ? x - tq : -tq;
}

}  // namespace lessdec
