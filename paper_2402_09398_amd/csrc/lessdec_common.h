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
// Q(t) = exp(-t^2/2) u q(u), u = 1 / (1 + 0.2 t), q a polynomial of degree 16 about u = 0.6875 (interpolated in 50 digits,
// fit_gelu_f64.py: t Q(t) to 1.1e-17), and gelu(x) = x - t Q(t) or -t Q(t).  Within a unit in the last place of max(|x|, 1 / 4);
// against 0.5 x erfc(-x / sqrt 2) of the math library root mean square errors of 2.8e-17 and 1.3e-17 on [-1/2, 1/2], 4.7e-17
// and 6.4e-17 up to 2, 3.1e-17 and 1.2e-16 up to 4, in less than half of the instructions and without its branches.
__device__ inline double gelu_f64(double x)
{
  const double t = fabs(x), d = fma(0.2, t, 1.0);
  double u = __builtin_amdgcn_rcp(d);                      // 1 / d by two Newton steps
  u = fma(fma(-d, u, 1.0), u, u);
  u = fma(fma(-d, u, 1.0), u, u);
  const double w = u - 0.6875;
  double a = -3.55819588174844563e-03;
  a = fma(a, w, 3.45149954721361710e-03);
  a = fma(a, w, 7.48983270522050448e-03);
  a = fma(a, w, -9.37836653226709928e-03);
  a = fma(a, w, -1.56020597849275289e-02);
  a = fma(a, w, 1.96166533753664926e-02);
  a = fma(a, w, 4.12068857683245693e-02);
  a = fma(a, w, -2.84153602293953679e-02);
  a = fma(a, w, -1.26634321580951476e-01);
  a = fma(a, w, -5.47639946791622714e-02);
  a = fma(a, w, 2.95093219366276860e-01);
  a = fma(a, w, 7.74383671810909502e-01);
  a = fma(a, w, 1.09561215376561027e+00);
  a = fma(a, w, 1.09088564683540157e+00);
  a = fma(a, w, 8.24213663575876110e-01);
  a = fma(a, w, 4.84700660274498263e-01);
  a = fma(a, w, 2.21746856547500759e-01);
  // exp(-t^2/2) = 2^n e^r, |r| <= ln 2 / 2, Taylor polynomial of degree 12 (2e-16 at the ends)
  const double s = -0.5 * t * t, n = __builtin_rint(s * 1.44269504088896338700e+00);
  double r = fma(n, -6.93147180369123816490e-01, s);
  r = fma(n, -1.90821492927058770002e-10, r);
  double e = 2.08767569878680989792e-09;                   // 1 / 12!
  e = fma(e, r, 2.50521083854417187751e-08);
  e = fma(e, r, 2.75573192239858906526e-07);
  e = fma(e, r, 2.75573192239858906526e-06);
  e = fma(e, r, 2.48015873015873015873e-05);
  e = fma(e, r, 1.98412698412698412698e-04);
  e = fma(e, r, 1.38888888888888888889e-03);
  e = fma(e, r, 8.33333333333333333333e-03);
  e = fma(e, r, 4.16666666666666666667e-02);
  e = fma(e, r, 1.66666666666666666667e-01);
  e = fma(e, r, 0.5);
  e = fma(e, r, 1.0);
  e = fma(e, r, 1.0);
  const double tq = t * (a * u * __builtin_ldexp(e, (int)n));
  // beyond 40 the tail is 0 (the formula's infinities would meet); of -infinity and of what is no number, no number
  const bool near = t < 40.0;
  return x >= 0.0 ? (near ? x - tq : x) : (near ? -tq : x * 0.0);
}

// Branch-free fp32 GELU for the matrix-core feature maps.  With t = |x| the upper normal
// tail is Q(t) = exp(-t^2/2) * (c1 u + ... + c7 u^7), u = 1 / (1 + 0.24 t) (polynomial error
// 1e-9; constants from fit_gelu_poly.py), and gelu(x) = x - t Q(t) for x >= 0, -t Q(t) else.
// Absolute error in fp32: 2.5e-7 on [-4, 4], one ulp of x beyond.  (No kernel uses it.)
__device__ inline float gelu_fast_f32(float x)
{
  const float t = fabsf(x);
  const float u = __builtin_amdgcn_rcpf(fmaf(0.24f, t, 1.0f));
  float a = -1.2459717568e-01f;
  a = fmaf(a, u, 5.5222350684e-01f);
  a = fmaf(a, u, -6.4138824846e-01f);
  a = fmaf(a, u, 6.2064721284e-01f);
  a = fmaf(a, u, -1.5113306584e-01f);
  a = fmaf(a, u, 1.5460257740e-01f);
  a = fmaf(a, u, 8.9645194151e-02f);
  a *= u;
  const float e = __builtin_amdgcn_exp2f(t * t * -0.72134752044448170368f);   // exp(-t^2/2)
  const float tq = t * (a * e);
  // max(x, 0) on the bits: one instruction, where fmaxf quiets its input in another (a NaN stays one through tq)
  const int xi = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, xi > 0 ? xi : 0) - tq;
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
