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
// Absolute error in fp32: 2.5e-7 on [-4, 4], one ulp of x beyond.
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

// The same activation for the hidden layers with one transcendental: log2 Q(t) is smooth, a polynomial of degree 8 with
// log2 Q(0) = -1 kept exact takes t Q(t) to 1e-8 (fit_gelu_poly.py; the leading term is negative, so that it goes to
// -infinity beyond), and gelu(x) = max(x, 0) - t 2^poly(t): 11 instructions where the form above takes 16, and closer to erfc
// in fp32 (root mean square error on [-2, 2] 2.9e-8 against 3.1e-8; the largest on [-4, 4], 2.6e-7 and 2.5e-7, is the
// rounding of x there).  The hidden layers of the matrix-core maps use this one; the other remains as the form that the fp64
// one below shares its constants with, and the yardstick of the tests.
__device__ inline float gelu_exp2_f32(float x)
{
  const float t = fabsf(x);
  float p = -2.0174934872e-06f;
  p = fmaf(p, t, 2.9592299348e-05f);
  p = fmaf(p, t, -1.3967072405e-04f);
  p = fmaf(p, t, -2.4949272248e-04f);
  p = fmaf(p, t, 7.2111265152e-03f);
  p = fmaf(p, t, -5.2599315427e-02f);
  p = fmaf(p, t, -4.5917365010e-01f);
  p = fmaf(p, t, -1.1511093201e+00f);
  p = fmaf(p, t, -1.0f);
  const float e = __builtin_amdgcn_exp2f(p);
  // max(x, 0) on the bits (as above)
  const int xi = __builtin_bit_cast(int, x);
  return fmaf(-t, e, __builtin_bit_cast(float, xi > 0 ? xi : 0));
}

// The approximation of gelu_fast_f32 evaluated in fp64 (absolute error 1e-9): for the handful of
// layer-2 activations per row, whose inputs already carry the fp32 rounding of layer 1.
// Much lighter on registers than the library erfc.
__device__ inline double gelu_poly_f64(double x)
{
  const double t = fabs(x), d = fma(0.24, t, 1.0);
  // 1 / d by two Newton steps: d >= 1 needs none of the scaling and fixing of a division
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
  const double tq = t * (a * exp_softmax_f64(-0.5 * t * t));
  return x >= 0.0 ? x - tq : -tq;
}

}  // namespace lessdec
