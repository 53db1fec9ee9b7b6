// Exact dot products of fp16 rows on the integer matrix cores.
//
// The prompt phase needs q . k to fp64 precision (the scores decide which tokens are kept), and the
// fp64 matrix instruction is the slowest way to it on this chip: 64 cycles per 16 x 16 x 4 block,
// 32 times the time per multiply of v_mfma_i32_16x16x64_i8, and no vector instruction runs beside it.
// A half is a multiple of 2^-24, so below kDigitMax a value times 2^24 is an integer of 31 bits
// and sign, written here as four signed base-256 digits (each in [-128, 127]):
//     x 2^24 = d0 + 256 d1 + 256^2 d2 + 256^3 d3,      |d3| <= 127.
// A dot product is then sixteen dot products of digit planes, whose 32-bit integer sums are exact;
// planes with the same weight share an accumulator (seven groups, group s = sum of di dj, i + j = s).
// With D <= 128 the largest sums are
//     |g6| <= 128 * 127^2, |g5| <= 128 * 2 * 127 * 128, |g4| <= 128 (2 * 127 * 128 + 128^2),
//     |g3| <= 128 (2 * 127 * 128 + 2 * 128^2), |g2| <= 128 * 3 * 128^2,
// so that 256 g6 + g5, 256 g3 + g2 and 256 g1 + g0 fit 32 bits (the tightest: 2145386496): four
// integers per product, each exact in fp64, joined by four fused multiply-adds that also apply the
// scale and the shift of the exponent.  Four roundings in all, against D / 4 and more in the
// fp64 matrix sum.
//
// Layout of v_mfma_i32_16x16x64_i8 (wave64, lane = 16 g + c): A row / B column c takes the 16
// consecutive k = 16 g .. 16 g + 15 of a 64-wide block from lane (g, c); result register w of lane
// (g, c) is element [4 g + w][c].
#pragma once

#include "lessdec_common.h"

namespace lessdec {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

// Values of this magnitude and above (infinities and NaN among them) have no digits: the tile that
// holds one is multiplied in fp64 (dot_tiles_f64).  127.0 as a half.
constexpr unsigned kDigitMax = 0x57F0;

// Joined sums of one lane's four elements of a tile.
struct DotParts {
  v4i p65, p4, p32, p10;
};
// weight of the least digit pair in a dot product
constexpr double kDotUnit = 0x1p-48;

// Digits of 4 halves (two dwords): plane p's dword holds digit p of the four.
__device__ inline void digits_of4(unsigned h01, unsigned h23, unsigned (&plane)[4], float unit = 0x1p24f)
{
  auto digit_word = [unit](unsigned short h) {
    const float f = fmaf((float)__builtin_bit_cast(_Float16, h), unit, 0.f);   // exact
    // adding 128 to every digit makes the digits the bytes of the sum; the sign bits flip back below
    return (unsigned)(int)f + 0x80808080u;
  };
  const unsigned u0 = digit_word((unsigned short)h01), u1 = digit_word((unsigned short)(h01 >> 16));
  const unsigned u2 = digit_word((unsigned short)h23), u3 = digit_word((unsigned short)(h23 >> 16));
  const unsigned a = __builtin_amdgcn_perm(u1, u0, 0x05010400u), b = __builtin_amdgcn_perm(u1, u0, 0x07030602u);
  const unsigned c = __builtin_amdgcn_perm(u3, u2, 0x05010400u), d = __builtin_amdgcn_perm(u3, u2, 0x07030602u);
  plane[0] = __builtin_amdgcn_perm(c, a, 0x05040100u) ^ 0x80808080u;
  plane[1] = __builtin_amdgcn_perm(c, a, 0x07060302u) ^ 0x80808080u;
  plane[2] = __builtin_amdgcn_perm(d, b, 0x05040100u) ^ 0x80808080u;
  plane[3] = __builtin_amdgcn_perm(d, b, 0x07060302u) ^ 0x80808080u;
}

// Whether any of the N dwords holds a half without digits.
template <int N>
__device__ inline bool without_digits(const unsigned (&w)[N])
{
  typedef unsigned short us2 __attribute__((ext_vector_type(2)));
  us2 m = {0, 0};
#pragma unroll
  for (int i = 0; i < N; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(us2, w[i] & 0x7fff7fffu));
  return m.x >= kDigitMax || m.y >= kDigitMax;
}

// A row of D halves in operand order: the lane's 16 elements of every 64-wide block, all planes.
template <int D>
struct RowDigits {
  static constexpr int KC = D / 64;
  v4i d[KC][4];
  // returns whether the lane's elements all have digits
  __device__ inline bool load(const __half *row, int g)
  {
    bool bad = false;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      const uint4 x = reinterpret_cast<const uint4 *>(row + 64 * kc + 16 * g)[0];
      const uint4 y = reinterpret_cast<const uint4 *>(row + 64 * kc + 16 * g)[1];
      const unsigned w[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
      bad |= without_digits(w);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        unsigned p[4];
        digits_of4(w[2 * i], w[2 * i + 1], p);
#pragma unroll
        for (int q = 0; q < 4; ++q) d[kc][q][i] = (int)p[q];
      }
    }
    return !bad;
  }
};

// Digits of rows scaled by a power of two, so that the largest value uses the top digit in full.  A half has 11 significant
// bits, so the lowest of four digits is then zero but for values 2^-12 of the largest and below: few blocks of 16 rows x 64
// elements hold one (about a third with normal values), and without it a dot product takes nine products
// of planes instead of sixteen.  A lane's 16 elements of a 64-wide block are 64 kc + 8 g .. + 7 and 32 further:
// the order within a dot product is free as long as both sides keep to it.
template <int D>
struct ScaledDigits {
  static constexpr int KC = D / 64;
  v4i d[KC][4];
  int scale;                                              // the digits are those of the values times 2^scale, 0 .. 20
  // row: the lane's; every lane of the wave must call.  ALL: one scale for all 16 rows, else one per row.  Returns
  // whether the lane's elements all have digits.
  template <bool ALL>
  __device__ inline bool load(const __half *row, int g)
  {
    unsigned w[KC][8], top = 0;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint4 x = *reinterpret_cast<const uint4 *>(row + 64 * kc + 8 * g + 32 * i);
        w[kc][4 * i] = x.x; w[kc][4 * i + 1] = x.y; w[kc][4 * i + 2] = x.z; w[kc][4 * i + 3] = x.w;
      }
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    us2 m = {0, 0};
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int i = 0; i < 8; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(us2, w[kc][i] & 0x7fff7fffu));
    top = m.x > m.y ? m.x : m.y;
    const bool ok = top < kDigitMax;
    unsigned all = ok ? top : 0;
#pragma unroll
    for (int o = ALL ? 1 : 16; o < 64; o *= 2) {
      const unsigned t = (unsigned)__shfl_xor((int)all, o);
      all = t > all ? t : all;
    }
    // 2^e (1 + f) 2^(6 - e) < 128; below 127 unless f >= 63 / 64
    const int e = (all >> 10 ? (int)(all >> 10) : 1) - 15;
    scale = 6 - e - ((all & 0x3ffu) >= 0x3f0u ? 1 : 0);
    scale = scale > 0 ? scale : 0;
    const float unit = __builtin_ldexpf(1.f, 24 + scale);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        unsigned p[4];
        digits_of4(w[kc][2 * i], w[kc][2 * i + 1], p, unit);
#pragma unroll
        for (int q = 0; q < 4; ++q) d[kc][q][i] = (int)p[q];
      }
    return ok;
  }
  // bit kc: some lane has a lowest digit in that block
  __device__ inline unsigned lowest() const
  {
    unsigned r = 0;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) r |= __any((d[kc][0][0] | d[kc][0][1] | d[kc][0][2] | d[kc][0][3]) != 0) ? 1u << kc : 0u;
    return r;
  }
};

// One 64-wide block and one digit plane `pa` of the A operand against all planes of B.
__device__ inline void dot_planes(const v4i a, const v4i (&b)[4], int pa, v4i (&s)[7])
{
#pragma unroll
  for (int pb = 0; pb < 4; ++pb) s[pa + pb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b[pb], s[pa + pb], 0, 0, 0);
}
__device__ inline DotParts dot_join(const v4i (&s)[7])
{
  DotParts r;
  r.p65 = (s[6] << 8) + s[5];
  r.p4 = s[4];
  r.p32 = (s[3] << 8) + s[2];
  r.p10 = (s[1] << 8) + s[0];
  return r;
}
// c (dot product of element w) + shift, c folded into the four weights
__device__ inline double dot_affine(const DotParts &p, int w, double c, double shift)
{
  return fma((double)p.p65[w], c * (kDotUnit * 0x1p40),
             fma((double)p.p4[w], c * (kDotUnit * 0x1p32),
                 fma((double)p.p32[w], c * (kDotUnit * 0x1p16), fma((double)p.p10[w], c * kDotUnit, shift))));
}

// half e of a 16-byte piece
__device__ inline double half_of(const uint4 &x, int e)
{
  const unsigned w = e < 2 ? x.x : e < 4 ? x.y : e < 6 ? x.z : x.w;
  const __half2 h = __builtin_bit_cast(__half2, w);
  return (double)(e % 2 ? __high2float(h) : __low2float(h));
}

// The same in fp64, for operands that have no digits: N tiles of 16 keys against 16 queries, element w of lane (g, c)
// of tile t is key[16 t + 4 g + w] . query[c].  krow(i): row of key i (any readable row), qrow: the lane's query.
// Lane group g supplies the D / 4 elements from g D / 4 on of its row, read as 16-byte pieces, all ahead of the products;
// a query element is widened once for the N tiles.
template <int D, int N, typename KRow>
__device__ inline void dot_tiles_f64(KRow krow, const __half *qrow, int g, int c, v4d (&acc)[N])
{
  constexpr int NV = D / 32;                              // pieces of 8 halves
  uint4 k[N][NV], q[NV];
  // result register v of v_mfma_f64_16x16x4 holds row g + 4 v, so matrix row i stands for key 4 (i % 4) + i / 4
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const uint4 *kr = reinterpret_cast<const uint4 *>(krow(16 * t + 4 * (c % 4) + c / 4) + g * (D / 4));
#pragma unroll
    for (int i = 0; i < NV; ++i) k[t][i] = kr[i];
    acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) q[i] = reinterpret_cast<const uint4 *>(qrow + g * (D / 4))[i];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double qe = half_of(q[i], e);
#pragma unroll
      for (int t = 0; t < N; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(half_of(k[t][i], e), qe, acc[t], 0, 0, 0);
    }
}
// One tile, a piece of 8 halves at a time: for kernels without the registers to hold all pieces.
template <int D, typename KRow>
__device__ inline v4d dot_tile_f64(KRow krow, const __half *qrow, int g, int c)
{
  const __half *kr = krow(4 * (c % 4) + c / 4) + g * (D / 4), *qr = qrow + g * (D / 4);
  v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int i = 0; i < D / 32; ++i) {
    const uint4 k = reinterpret_cast<const uint4 *>(kr)[i], q = reinterpret_cast<const uint4 *>(qr)[i];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(half_of(k, e), half_of(q, e), acc, 0, 0, 0);
  }
  return acc;
}

// 2^y of N values in fp64, y <= a few: y = n + f with |f| <= 1/2, polynomial of degree 9 in f
// (interpolated at Chebyshev points, fit_exp2_poly.py, 1.9e-14 relative), scaled by 2^n; 0 where that underflows.
// Scores come in base-2 units, so no reduction by ln 2 is needed.  The N chains run side by
// side: one alone would wait for every multiply-add.
template <int N>
__device__ inline void exp2_f64(const double (&y)[N], double (&e)[N])
{
  constexpr double kPoly[9] = {1.325964524488711e-06, 1.5252672924850737e-05, 0.0001540343375125101,
                               0.0013333558200794592, 0.009618129193934313,   0.05550410866465167,
                               0.2402265069564034,    0.6931471805599462,     1.0000000000000135};
  double f[N], p[N];
  int n[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double r = __builtin_rint(y[i]);
    f[i] = y[i] - r;
    n[i] = (int)r;
    p[i] = 1.0205905413765595e-07;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k)
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], f[i], kPoly[k]);
#pragma unroll
  for (int i = 0; i < N; ++i) e[i] = __builtin_ldexp(p[i], n[i]);
}

constexpr double kLog2E = 1.4426950408889634074;
constexpr double kLn2 = 0.69314718055994530942;

}  // namespace lessdec
