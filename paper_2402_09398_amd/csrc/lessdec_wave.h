// Wave-level helpers shared by the decode-step kernels (gfx950, wave64): DPP reductions,
// non-temporal 16-byte loads, and the encoding of the work a step leaves pending.
#pragma once

#include "lessdec_common.h"
#include "lessdec_internal.h"

namespace lessdec {

typedef unsigned int u4v __attribute__((ext_vector_type(4)));

// Polls of the feature-map entries, with s_sleep(sleep) of 64 x sleep cycles ahead of each, before a wave gives up: the sleeps alone add
// up to 2^25 cycles (16 ms at 2.1 GHz), however short one of them is; the ways to memory come on top.
constexpr int poll_limit(int sleep) { return (1 << 19) / sleep; }

// ---- cross-lane helpers (DPP within 16-lane rows, readlane across rows) -------------------
template <int CTRL>
__device__ inline int dpp_mov(int x)
{
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ inline double dpp_mov(double x)
{
  return __hiloint2double(dpp_mov<CTRL>(__double2hiint(x)), dpp_mov<CTRL>(__double2loint(x)));
}
// All-reduce over the 16 lanes of a DPP row: quad_perm [1,0,3,2], quad_perm [2,3,0,1],
// row_ror 4, row_ror 8.  Every lane ends with the row's result.
template <typename V, typename Op>
__device__ inline V row16_allreduce(V v, Op op)
{
  v = op(v, dpp_mov<0xB1>(v));
  v = op(v, dpp_mov<0x4E>(v));
  v = op(v, dpp_mov<0x124>(v));
  v = op(v, dpp_mov<0x128>(v));
  return v;
}
__device__ inline int readlane_v(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ inline double readlane_v(double x, int l)
{
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                          __builtin_amdgcn_readlane(__double2loint(x), l));
}
// All-reduce over the wave, combined in the fixed order ((row0, row1), row2), row3.
template <typename V, typename Op>
__device__ inline V wave_allreduce(V v, Op op)
{
  v = row16_allreduce(v, op);
  return op(op(op(readlane_v(v, 0), readlane_v(v, 16)), readlane_v(v, 32)), readlane_v(v, 48));
}
struct OpAdd { __device__ double operator()(double a, double b) const { return a + b; } };
struct OpMax { __device__ double operator()(double a, double b) const { return fmax(a, b); } };
struct OpMin { __device__ double operator()(double a, double b) const { return fmin(a, b); } };
struct OpMinI { __device__ int operator()(int a, int b) const { return a < b ? a : b; } };

// x of the lane 16 further in a pair of 16-lane rows, added: after a row's all-reduce every lane of the pair has the pair's sum.
// (v_permlane16_swap: the odd rows of the first operand and the even rows of the second change places)
__device__ inline double add_other_row16(double x)
{
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  const v2u lo = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(x), false, false));
  const v2u hi = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(x), false, false));
  return __hiloint2double((int)hi.x, (int)lo.x) + __hiloint2double((int)hi.y, (int)lo.y);
}
// Sum over the LPR lanes that hold a cache row, in every one of them, without a trip through the LDS (a shuffle waits for
// one at every step; a row's 32 lanes took five).
template <int LPR>
__device__ inline double row_sum(double v)
{
  static_assert(LPR == 8 || LPR == 16 || LPR == 32, "a row spans 8, 16 or 32 lanes");
  if constexpr (LPR == 8) {
    v += dpp_mov<0xB1>(v);
    v += dpp_mov<0x4E>(v);
    return v + dpp_mov<0x141>(v);                          // row_half_mirror: the other quad of eight lanes
  } else {
    v = row16_allreduce(v, OpAdd{});
    return LPR == 32 ? add_other_row16(v) : v;
  }
}
// Sums of four values over the LPR lanes of a row: lane lr % 4 == h of the row gets that of v[h].  The first two stages halve
// what is carried on: 27 vector instructions where four row_sum take 48; the same sums in the same order.
template <int LPR>
__device__ inline double row_sum4(const double (&v)[4], int lane)
{
  static_assert(LPR == 8 || LPR == 16, "");
  const bool b0 = lane & 1, b1 = lane & 2;
  const double s01 = (b0 ? v[1] : v[0]) + dpp_mov<0xB1>(b0 ? v[0] : v[1]);
  const double s23 = (b0 ? v[3] : v[2]) + dpp_mov<0xB1>(b0 ? v[2] : v[3]);
  double s = (b1 ? s23 : s01) + dpp_mov<0x4E>(b1 ? s01 : s23);
  if constexpr (LPR == 16) {
    s += dpp_mov<0x124>(s);
    return s + dpp_mov<0x128>(s);
  } else {
    return s + dpp_mov<0x141>(dpp_mov<0x1B>(s));           // the lane four away: quad reversed, then row_half_mirror
  }
}
// Sums of two values over the LPR lanes of a row: even lanes get a's, odd ones b's.  The first stage halves what is carried on;
// the same sums in the same order as row_sum.
template <int LPR>
__device__ inline double row_sum2(double a, double b, int lane)
{
  static_assert(LPR == 8 || LPR == 16, "");
  const bool odd = lane & 1;
  double s = (odd ? b : a) + dpp_mov<0xB1>(odd ? a : b);
  s += dpp_mov<0x4E>(s);
  if constexpr (LPR == 16) {
    s += dpp_mov<0x124>(s);
    return s + dpp_mov<0x128>(s);
  } else {
    return s + dpp_mov<0x141>(dpp_mov<0x1B>(s));           // the lane four away: quad reversed, then row_half_mirror
  }
}

// x of the lane X away added, X = 8, 16 or 32: DPP or a lane swap, without a trip through the LDS.
template <int X>
__device__ inline float add_xor(float x)
{
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  static_assert(X == 8 || X == 16 || X == 32, "");
  const unsigned u = __float_as_uint(x);
  if constexpr (X == 8) {
    return x + __uint_as_float((unsigned)dpp_mov<0x128>((int)u));       // row_ror 8
  } else {
    const v2u p = X == 16 ? __builtin_bit_cast(v2u, __builtin_amdgcn_permlane16_swap(u, u, false, false))
                          : __builtin_bit_cast(v2u, __builtin_amdgcn_permlane32_swap(u, u, false, false));
    return __uint_as_float(p.x) + __uint_as_float(p.y);
  }
}
// Half of a reduce-scatter: lanes whose bit X is clear get the pair's sum of `lo`, the others that of `hi`.
template <int X>
__device__ inline float scatter_add(float lo, float hi, int lane)
{
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  static_assert(X == 8 || X == 16, "");
  if constexpr (X == 8) {
    const float send = lane & X ? lo : hi, keep = lane & X ? hi : lo;
    return keep + __uint_as_float((unsigned)dpp_mov<0x128>((int)__float_as_uint(send)));
  } else {
    const v2u p = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false));
    return __uint_as_float(p.x) + __uint_as_float(p.y);
  }
}
// Combines the 64 / LPR row groups' partial sums of the same eight columns: a lane ends with four of them (the upper four where its bit
// LPR is set), summed over all groups, and with f summed over the groups that differ in more than that bit.
template <int LPR>
__device__ inline void combine_row_groups(float (&o)[8], float (&f)[4], int lane)
{
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = scatter_add<LPR>(o[i], o[i + 4], lane);
  if constexpr (LPR == 8) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[i] = add_xor<16>(o[i]);
      f[i] = add_xor<16>(f[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[i] = add_xor<32>(o[i]);
    f[i] = add_xor<32>(f[i]);
  }
}
// Four heads' partial sums of the same eight columns in the 64 / LPR row groups: lanes 16 h .. 16 h + 15 end with head h's, summed
// over all groups (LPR = 8: every column twice).
template <int LPR>
__device__ inline void combine_four_heads(const float (&o)[4][8], float (&r)[8])
{
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  auto sum32 = [](float a, float b) {
    const v2u p = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false));
    return __uint_as_float(p.x) + __uint_as_float(p.y);
  };
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float even = sum32(o[0][i], o[2][i]), odd = sum32(o[1][i], o[3][i]);
    r[i] = scatter_add<16>(even, odd, 0);
    if constexpr (LPR == 8) r[i] = add_xor<8>(r[i]);
  }
}
// Two heads' partial sums of the same eight columns in the 64 / LPR row groups: a lane ends with four of the columns (the upper
// four where its bit LPR is set) of head lane / 32, summed over all groups.
template <int LPR>
__device__ inline void combine_two_heads(const float (&o)[2][8], float (&r)[4], int lane)
{
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  float t[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const v2u p = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane32_swap(__float_as_uint(o[0][i]), __float_as_uint(o[1][i]), false, false));
    t[i] = __uint_as_float(p.x) + __uint_as_float(p.y);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r[i] = scatter_add<LPR>(t[i], t[i + 4], lane);
    if constexpr (LPR == 8) r[i] = add_xor<16>(r[i]);
  }
}

// Stores of state that go through the L2 to memory as they are issued (system scope).  A line
// that stays dirty in an L2 is written back when the kernel ends, before the next launch can
// start: with 16 MB written per launch that takes 2.4 us after plain stores, 1.3 us after
// non-temporal ones and under 0.1 us after these.
__device__ inline void store_wt(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
__device__ inline void store_wt(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
__device__ inline void store_wt(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
__device__ inline void store_wt8(void *p, const uint2 &v)
{
  unsigned long long t;
  __builtin_memcpy(&t, &v, 8);
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// 16 bytes per lane at base + offset: base must be the same for the whole wave (it goes into a
// buffer descriptor, which is how a 16-byte store gets its scope bits)
__device__ inline void store_wt16(void *base, int offset_bytes, const uint4 &v)
{
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00020000);
  u4v t;
  __builtin_memcpy(&t, &v, 16);
  __builtin_amdgcn_raw_buffer_store_b128(t, rs, offset_bytes, 0, 17 /* sc0 sc1 */);
}
__device__ inline void store_wt16(void *base, int offset_bytes, const float4 &v)
{
  uint4 t;
  __builtin_memcpy(&t, &v, 16);
  store_wt16(base, offset_bytes, t);
}

template <typename T>
__device__ inline typename Store<T>::Vec buffer_load_nt(__amdgpu_buffer_rsrc_t rsrc, int voffset, int soffset)
{
  typename Store<T>::Vec v;
  const u4v t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voffset, soffset, 2 /* nt */);
  __builtin_memcpy(&v.raw, &t, 16);
  return v;
}

// The pending work a step leaves behind (pend_slot): -1 nothing; otherwise the low bits name
// a slot.  Slot s < C: psi[s] is to become the psi of the key that now sits there (kept in
// pend_psi) and, unless kPendNoFold is set, the pair that sat there before (psi still in
// psi[s], value row in pend_v) is to be folded into H, z.  Slot C: the step's own pair was
// discarded; its psi is the pend_psi entry itself.
struct Pending {
  int slot;
  bool fold;
};
// A word that no step wrote (buffers never reset) still decodes to a slot in [-1, C]: every use
// of the slot is then an access inside the unit's own arrays.
__device__ inline Pending decode_pending(int ps, int C)
{
  Pending p;
  const int s = ps & 0xffff;
  p.slot = ps < 0 ? -1 : (s < C ? s : C);
  p.fold = ps >= 0 && !(ps & kPendNoFold);
  return p;
}
// Tokens seen by a unit, as loaded: a step on buffers that were never reset must stay inside the
// unit's arrays whatever the word holds, so a negative count reads as an empty cache (and a huge
// one stays clear of overflow when it is advanced and compared with positions).
__device__ inline int sane_n_seen(int n) { return n < 0 ? 0 : (n > (1 << 30) ? (1 << 30) : n); }

}  // namespace lessdec
