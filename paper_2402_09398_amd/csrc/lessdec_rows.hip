// Prompt phase, fp16 storage: causal rows (log-sums and attention outputs) and exact column sums,
// with the scores as exact integer products of digit planes (lessdec_digits.h).
#include <type_traits>

#include "lessdec_digits.h"
#include "lessdec_internal.h"
#include "lessdec_prefill.h"

namespace lessdec {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// -------------------------------------------------------------------------------------
// Row pass.  A workgroup of four waves owns 64 consecutive queries, a wave 16 of them; the workgroup
// sweeps the key tiles of 32 up to its last diagonal.  Per tile all threads
// fetch the keys, split them into digit planes and put those into the LDS in operand order, and the
// values transposed, as the A operand of p V.  A wave multiplies each 16-key half with its queries
// (digits in registers): scores S^T[key][query], lane (g, c) holding keys 4 g + w of query c.
// The running maximum m is an integer in base-2 units, the one below the largest score of the first tile (so that
// the largest weight is above 1 and the fp16 pairs' floor of 2^-24 as far below it as with weights up to 1), moved when a
// score passes it by kSlack, which is rare and exact.  The weights are fp64; their sum gives lse, and p V takes
// them as an fp16 pair hi + lo (22 bits) with fp32 accumulation.  Leaves lse_i = ln sum_j e^{s_ij}.
// A tile with a value that has no digits (|x| >= 127), and every tile of a wave whose queries hold one, is multiplied
// in fp64 instead, from rows read as 16-byte pieces: 512 units x 1024 tokens with such a key channel in every token take
// 2907 us in all against 1486 with digits throughout and 3010 with fp64 products throughout (10560 with halves read
// singly, each product waiting for its own).
//
// Per 16 x 16 tile the matrix units need 32 x 16 cycles for the digit products and 8 x 16 for p V, the
// vector units 222 instructions (8192 tokens; 246 at 1024) of 4 to 5 cycles; a tile takes 1570 cycles of a SIMD (1950), issue
// two thirds of them: the rest are dependent fp64 chains, LDS reads and the barrier, which two waves a SIMD do not cover,
// and with short sweeps the wait for a workgroup's longest wave.  The two kinds run side by side (fp64 matrix instructions
// overlap with nothing), but a wave issues in order, so the loop is pipelined by one tile: the
// products of a tile stand in one basic block with the weights and p V of the tile before and the staging
// of the tile after.  One barrier per tile: keys in two buffers, values in
// three (p V of tile kt - 1 runs after the barrier of tile kt).
// 7390 us for 2048 units x 1024 tokens and 23540 for 128 x 8192 with fp64 matrix products; 3530 and 10900 to 11200 now.
// Eight waves to a workgroup split each key half as often, but wait longer for the waves whose diagonal
// comes last: 4560 and 11330.
// -------------------------------------------------------------------------------------
constexpr int kRowKeys = 32;
constexpr double kSlack = 15.0;                           // weights up to 2^15: they fit a half
constexpr double kNoWeight = -5000.0;                     // the weight of this score is 0

// One key tile in the LDS.  Both operands lie as 1 KiB blocks [lane group g][16 rows] of 16 bytes, in
// which a wave's read is one contiguous run; the row's place is turned by the block, so that writes of
// one row to several blocks fall into different banks.
template <int D>
struct RowTile {
  static constexpr int KC = D / 64, DB = D / 16;
  static constexpr int kHalfBytes = 4 * KC * 1024;        // planes of 16 keys
  static constexpr int kPlaneBytes = KC * 1024;
  static constexpr int kKeyBytes = 2 * kHalfBytes, kValBytes = DB * 1024;
  // 16 digits of plane `plane` of key `row` of a half: elements 64 kc + 16 g ..
  static __device__ inline int key_at(int half, int plane, int kc, int g, int row)
  {
    return half * kHalfBytes + plane * kPlaneBytes + (kc * 4 + g) * 256 + (row ^ (2 * (kc * 4 + g))) * 16;
  }
  // value column d = DB i + b as A operand row i of block b; key slot 8 g + 4 half + w stands for key 16 half + 4 g + w
  static __device__ inline int val_at(int b, int i, int g) { return b * 1024 + g * 256 + (i ^ (2 * b % 16)) * 16; }
};

// OUT: attention outputs are wanted too
template <int D, bool OUT>
__global__ __launch_bounds__(64 * kPrefillWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void rows_f16_kernel(
    const __half *__restrict__ Q, const __half *__restrict__ K, const __half *__restrict__ V, unsigned U, int G, int P,
    double *__restrict__ lse, __half *__restrict__ out, unsigned *__restrict__ zero0, unsigned *__restrict__ zero1)
{
  // U counts query rows here: unit u's G query heads are rows u G .. u G + G - 1 of Q, out and
  // lse, and attend over unit u's keys and values
  using Tile = RowTile<D>;
  constexpr int W = kPrefillWaves, KC = D / 64, DB = D / 16, BQ = 16 * W;
  constexpr int EPT = kRowKeys * D / (64 * W);            // consecutive key elements a thread splits: 8 or 16
  constexpr int VK = EPT / 2;                             // value rows a thread takes two columns of
  __shared__ __attribute__((aligned(16))) unsigned char s_key[2][Tile::kKeyBytes], s_val[3][Tile::kValBytes];
  __shared__ int s_bad[3];                                // last tile of this key buffer that lacks digits; [2]: any other
  const int ngrp = (P + BQ - 1) / BQ;
  const PrefillBlock pb = prefill_block(blockIdx.x, ngrp);
  if (pb.u >= U) return;                                  // uniform over the workgroup
  const int grp = ngrp - 1 - pb.grp;                      // long rows first
  const size_t u = pb.u, ukv = u / (unsigned)G;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64, g = l / 16, c = l % 16;
  const __half *Qu = Q + u * (size_t)P * D, *Ku = K + ukv * (size_t)P * D, *Vu = V + ukv * (size_t)P * D;
  const int q0 = grp * BQ + wave * 16;                    // the wave's first query
  const int qi = q0 + c, qrow = qi < P ? qi : P - 1;
  const int kt_last = ((grp * BQ + BQ < P ? grp * BQ + BQ : P) - 1) / kRowKeys;   // the workgroup's last tile
  const int kt_wave = q0 < P ? q0 / kRowKeys : -1;        // the wave's last tile; none
  const double cs = kLog2E / sqrt((double)D);             // q . k to base-2 units

  // this thread's share of a tile: EPT consecutive elements of key row kr, and columns vd, vd + 1 of VK
  // value rows, which lie in one lane group's slots
  const int kr = tid / (D / EPT), ke = tid % (D / EPT) * EPT;
  const int k_dst = Tile::key_at(kr / 16, 0, ke / 64, ke % 64 / 16, kr % 16) + ke % 16;
  const int vd = 2 * (tid % (D / 2)), vs = VK * (tid / (D / 2));               // first of the VK slots
  const int v_dst0 = Tile::val_at(vd % DB, vd / DB, vs / 8) + vs % 8 * 2, v_dst1 = Tile::val_at((vd + 1) % DB, (vd + 1) / DB, vs / 8) + vs % 8 * 2;
  const int k_src = (kr * D + ke) * 2, v_src = ((16 * (vs / 4 % 2) + 4 * (vs / 8) + vs % 4) * D + vd) * 2;
  unsigned kraw[EPT / 2], vraw[VK];
  // Rows past the prompt read as zeros: a buffer load is in range where its vector offset lies below num_records less
  // the scalar offset, so the latter never passes num_records (the row steps of a short last tile would).
  auto fetch = [&](int kt) __attribute__((always_inline)) {
    const int r0 = kt * kRowKeys, bytes = (P - r0 < kRowKeys ? P - r0 : kRowKeys) * D * 2;
    const __amdgpu_buffer_rsrc_t rk =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(Ku + (size_t)r0 * D), 0, bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < EPT / 8; ++i) {
      const v4u x = __builtin_amdgcn_raw_buffer_load_b128(rk, k_src, 16 * i, 0);
      kraw[4 * i] = x.x; kraw[4 * i + 1] = x.y; kraw[4 * i + 2] = x.z; kraw[4 * i + 3] = x.w;
    }
    if constexpr (OUT) {
      const __amdgpu_buffer_rsrc_t rv =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(Vu + (size_t)r0 * D), 0, bytes, 0x00020000);
#pragma unroll
      for (int i = 0; i < VK; ++i)                        // slots vs + 4 ..: the tile's second half
        vraw[i] = __builtin_amdgcn_raw_buffer_load_b32(rv, v_src, min((i / 4 * 16 + i % 4) * D * 2, bytes), 0);
    }
  };
  auto stage = [&](int kt, unsigned char *val) __attribute__((always_inline)) {
    unsigned char *buf = s_key[kt & 1];
    unsigned plane[4][EPT / 4];
#pragma unroll
    for (int i = 0; i < EPT / 4; ++i) {
      unsigned p[4];
      digits_of4(kraw[2 * i], kraw[2 * i + 1], p);
#pragma unroll
      for (int q = 0; q < 4; ++q) plane[q][i] = p[q];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      unsigned char *dst = buf + k_dst + q * Tile::kPlaneBytes;
      if constexpr (EPT == 16) *reinterpret_cast<uint4 *>(dst) = uint4{plane[q][0], plane[q][1], plane[q][2], plane[q][3]};
      else *reinterpret_cast<uint2 *>(dst) = uint2{plane[q][0], plane[q][1]};
    }
    s_bad[without_digits(kraw) ? kt & 1 : 2] = kt;        // (a branch here would end the block the products stand in)
    if constexpr (OUT) {
      unsigned lo[VK / 2], hi[VK / 2];                    // columns vd and vd + 1 of the thread's keys
#pragma unroll
      for (int i = 0; i < VK / 2; ++i) {
        lo[i] = __builtin_amdgcn_perm(vraw[2 * i + 1], vraw[2 * i], 0x05040100u);
        hi[i] = __builtin_amdgcn_perm(vraw[2 * i + 1], vraw[2 * i], 0x07060302u);
      }
      if constexpr (VK == 8) {
        *reinterpret_cast<uint4 *>(val + v_dst0) = uint4{lo[0], lo[1], lo[2], lo[3]};
        *reinterpret_cast<uint4 *>(val + v_dst1) = uint4{hi[0], hi[1], hi[2], hi[3]};
      } else {
        *reinterpret_cast<uint2 *>(val + v_dst0) = uint2{lo[0], lo[1]};
        *reinterpret_cast<uint2 *>(val + v_dst1) = uint2{hi[0], hi[1]};
      }
    }
  };

  RowDigits<D> qd;
  const bool qbad = __any(!qd.load(Qu + (size_t)qrow * D, g));
  // m: an integer below the query's maximum when it was last moved; lim: by how much a score may pass it, -inf
  // before the first one
  double m = 0.0, lim = -__builtin_inf(), L = 0.0;
  v4f O[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) O[b] = v4f{0.f, 0.f, 0.f, 0.f};
  // the tile whose weights are still to come: base-2 scores less m of its two halves
  double y[2][4];
  auto no_weight = [&](double (&yy)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < 4; ++w) yy[w] = kNoWeight;
  };
  no_weight(y[0]);
  no_weight(y[1]);

  auto products = [&](int kt, int half, v4i (&s)[7]) __attribute__((always_inline)) {
    const unsigned char *buf = s_key[kt & 1];
#pragma unroll
    for (int i = 0; i < 7; ++i) s[i] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int pa = 0; pa < 4; ++pa)
        dot_planes(*reinterpret_cast<const v4i *>(buf + Tile::key_at(half, pa, kc, g, c)), qd.d[kc], pa, s);
  };
  auto raise_max = [&](double (&y)[2][4]) __attribute__((always_inline)) {
    double top = fmax(fmax(fmax(y[0][0], y[0][1]), fmax(y[0][2], y[0][3])), fmax(fmax(y[1][0], y[1][1]), fmax(y[1][2], y[1][3])));
    if (__any(top > lim)) {
      top = fmax(top, __shfl_xor(top, 16));
      top = fmax(top, __shfl_xor(top, 32));
      const bool none = top == -__builtin_inf();          // nothing to see yet
      const double d = none ? 0.0 : lim == -__builtin_inf() ? ceil(top) - 1.0 : fmax(0.0, ceil(top) - 1.0);
      const int k = d <= 0.0 ? 0 : d < 2000.0 ? -(int)d : -2000;   // the rescaling is a power of two
      const float af = __builtin_ldexpf(1.f, k);
      L = __builtin_ldexp(L, k);
#pragma unroll
      for (int b = 0; b < DB; ++b) O[b] *= af;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        y[0][w] -= d;
        y[1][w] -= d;
      }
      m += d;
      lim = none ? lim : kSlack;
    }
  };
  auto scores = [&](const v4i (&s)[7], double (&yy)[4]) __attribute__((always_inline)) {
    const DotParts p = dot_join(s);
#pragma unroll
    for (int w = 0; w < 4; ++w) yy[w] = dot_affine(p, w, cs, -m);
  };
  // the weights of half `half` out of its scores, into hi + lo pairs and L
  v8h ph, pl;
  auto weigh = [&](const double (&yy)[4], int half) __attribute__((always_inline)) {
    double e[4];
    exp2_f64(yy, e);
    float ef[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      ef[w] = (float)e[w];
      // keep the fp32 value: folded into one fp64 -> fp16 conversion this becomes a long software
      // sequence (there is no such instruction)
      asm("" : "+v"(ef[w]));
    }
    L += (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const _Float16 hi = (_Float16)ef[w];
      ph[4 * half + w] = hi;
      pl[4 * half + w] = (_Float16)(ef[w] - (float)hi);
    }
  };
  // O += V^T p; only0: the tile's second half lies after all of the wave's queries
  auto add_values = [&](const unsigned char *val, bool only0) __attribute__((always_inline)) {
    if constexpr (!OUT) return;
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      uint4 raw = *reinterpret_cast<const uint4 *>(val + Tile::val_at(b, c, g));
      if (only0) raw.z = raw.w = 0;                       // whatever is there, infinities too, has no part in it
      const v8h a = __builtin_bit_cast(v8h, raw);
      O[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ph, O[b], 0, 0, 0);
      O[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, pl, O[b], 0, 0, 0);
    }
  };
  if (tid < 2) s_bad[tid] = -1;
  if (tid == 0 && pb.grp == 0 && u == ukv * (size_t)G) zero0[ukv] = zero1[ukv] = 0u;
  if constexpr (OUT)                                      // the values of the tile before the first: weighed 0
    for (int i = tid; i < Tile::kValBytes / 4; i += 64 * W) reinterpret_cast<unsigned *>(s_val[2])[i] = 0u;
  fetch(0);
  __syncthreads();
  unsigned char *v_prev = s_val[2], *v_cur = s_val[0], *v_next = s_val[1];
  stage(0, v_cur);
  fetch(kt_last > 0 ? 1 : 0);
  for (int kt = 0; kt <= kt_last; ++kt) {
    // tile kt is complete; nobody still reads the buffers that tile kt + 1 will go into
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    const int j0 = kt * kRowKeys;
    v4i s[7];
    const bool slow = qbad || __builtin_amdgcn_readfirstlane(s_bad[kt & 1]) == kt;
    if (kt < kt_wave && !slow) {                          // wave-uniform: every key before every query
      double yn[2][4];
      // one matrix instruction, then the vector instructions it runs beside
      auto interleave = [](auto count) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < count.value; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // (4: 7 % slower)
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      products(kt, 0, s);
      weigh(y[0], 0);                                     // the tile before
      weigh(y[1], 1);
      interleave(std::integral_constant<int, 16 * KC>{});
      scores(s, yn[0]);
      products(kt, 1, s);
      add_values(v_prev, false);
      stage(kt + 1, v_next);
      fetch(kt + 2 <= kt_last ? kt + 2 : kt_last);
      interleave(std::integral_constant<int, (OUT ? 2 * DB : 0) + 16 * KC>{});
      scores(s, yn[1]);
      raise_max(yn);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        y[0][w] = yn[0][w];
        y[1][w] = yn[1][w];
      }
    } else {
      if (kt <= kt_wave) {
        if (kt > 0) {                                     // the tile before
          weigh(y[0], 0);
          weigh(y[1], 1);
          add_values(v_prev, false);
        }
        const bool only0 = j0 + 16 > q0 + 15;             // the second half lies after all of the wave's queries
        if (slow) {
          v4d d[2];
          dot_tiles_f64<D, 2>([&](int i) { return Ku + (size_t)(j0 + i < P ? j0 + i : P - 1) * D; }, Qu + (size_t)qrow * D, g, c, d);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            y[0][w] = fma(d[0][w], cs, -m);
            y[1][w] = fma(d[1][w], cs, -m);
          }
        } else {
          products(kt, 0, s);
          scores(s, y[0]);
          if (!only0) {                                   // (else masked below)
            products(kt, 1, s);
            scores(s, y[1]);
          }
        }
        if (kt == kt_wave) {
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            y[0][w] = (j0 + 4 * g + w <= qi) ? y[0][w] : -__builtin_inf();
            y[1][w] = (j0 + 16 + 4 * g + w <= qi) ? y[1][w] : -__builtin_inf();
          }
        }
        raise_max(y);
        // no weight for keys after the query, scores of -inf and what is not a number
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          y[0][w] = y[0][w] > kNoWeight ? y[0][w] : kNoWeight;
          y[1][w] = y[1][w] > kNoWeight ? y[1][w] : kNoWeight;
        }
        if (kt == kt_wave) {                              // the wave's last tile
          weigh(y[0], 0);
          weigh(y[1], 1);
          add_values(v_cur, only0);
        }
      }
      if (kt < kt_last) {
        stage(kt + 1, v_next);
        fetch(kt + 2 <= kt_last ? kt + 2 : kt_last);
      }
    }
    unsigned char *t = v_prev;
    v_prev = v_cur; v_cur = v_next; v_next = t;
  }
  L += __shfl_xor(L, 16);
  L += __shfl_xor(L, 32);
  if (qi < P) {
    if (g == 0) lse[u * (size_t)P + qi] = fma(m, kLn2, log(L));
    if constexpr (OUT) {
      // O[b][w] is output element DB (4 g + w) + b: the lane's elements are one run of 4 DB halves
      const float inv = (float)(1.0 / L);
      __half run[4 * DB];
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int b = 0; b < DB; ++b) run[DB * w + b] = __float2half_rn(O[b][w] * inv);
      __half *orow = out + (u * (size_t)P + qi) * D + 4 * DB * g;
#pragma unroll
      for (int i = 0; i < 4 * DB / 8; ++i) reinterpret_cast<uint4 *>(orow)[i] = reinterpret_cast<const uint4 *>(run)[i];
    }
  }
}

template <int D>
static hipError_t launch_rows_t(const void *Q, const void *K, const void *V, unsigned UG, int G, int P, double *lse,
                                void *out, unsigned *zero0, unsigned *zero1, hipStream_t st)
{
  const unsigned ngrp = (unsigned)((P + 16 * kPrefillWaves - 1) / (16 * kPrefillWaves));
  if (out != nullptr)
    rows_f16_kernel<D, true><<<prefill_grid(UG, ngrp), 64 * kPrefillWaves, 0, st>>>(
        (const __half *)Q, (const __half *)K, (const __half *)V, UG, G, P, lse, (__half *)out, zero0, zero1);
  else
    rows_f16_kernel<D, false><<<prefill_grid(UG, ngrp), 64 * kPrefillWaves, 0, st>>>(
        (const __half *)Q, (const __half *)K, (const __half *)V, UG, G, P, lse, nullptr, zero0, zero1);
  return hipGetLastError();
}

hipError_t launch_rows_f16(const void *Q, const void *K, const void *V, unsigned UG, int G, int P, int D, double *lse,
                           void *out, unsigned *zero0, unsigned *zero1, hipStream_t st)
{
  return D == 128 ? launch_rows_t<128>(Q, K, V, UG, G, P, lse, out, zero0, zero1, st)
                  : launch_rows_t<64>(Q, K, V, UG, G, P, lse, out, zero0, zero1, st);
}

// -------------------------------------------------------------------------------------
// Exact column sums sum_i e^{s_ij - lse_i} of listed keys (list == nullptr: of every key): the accumulated
// attention probability of each prompt token (H2O's score, Sec. 2.1).  A workgroup takes 16 NT
// listed keys, ascending, splits their rows into digit planes once, into the LDS, and deals the query
// tiles of 16, from the one of its earliest key on and over all the unit's query heads, to its W
// waves.  A wave splits a query tile in registers and multiplies it with every key tile that
// begins before the tile ends (a prefix of them).  No atomics: every wave sums its query tiles in order, and
// the waves' sums are added in order.  The length of the list is only known on the device: a unit gets
// enough workgroups for a list a little longer than the budget, and they loop should it be longer.
// grid = ceil(U / 8) * 8 * groups.
// -------------------------------------------------------------------------------------
template <int D, int NT, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void columns_f16_kernel(
    const __half *__restrict__ Q, const __half *__restrict__ K, unsigned U, int G, int P, const double *__restrict__ lse,
    const int32_t *__restrict__ list, const int32_t *__restrict__ count, int groups, double *__restrict__ colsum)
{
  constexpr int KC = D / 64, KEYS = 16 * NT, kTile = 4 * KC * 1024;
  __shared__ __attribute__((aligned(16))) unsigned char s_key[NT * kTile];
  __shared__ double s_sum[W][KEYS];
  __shared__ int s_pos[KEYS], s_bad[NT];
  const PrefillBlock pb = prefill_block(blockIdx.x, groups);
  if (pb.u >= U) return;
  const size_t u = pb.u;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64, g = l / 16, c = l % 16;
  const __half *Ku = K + u * (size_t)P * D;
  const int32_t *li = list ? list + u * (size_t)P : nullptr;
  const int n = list ? count[u] : P, nblk = (P + 15) / 16;
  const double cs = kLog2E / sqrt((double)D);
  // block of 16 digits [(kc, g)][key], the key's place turned by the block as in the row pass
  auto key_at = [](int t, int plane, int kc, int gg, int row) {
    return t * kTile + plane * (KC * 1024) + (kc * 4 + gg) * 256 + (row ^ (2 * (kc * 4 + gg))) * 16;
  };
  for (int grp = pb.grp; grp * KEYS < n; grp += groups) {
    const int nk = n - grp * KEYS < KEYS ? n - grp * KEYS : KEYS, nt = (nk + 15) / 16;
    if (tid < KEYS) s_pos[tid] = tid < nk ? (li ? li[grp * KEYS + tid] : grp * KEYS + tid) : INT_MAX;
    if (tid < NT) s_bad[tid] = 0;
    __syncthreads();
    for (int i = tid; i < nt * 16 * (D / 16); i += 64 * W) {    // a piece of 16 elements of a listed key
      const int key = i / (D / 16), e = i % (D / 16) * 16;
      const uint4 *src = reinterpret_cast<const uint4 *>(Ku + (size_t)s_pos[key < nk ? key : 0] * D + e);
      const uint4 x = src[0], y = src[1];
      const unsigned w[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
      unsigned plane[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        unsigned p[4];
        digits_of4(w[2 * j], w[2 * j + 1], p);
#pragma unroll
        for (int q = 0; q < 4; ++q) plane[q][j] = p[q];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint4 *>(s_key + key_at(key / 16, q, e / 64, e % 64 / 16, key % 16)) =
            uint4{plane[q][0], plane[q][1], plane[q][2], plane[q][3]};
      if (without_digits(w)) s_bad[key / 16] = 1;
    }
    __syncthreads();
    const int it0 = s_pos[0] / 16, per = nblk - it0;      // query tiles per head
    double sum[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int w = 0; w < 4; ++w) sum[t][w] = 0.0;
    for (int idx = wave; idx < G * per; idx += W) {
      const int h = idx / per, it = it0 + idx - h * per, qi = it * 16 + c, qrow = qi < P ? qi : P - 1;
      const __half *qp = Q + ((u * G + h) * (size_t)P + qrow) * D;
      const double lq = lse[(u * G + h) * (size_t)P + qrow];
      RowDigits<D> qd;
      const bool qbad = __any(!qd.load(qp, g));
      // rows past the prompt, and rows without a log-sum, have no part in any column
      const bool has_sum = qi < P && fabs(lq) < 1e300;
      const double shift = has_sum ? -lq * kLog2E : -1e300;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t >= nt || s_pos[16 * t] > it * 16 + 15) break;             // wave-uniform
        double y[4], e[4];
        if (!qbad && !s_bad[t]) {
          v4i s[7];
#pragma unroll
          for (int i = 0; i < 7; ++i) s[i] = v4i{0, 0, 0, 0};
#pragma unroll
          for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int pa = 0; pa < 4; ++pa)
              dot_planes(*reinterpret_cast<const v4i *>(s_key + key_at(t, pa, kc, g, c)), qd.d[kc], pa, s);
          const DotParts p = dot_join(s);
#pragma unroll
          for (int w = 0; w < 4; ++w) y[w] = dot_affine(p, w, cs, shift);
        } else {
          v4d s[1];
          dot_tiles_f64<D, 1>([&](int i) { return Ku + (size_t)s_pos[16 * t + i < nk ? 16 * t + i : 0] * D; }, qp, g, c, s);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            // (a row without a log-sum may hold infinite scores)
            y[w] = fma(s[0][w], cs, shift);
            y[w] = has_sum && y[w] > kNoWeight ? y[w] : kNoWeight;
          }
        }
        exp2_f64(y, e);
        if (s_pos[16 * t + 15] > it * 16) {                             // wave-uniform: not every key precedes every query
#pragma unroll
          for (int w = 0; w < 4; ++w) e[w] = s_pos[16 * t + 4 * g + w] <= qi ? e[w] : 0.0;
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) sum[t][w] += e[w];
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) sum[t][w] += __shfl_xor(sum[t][w], o);
        if (c == 0) s_sum[wave][16 * t + 4 * g + w] = sum[t][w];
      }
    __syncthreads();
    if (tid < nk) {
      double total = 0.0;
#pragma unroll
      for (int w = 0; w < W; ++w) total += s_sum[w][tid];
      colsum[u * (size_t)P + s_pos[tid]] = total;
    }
    __syncthreads();                                      // before the next list's positions
  }
}

template <int D, int NT, int W>
static hipError_t launch_columns_t(const void *Q, const void *K, unsigned U, int G, int P, const double *lse,
                                   const int32_t *list, const int32_t *count, int keys, double *colsum, hipStream_t st)
{
  const int groups = (keys + 16 * NT - 1) / (16 * NT);
  columns_f16_kernel<D, NT, W><<<prefill_grid(U, (unsigned)groups), 64 * W, 0, st>>>(
      (const __half *)Q, (const __half *)K, U, G, P, lse, list, count, groups, colsum);
  return hipGetLastError();
}

hipError_t launch_columns_f16(const void *Q, const void *K, unsigned U, int G, int P, int D, const double *lse,
                              const int32_t *list, const int32_t *count, int C, double *colsum, hipStream_t st)
{
  const int keys = list && C + 16 < P ? C + 16 : P;       // a handful of tokens in doubt behind the budget
  const int tiles = (keys + 15) / 16;
#define LESSDEC_COLUMNS(NT, W)                                                                       \
  return D == 128 ? launch_columns_t<128, NT, W>(Q, K, U, G, P, lse, list, count, keys, colsum, st)  \
                  : launch_columns_t<64, NT, W>(Q, K, U, G, P, lse, list, count, keys, colsum, st)
  // (NT key tiles to a workgroup, W waves; microseconds of a prompt phase.)  Few units: many waves divide a sweep, and a
  // unit's keys, whose sweeps differ in length, are spread thin (<2, 8>: 8 units x 2048 tokens 188, <8, 8> 239; 128 x
  // 4 heads x 2048, 204 kept: 3480 against 3590), unless there are so many keys that splitting the queries anew for every
  // 32 costs more (64 x 500, all kept: <8, 8> 144, <2, 8> 153).  Else long sweeps: many keys to a split query tile
  // (256 x 2 heads x 1000: <8, 8> 766, <8, 4> 786, <2, 8> 834; 1024 x 500: <8, 4> 610, <8, 8> 631, <4, 2> 662).  Short
  // ones, where a workgroup has few query tiles to deal out: two waves, and four key tiles where they come out
  // filled (2048 x 64, all kept: <4, 2> 108, <8, 8> 162; 2048 x 200: <2, 2> 439, <4, 2> 482, <8, 8> 566; 2048 x 300:
  // <4, 2> 653, <2, 2> 694, <8, 4> 685; 512 x 400: <4, 2> 274, <2, 2> 277, <8, 4> 314).
  const size_t wide = (size_t)U * ((tiles + 7) / 8);      // workgroups of eight key tiles
  if (U < 256 && (tiles < 24 || wide < 256)) LESSDEC_COLUMNS(2, 8);
  if ((long)G * P > 448) {
    if (wide < 768) LESSDEC_COLUMNS(8, 8);
    LESSDEC_COLUMNS(8, 4);
  }
  if (tiles % 4 == 0 || tiles % 4 == 3) LESSDEC_COLUMNS(4, 2);
  LESSDEC_COLUMNS(2, 2);
#undef LESSDEC_COLUMNS
}

}  // namespace lessdec
