// Prompt phase, fp16 storage: causal rows (log-sums and attention outputs) and exact column sums,
// with the scores as exact integer products of digit planes (lessdec_digits.h).
#include <type_traits>

#include "lessdec_digits.h"
#include "lessdec_internal.h"
#include "lessdec_lds.h"
#include "lessdec_mlp.h"
#include "lessdec_prefill.h"

namespace lessdec {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

// -------------------------------------------------------------------------------------
// Row pass.  key_digits_kernel splits every key into digit planes once; then a workgroup of four waves owns 64 consecutive
// queries, a wave 16 of them, and sweeps the key tiles of 32 up to its last diagonal.  The tiles go from memory into the
// LDS without passing through registers: digits in operand order, value rows as they are, transposed by the reads of
// p V.  A wave multiplies each 16-key half with its queries (digits in registers): scores S^T[key][query], lane (g, c)
// holding keys 4 g + w of query c.
// The running maximum m is an integer in base-2 units, the one below the largest score of the first tile (so that
// the largest weight is above 1 and the fp16 pairs' floor of 2^-24 as far below it as with weights up to 1), moved when a
// score passes it by kSlack, which is rare and exact.  The weights are fp64; their sum gives lse, and p V takes
// them as an fp16 pair hi + lo (22 bits) with fp32 accumulation.  Leaves lse_i = ln sum_j e^{s_ij}.
// A tile with a value that has no digits (|x| >= 127), and every tile of a wave whose queries hold one, is multiplied
// in fp64 instead, from rows read as 16-byte pieces: 512 units x 1024 tokens with such a key channel in every token took
// 2907 us in all against 1486 with digits throughout and 3010 with fp64 products throughout (10560 with halves read
// singly, each product waiting for its own).
//
// What bounds it: issue (an instruction in 98 % of the SIMD cycles at 8192 tokens) and power.  With the matrix units busy
// half of the time the card lowers its clock, from 2.35 GHz to 2.0 here, more so the more the operands' bits change: a
// schedule without gaps gained cycles and no time, fewer products and fewer vector instructions do.  Hence
//   - keys are split once, not by every workgroup that meets them (62 of 222 vector instructions per 16 x 16 tile);
//   - rows are scaled by powers of two, so that most blocks have an empty lowest plane and are nine products of
//     planes, not sixteen (ScaledDigits; 30 matrix instructions per 16 x 16 tile, p V's 8 among them, where there were 40);
//   - one path for all tiles: with a second one for those before the diagonal the compiler moved the scores and the
//     accumulators between registers in every tile (30 instructions);
//   - three waves a SIMD in place of two and a software pipeline: no slower with long sweeps, and with short ones the
//     start and the end of a workgroup, in which its waves wait, are covered (2810 against 3040 us at 1024 tokens).
//
// MASKED: Lambda-masking taken through the prompt token by token (Sec. 4, "Setup"; Sec. 3.2 builds the same matrix for
// training), all rows at once.  Under that policy the cache that token t meets is known beforehand: the first Nh tokens and
// the Nr tokens before it; the pairs discarded by then are Nh .. t - Nr - 1.  Row t of the attention matrix therefore
// has e^{q_t k_j / sqrt(D)} where pair j is cached (or is t itself) and phi(q_t) psi(k_j)^T where it was discarded, and
// out_t = (row t) V / (row t) 1 is Eq. 3 with H, z of Eq. 6.  The workgroup sweeps the tiles that can hold cached pairs
// of any of its queries, other entries masked out; then the discarded pairs: those before the last prefix state (every 64
// keys) older than a wave's windows come with that state, on fp32 matrix tiles, the few tiles after it entry by entry
// (psi(K) phi(Q)^T on fp64 matrix tiles, R / 4 instructions; values through the LDS as before).  m rises once to the integer
// below log2 of an upper bound of the low-rank weights, phi(q) . max_j psi(k_j).  Leaves lse_t = m_t ln 2 + ln(sum of the
// entries that H2O's scores are normalised by): all, or with the sparse-denominator flag the exponentials.
// 320 units x 2048 tokens, window 158, rank 16: 551 us and 72 for the digits, 1158 with scores on fp64 matrix tiles.
//
// 2048 units x 1024 tokens: 3600 us before, 2480 now and 217 for the digits (1.34 GB at 6.2 TB/s), three shares of units; 128 x
// 8192: 11000, 8030 and 109, two; 32 x 777: 65, 51 and 6.
// -------------------------------------------------------------------------------------
constexpr int kRowKeys = 32;
constexpr double kSlack = 15.0;                           // weights up to 2^15: they fit a half
constexpr double kNoWeight = -5000.0;                     // the weight of this score is 0

// One tile of keys and values in the LDS.  Key digits lie as in memory (key_digits_kernel): a wave's read of a plane is one
// contiguous KiB.  Value rows are whole, their 16-byte chunks permuted by val_swizzle.
template <int D>
struct RowTile {
  static constexpr int KC = D / 64;
  static constexpr int kHalfBytes = 4 * KC * 1024;        // planes of 16 keys
  static constexpr int kKeyBytes = 2 * kHalfBytes, kValBytes = kRowKeys * D * 2;
  // 16 lanes of a transposing read touch 8 bytes in each of four chunks of four consecutive rows
  static __device__ inline int val_swizzle(int row) { return D == 128 ? row & 3 : (row >> 1) & 1; }
};
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;
// The 16-lane groups' transposing read: lane i of a group points at 4 halves, element i % 4 .. of row i / 4 of the group's
// four rows by pieces of 4 columns, and gets column i of the four rows.
__device__ inline v4s lds_read_transposed(unsigned offset)
{
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)(unsigned long long)offset);
}
// What the row pass has to know of a tile of 32 keys besides its digits, one word: bit 0: a value has no digits; bits 2 + 2
// half + kc: that block has lowest digits; bits 8 + 8 half ..: scale of the half.
struct TileWord {
  unsigned w;
  __device__ inline bool bad() const { return w & 1; }
  __device__ inline unsigned lowest(int half) const { return w >> (2 + 2 * half) & 3; }
  __device__ inline int scale(int half) const { return w >> (8 + 8 * half) & 0xff; }
};

// Digit planes of every key, laid out as the row pass wants them in the LDS: per unit, per 16 keys (past the prompt the last
// one again, up to a whole tile of 32) a block [plane][kc][lane = 16 g + row] of 16 digits.  One scale per 16 keys.
// Lowest planes that are empty are not written (nothing reads them).  Bound by memory.
// fill: words of the decode step's exchange array to be emptied on the way, which saves a launch.
template <int D>
__global__ __launch_bounds__(128) void key_digits_kernel(const __half *__restrict__ K, unsigned tiles, int P,
                                                         unsigned char *__restrict__ digits, unsigned *__restrict__ words,
                                                         unsigned *__restrict__ fill, size_t fill_count)
{
  constexpr int KC = D / 64;
  __shared__ unsigned s_word[2];
  for (size_t i = (size_t)blockIdx.x * 128 + threadIdx.x; i < fill_count; i += (size_t)gridDim.x * 128) fill[i] = kMlpEmpty;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), l = threadIdx.x % 64, g = l / 16, c = l % 16;
  const unsigned u = blockIdx.x / tiles, t = blockIdx.x % tiles;
  const int row = (int)t * kRowKeys + 16 * wave + c;
  ScaledDigits<D> kd;
  const bool bad = __any(!kd.template load<true>(K + ((size_t)u * P + (row < P ? row : P - 1)) * D, g));
  const unsigned lowest = kd.lowest();
  unsigned char *dst = digits + ((size_t)blockIdx.x * 2 + wave) * RowTile<D>::kHalfBytes + l * 16;
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
      if (p > 0 || (lowest >> kc & 1)) *reinterpret_cast<v4i *>(dst + (p * KC + kc) * 1024) = kd.d[kc][p];
  if (l == 0) s_word[wave] = (bad ? 1u : 0u) | lowest << (2 + 2 * wave) | (unsigned)kd.scale << (8 + 8 * wave);
  __syncthreads();
  if (threadIdx.x == 0) words[blockIdx.x] = s_word[0] | s_word[1];
}

// OUT: attention outputs are wanted too.  MASKED: the rows of Lambda-masking taken through the prompt (above).  MAPS: the
// workgroups from n_rows on evaluate psi of the prompt's keys, which nothing here needs: few units leave the chip room for them.
template <int D, bool OUT, bool MASKED, bool MAPS>
__global__ __launch_bounds__(64 * kPrefillWaves) __attribute__((amdgpu_waves_per_eu(3, 3))) void rows_f16_kernel(
    const __half *__restrict__ Q, const __half *__restrict__ K, const __half *__restrict__ V, unsigned U, int G, int P,
    const unsigned char *__restrict__ digits, const unsigned *__restrict__ words,
    double *__restrict__ lse, __half *__restrict__ out, unsigned *__restrict__ zero0, unsigned *__restrict__ zero1, const MaskedArgs mk, const MlpArgs maps, unsigned n_rows)
{
  // two buffers of keys and two of values, and 64 bytes of zeros
  constexpr int kZero = 2 * (RowTile<D>::kKeyBytes + RowTile<D>::kValBytes), kRows = kZero + 64;
  constexpr int kLds = MAPS && mlp_psi_lds(kPsiTiles) > kRows ? mlp_psi_lds(kPsiTiles) : kRows;   // the maps' sums lie in the tiles' place
  __shared__ __attribute__((aligned(64))) unsigned char s_lds[kLds];
  if constexpr (MAPS) {
    if (blockIdx.x >= n_rows) {
      mlp_psi_block<D, kPsiTiles>(maps, blockIdx.x - n_rows, s_lds);
      return;
    }
  }
  // U counts query rows here: unit u's G query heads are rows u G .. u G + G - 1 of Q, out and
  // lse, and attend over unit u's keys and values
  using Tile = RowTile<D>;
  constexpr int W = kPrefillWaves, KC = D / 64, DB = D / 16, BQ = 16 * W;
  const int ngrp = (P + BQ - 1) / BQ;
  const PrefillBlock pb = prefill_block(blockIdx.x, ngrp);
  if (pb.u >= U) return;                                  // uniform over the workgroup
  const int grp = ngrp - 1 - pb.grp;                      // long rows first
  const size_t u = pb.u, ukv = u / (unsigned)G;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64, g = l / 16, c = l % 16;
  const __half *Qu = Q + u * (size_t)P * D, *Ku = K + ukv * (size_t)P * D, *Vu = V + ukv * (size_t)P * D;
  const int tiles = (P + kRowKeys - 1) / kRowKeys;
  const unsigned char *Du = digits + ukv * (size_t)tiles * Tile::kKeyBytes;
  const unsigned *wu = words + ukv * (size_t)tiles;
  const int q0 = grp * BQ + wave * 16;                    // the wave's first query
  const int qi = q0 + c, qrow = qi < P ? qi : P - 1;
  const int kt_last = ((grp * BQ + BQ < P ? grp * BQ + BQ : P) - 1) / kRowKeys;   // the workgroup's last tile
  const int kt_wave = q0 < P ? q0 / kRowKeys : -1;        // the wave's last tile; none
  const double cs = kLog2E / sqrt((double)D);             // q . k to base-2 units

  // Tile kt into the LDS: the workgroup's waves bring 1 KiB pieces, key digits as they lie, value rows with their 16-byte
  // chunks permuted within a row (val_swizzle) so that the four rows of a 16-lane group lie in different banks.  (Two groups,
  // whose rows are four apart, still meet in them: two cycles more for each transposing read, 27 % of the cycles that the LDS is
  // busy at 8192 tokens.)  Rows past the prompt repeat the last one: they come after every query.
  constexpr int RB = 2 * D, kRowsPer = 1024 / RB, CH = RB / 16;       // bytes, rows and chunks of a value piece
  auto load_tile = [&](int kt, unsigned char *key, unsigned char *val, bool keys) __attribute__((always_inline)) {
    int lane = l;
    asm("" : "+v"(lane));                                 // (as in add_values)
    const int vr = lane / CH, vch = lane % CH;            // row and chunk within the piece
    if (keys)
#pragma unroll
    for (int i = 0; i < Tile::kKeyBytes / 1024 / W; ++i) {
      const int piece = (wave * (Tile::kKeyBytes / 1024 / W) + i) * 1024;
      lds_load<16>(Du + (size_t)kt * Tile::kKeyBytes + piece, 1024, lane * 16, key + piece);
    }
    if constexpr (OUT) {
      const int r0 = kt * kRowKeys, last = P - 1 - r0;    // last row of the tile that exists
#pragma unroll
      for (int i = 0; i < Tile::kValBytes / 1024 / W; ++i) {
        const int piece = wave * (Tile::kValBytes / 1024 / W) + i, row = piece * kRowsPer + vr;
        const int from = (row < last ? row : last) * RB + (vch ^ Tile::val_swizzle(row)) * 16;
        lds_load<16>(Vu + (size_t)r0 * D, Tile::kValBytes, from, val + piece * 1024);
      }
    }
  };

  // The tiles to sweep: all up to the last diagonal; MASKED: those that can hold a cached pair of the workgroup's queries
  const int q0b = grp * BQ, q_end = (q0b + BQ < P ? q0b + BQ : P) - 1;
  int nfirst = 0, band0 = 0, tiles_here = kt_last + 1;
  if constexpr (MASKED) {
    nfirst = min((mk.Nh + kRowKeys - 1) / kRowKeys, kt_last + 1);
    band0 = max(nfirst, q0b > mk.Nr ? (q0b - mk.Nr) / kRowKeys : 0);
    tiles_here = nfirst + kt_last + 1 - band0;
  }
  auto tile_of = [&](int i) { return !MASKED || i < nfirst ? i : band0 + i - nfirst; };
  unsigned char *k_cur = s_lds, *k_next = k_cur + Tile::kKeyBytes, *v_cur = k_next + Tile::kKeyBytes, *v_next = v_cur + Tile::kValBytes;
  unsigned char *s_zero = s_lds + kZero;
  auto swap_buffers = [&] {
    unsigned char *t = v_cur;
    v_cur = v_next; v_next = t;
    t = k_cur; k_cur = k_next; k_next = t;
  };
  load_tile(tile_of(0), k_cur, v_cur, true);
  TileWord word = {wu[tile_of(0)]};
  ScaledDigits<D> qd;
  const bool qbad = __any(!qd.template load<false>(Qu + (size_t)qrow * D, g));
  const unsigned qlow = qd.lowest();
  const double cq = __builtin_ldexp(cs * kDotUnit, -qd.scale);         // a product of digit planes to base-2 units, but for the keys' scale
  // m: an integer below the query's maximum when it was last moved, which a score may pass by kSlack
  double m = 0.0, L = 0.0;
  v4f O[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) O[b] = v4f{0.f, 0.f, 0.f, 0.f};
  // base-2 scores less m of the keys of a half: nine products of the three upper planes, and those with the lowest
  // planes where there are any
  auto scores = [&](const unsigned char *key, const TileWord word, int half, double *yy) __attribute__((always_inline)) {
    const unsigned char *at = key + half * Tile::kHalfBytes + l * 16;
    auto plane = [&](int kc, int p) __attribute__((always_inline)) { return *reinterpret_cast<const v4i *>(at + (p * KC + kc) * 1024); };
    v4i s[7];
#pragma unroll
    for (int i = 2; i < 7; ++i) s[i] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      v4i k[4];
#pragma unroll
      for (int pa = 1; pa < 4; ++pa) k[pa] = plane(kc, pa);
#pragma unroll
      for (int pb = 1; pb < 4; ++pb)
#pragma unroll
        for (int pa = 1; pa < 4; ++pa) s[pa + pb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(k[pa], qd.d[kc][pb], s[pa + pb], 0, 0, 0);
    }
    const unsigned klow = word.lowest(half);
    const int e = -word.scale(half);
    const double c40 = __builtin_ldexp(cq, e + 40), c32 = __builtin_ldexp(cq, e + 32), c16 = __builtin_ldexp(cq, e + 16);
#pragma unroll
    for (int w = 0; w < 4; ++w) yy[w] = -m;
    if (klow | qlow) {                                    // wave-uniform
      s[0] = s[1] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        if (klow >> kc & 1) {
          const v4i k0 = plane(kc, 0);
#pragma unroll
          for (int pb = 0; pb < 4; ++pb) s[pb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(k0, qd.d[kc][pb], s[pb], 0, 0, 0);
        }
        if (qlow >> kc & 1) {
#pragma unroll
          for (int pa = 1; pa < 4; ++pa) s[pa] = __builtin_amdgcn_mfma_i32_16x16x64_i8(plane(kc, pa), qd.d[kc][0], s[pa], 0, 0, 0);
        }
      }
      const double c0 = __builtin_ldexp(cq, e);
      const v4i p10 = (s[1] << 8) + s[0];
#pragma unroll
      for (int w = 0; w < 4; ++w) yy[w] = fma((double)p10[w], c0, -m);
    }
    const v4i p65 = (s[6] << 8) + s[5], p32 = (s[3] << 8) + s[2];
#pragma unroll
    for (int w = 0; w < 4; ++w)
      yy[w] = fma((double)p65[w], c40, fma((double)s[4][w], c32, fma((double)p32[w], c16, yy[w])));
  };
  // High word of the limit, least before the first maximum: as signed integers the high words order what matters, everything
  // below zero lies below kSlack.
  int lim_hi = INT_MIN;
  // weights of half `half` as hi + lo pairs
  v8h ph, pl;
  float one = 1.f;
  asm("" : "+s"(one));                                    // unknown to the compiler, which else makes a subtraction of the fma
  auto split = [&](const double (&e)[4], int half) __attribute__((always_inline)) {
    float ef[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      ef[w] = (float)e[w];
      // keep the fp32 value: folded into one fp64 -> fp16 conversion this becomes a long software
      // sequence (there is no such instruction)
      asm("" : "+v"(ef[w]));
    }
#pragma unroll
    for (int w = 0; w < 4; w += 2) {
      unsigned p = __builtin_bit_cast(unsigned, v2h{(_Float16)ef[w], (_Float16)ef[w + 1]});
      asm("" : "+v"(p));                                  // converted once, as a pair
      const v2h hi = __builtin_bit_cast(v2h, p);
      // x - hi is exact in fp32; as fused multiply-adds that take the halves as they are
      const v2h lo = {(_Float16)__builtin_fmaf(-(float)hi.x, one, ef[w]), (_Float16)__builtin_fmaf(-(float)hi.y, one, ef[w + 1])};
      ph[4 * half + w] = hi.x;
      ph[4 * half + w + 1] = hi.y;
      pl[4 * half + w] = lo.x;
      pl[4 * half + w + 1] = lo.y;
    }
  };
  // the same out of its scores, and their sum into L
  auto weigh = [&](const double *yy, int half) __attribute__((always_inline)) {
    double e[4];
    exp2_f64<4>({yy[0], yy[1], yy[2], yy[3]}, e);
    L += (e[0] + e[1]) + (e[2] + e[3]);
    split(e, half);
  };
  // everything so far times 2^-d, d an integer >= 0 (per query)
  auto rescale = [&](double d) __attribute__((always_inline)) {
    const int k = d <= 0.0 ? 0 : d < 2000.0 ? -(int)d : -2000;
    const float af = __builtin_ldexpf(1.f, k);
    L = __builtin_ldexp(L, k);
#pragma unroll
    for (int b = 0; b < DB; ++b) O[b] *= af;
    m += d;
  };
  auto raise_max = [&](double (&y)[8]) __attribute__((always_inline)) {
    double top = fmax(fmax(fmax(y[0], y[1]), fmax(y[2], y[3])), fmax(fmax(y[4], y[5]), fmax(y[6], y[7])));
    if (__any(lim_hi == INT_MIN || top > kSlack)) {
      top = fmax(top, __shfl_xor(top, 16));
      top = fmax(top, __shfl_xor(top, 32));
      const bool none = top == -__builtin_inf();          // nothing to see yet
      const double d = none ? 0.0 : lim_hi == INT_MIN ? ceil(top) - 1.0 : fmax(0.0, ceil(top) - 1.0);
      rescale(d);
#pragma unroll
      for (int w = 0; w < 8; ++w) y[w] -= d;
      lim_hi = none ? lim_hi : __double2hiint(kSlack);
    }
  };
  // O += V^T p; skip0, skip1: no key of that half has a weight for any of the wave's queries.  A lane's four rows of a 16-lane group
  // and the piece of four columns it points at: the transposing read hands lane i column i of the group's four rows.
  // A-operand row i of block b is value column 4 DB (i / 4) + 4 b + i % 4, so that a lane's outputs are one run.
  const int v_at = (4 * g + c / 4) * RB + (((DB / 2) * (c % 4)) ^ Tile::val_swizzle(4 * g + c / 4)) * 16;
  auto add_values = [&](const unsigned char *val, bool skip0, bool skip1) __attribute__((always_inline)) {
    if constexpr (!OUT) return;
    unsigned at0 = lds_offset(val) + v_at, at1 = skip1 ? lds_offset(s_zero) : at0 + 16 * RB;   // (values without a weight may be infinite)
    if (MASKED && skip0) at0 = lds_offset(s_zero);
    asm("" : "+v"(at0), "+v"(at1));                       // else the addresses of all blocks stay in registers between the tiles
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      const v4s h0 = lds_read_transposed((at0 ^ (b / 2 * 16)) + b % 2 * 8), h1 = lds_read_transposed((at1 ^ (b / 2 * 16)) + b % 2 * 8);
      const v8h a = __builtin_bit_cast(v8h, __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7));
      O[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ph, O[b], 0, 0, 0);
      O[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, pl, O[b], 0, 0, 0);
    }
  };
  if (tid < 16) reinterpret_cast<unsigned *>(s_zero)[tid] = 0u;        // (the first tile's barrier stands before its readers)
  if (tid == 0 && pb.grp == 0 && u == ukv * (size_t)G) zero0[ukv] = zero1[ukv] = 0u;
  int lo_wg = 0, nlow = 0;                                // MASKED: the tiles of the second sweep
  if constexpr (MASKED) {
    lo_wg = mk.first_low(q0b) / kRowKeys;
    nlow = max(0, (q_end - 1 - mk.Nr >= 0 ? (q_end - 1 - mk.Nr) / kRowKeys : -1) - lo_wg + 1);
  }
  for (int i = 0; i < tiles_here; ++i) {
    // the tile has arrived for all waves; nobody still reads the buffers that the next one will go into
    lds_arrived<0>();
    lds_barrier();
    const int kt = tile_of(i), j0 = kt * kRowKeys;
    const TileWord here = word;
    if (i + 1 < tiles_here) {
      const int next = tile_of(i + 1);
      load_tile(next, k_next, v_next, true);
      word.w = wu[next];
    } else if (MASKED && nlow > 0) {
      load_tile(lo_wg, k_next, v_next, false);
    }
    // wave-uniform, like all that follows
    if (kt <= kt_wave && (!MASKED || j0 < mk.Nh || j0 + kRowKeys - 1 >= q0 - mk.Nr)) {
      const bool slow = qbad || here.bad();
      // some keys come after some queries (MASKED: or are not cached for them)
      const bool some = MASKED ? j0 + kRowKeys - 1 > q0 || !(j0 + kRowKeys <= mk.Nh || j0 >= q0 + 15 - mk.Nr) : kt == kt_wave;
      // halves without a key for any of them: after them all, or (MASKED) discarded by them all, which come with the second sweep
      auto gone = [&](int a) { return MASKED && a >= mk.Nh && a + 15 < q0 - mk.Nr; };
      const bool skip0 = gone(j0), skip1 = j0 + 16 > q0 + 15 || gone(j0 + 16);
      double y[8];
      if (!slow) {
        if (!skip0) scores(k_cur, here, 0, &y[0]);        // (else masked below)
        if (!skip1) scores(k_cur, here, 1, &y[4]);
      } else {
        v4d d[2];
        dot_tiles_f64<D, 2>([&](int r) { return Ku + (size_t)(j0 + r < P ? j0 + r : P - 1) * D; }, Qu + (size_t)qrow * D, g, c, d);
#pragma unroll
        for (int w = 0; w < 8; ++w) y[w] = fma(d[w / 4][w % 4], cs, -m);
      }
      if (some) {
#pragma unroll
        for (int w = 0; w < 8; ++w) {
          const int kj = j0 + 16 * (w / 4) + 4 * g + w % 4;
          y[w] = kj <= qi && (!MASKED || kj < mk.Nh || kj >= qi - mk.Nr) ? y[w] : -__builtin_inf();
        }
      }
      int top = INT_MIN;
#pragma unroll
      for (int w = 0; w < 8; ++w) top = max(top, __double2hiint(y[w]));
      if (some || slow || __any(top >= lim_hi)) {
        raise_max(y);
        // no weight for keys without a part in it, scores of -inf and what is not a number
#pragma unroll
        for (int w = 0; w < 8; ++w) y[w] = y[w] > kNoWeight ? y[w] : kNoWeight;
      }
      weigh(&y[0], 0);
      __builtin_amdgcn_sched_barrier(0);
      weigh(&y[4], 1);
      __builtin_amdgcn_sched_barrier(0);
      add_values(v_cur, skip0, skip1);
    }
    swap_buffers();
  }
  double Lw = 0.0;                                        // sum of the low-rank entries
  if constexpr (MASKED) {
    const int R = mk.R, lo = mk.first_low(q0);            // first key that this wave's second sweep takes
    const float *psi_u = mk.psi + ukv * (size_t)P * R, *phi_q = mk.phi + (u * (size_t)P + qrow) * R;
    // phi of the lane's query: feature 4 s + g is the lane's operand of step s
    double fq[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r = 4 * s + g;
      const float x = phi_q[r < R ? r : R - 1];
      fq[s] = r < R ? (double)x : 0.0;
    }
    const bool discarded = q0 < P && mk.Nh < q0 + 15 - mk.Nr;     // before some query of the wave
    if (discarded) {
      // No weight of the query can exceed wb = phi(q) . max_j psi(k_j) (all features are >= 0), so m rises to the integer
      // below log2(wb) once, here, and every weight handed to p V below is at most 2.
      const float *pm = mk.psimax + ukv * (size_t)R;
      double wb = 0.0;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = 4 * s + g;
        wb = fma(fq[s], (double)pm[r < R ? r : R - 1], wb);       // fq is 0 past R
      }
      for (int r = 16 + g; r < R; r += 4) wb = fma((double)phi_q[r], (double)pm[r], wb);
      wb += __shfl_xor(wb, 16);
      wb += __shfl_xor(wb, 32);
      rescale(wb > 0.0 ? fmax(0.0, (double)(__builtin_amdgcn_frexp_exp(wb) - 1) - m) : 0.0);
      // Pairs before `lo` were discarded before every query of this wave (the first Nh are left out of the prefix
      // states): their share of Eq. 3 is phi(q) hpre 2^-m in the numerator, on fp32 matrix tiles in the layout
      // of p V, and phi(q) zpre 2^-m in the denominator.
      if (lo > mk.Nh) {
        const int kb = lo / kPrefixKeys, nkb = P / kPrefixKeys + 1, mi = -(int)m;
        const float *hk = mk.hpre + (ukv * (size_t)nkb + kb) * R * D + 4 * DB * (c / 4) + c % 4;
        const float *zk = mk.zpre + (ukv * (size_t)nkb + kb) * R;
        // one step = features 4 s + g: f the lane's phi entry (0 past R), rc its clamped row
        auto prefix_step = [&](double f, int rc) __attribute__((always_inline)) {
          f = __builtin_ldexp(f, mi);
          Lw = fma(f, (double)zk[rc], Lw);
          if constexpr (OUT) {
            const float bf = (float)f;
#pragma unroll
            for (int b = 0; b < DB; ++b) O[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(hk[(size_t)rc * D + 4 * b], bf, O[b], 0, 0, 0);
          }
        };
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (4 * s < R) prefix_step(fq[s], 4 * s + g < R ? 4 * s + g : R - 1);
        for (int s = 4; 4 * s < R; ++s) {
          const int r = 4 * s + g, rc = r < R ? r : R - 1;
          prefix_step(r < R ? (double)phi_q[rc] : 0.0, rc);
        }
      }
    }
    for (int i = 0; i < nlow; ++i) {
      lds_arrived<0>();
      lds_barrier();
      const int j0 = (lo_wg + i) * kRowKeys;
      if (i + 1 < nlow) load_tile(lo_wg + i + 1, k_next, v_next, false);
      if (discarded && j0 >= lo / kRowKeys * kRowKeys && j0 < q0 + 15 - mk.Nr) {    // wave-uniform
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          // psi(K) phi(Q)^T: result register v of v_mfma_f64_16x16x4 holds row g + 4 v, so matrix row i stands for key
          // 4 (i % 4) + i / 4
          const int kr = j0 + 16 * half + 4 * (c % 4) + c / 4;
          const float *prow = psi_u + (size_t)(kr < P ? kr : P - 1) * R;
          v4d wt = {0.0, 0.0, 0.0, 0.0};
          float x[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) x[s] = prow[4 * s + g < R ? 4 * s + g : R - 1];
#pragma unroll
          for (int s = 0; s < 4; ++s)
            if (4 * s < R) wt = __builtin_amdgcn_mfma_f64_16x16x4f64(4 * s + g < R ? (double)x[s] : 0.0, fq[s], wt, 0, 0, 0);
          for (int s = 4; 4 * s < R; ++s) {
            const int r = 4 * s + g;
            wt = __builtin_amdgcn_mfma_f64_16x16x4f64(r < R ? (double)prow[r] : 0.0, r < R ? (double)phi_q[r] : 0.0, wt, 0, 0, 0);
          }
          double e[4];
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int kj = j0 + 16 * half + 4 * g + w;
            e[w] = kj >= mk.Nh && kj < qi - mk.Nr ? __builtin_ldexp(wt[w], -(int)m) : 0.0;
          }
          Lw += (e[0] + e[1]) + (e[2] + e[3]);
          split(e, half);
        }
        add_values(v_cur, j0 + 16 <= lo, j0 + 16 > q0 + 14 - mk.Nr);
      }
      swap_buffers();
    }
  }
  double Ls = L;                                          // the exponentials alone
  L += Lw;
  L += __shfl_xor(L, 16);
  L += __shfl_xor(L, 32);
  if constexpr (MASKED) {
    Ls += __shfl_xor(Ls, 16);
    Ls += __shfl_xor(Ls, 32);
  }
  if (qi < P) {
    if (g == 0) lse[u * (size_t)P + qi] = fma(m, kLn2, log(MASKED && mk.sparse_den ? Ls : L));
    if constexpr (OUT) {
      // O[b][w] is output element 4 (DB g + b) + w: the lane's elements are one run of 4 DB halves
      const float inv = (float)(1.0 / L);
      __half run[4 * DB];
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int b = 0; b < DB; ++b) run[4 * b + w] = __float2half_rn(O[b][w] * inv);
      __half *orow = out + (u * (size_t)P + qi) * D + 4 * DB * g;
#pragma unroll
      for (int i = 0; i < 4 * DB / 8; ++i) reinterpret_cast<uint4 *>(orow)[i] = reinterpret_cast<const uint4 *>(run)[i];
    }
  }
}

template <int D>
static hipError_t launch_rows_t(const RowArgs &a, hipStream_t st)
{
  const unsigned tiles = (unsigned)((a.P + kRowKeys - 1) / kRowKeys);
  const unsigned ngrp = (unsigned)((a.P + 16 * kPrefillWaves - 1) / (16 * kPrefillWaves));
  // as many units at a time as the digits' part of the workspace holds, in shares of about the same size
  const size_t U = a.U, most = digit_units(U, a.P, D), shares = (U + most - 1) / most;
  size_t n = (U + shares - 1) / shares;
  if (most >= kXcds) n = (n + kXcds - 1) / kXcds * kXcds;
  unsigned char *digits = (unsigned char *)a.digits;
  unsigned *words = (unsigned *)(digits + most * tiles * RowTile<D>::kKeyBytes);
  for (size_t u = 0; u < U; u += n) {
    const unsigned nu = (unsigned)(U - u < n ? U - u : n);
    const size_t kv = u * a.P * D, q = kv * a.G, rows = u * a.G * a.P;
    const __half *K = (const __half *)a.K + kv;
    key_digits_kernel<D><<<nu * tiles, 128, 0, st>>>(K, tiles, a.P, digits, words, a.fill, u == 0 ? a.fill_count : 0);
    const unsigned grid = prefill_grid(nu * a.G, ngrp);
    const MaskedArgs mk = a.masked ? a.masked->from_unit(u, a.G, a.P, D) : MaskedArgs{};
#define LESSDEC_ROWS(OUT, MASKED, MAPS) rows_f16_kernel<D, OUT, MASKED, MAPS><<<grid + n_maps, 64 * kPrefillWaves, 0, st>>>(      \
      (const __half *)a.Q + q, K, (const __half *)a.V + kv, nu * a.G, a.G, a.P, digits, words, a.lse + rows, out, a.zero0 + u,      \
      a.zero1 + u, mk, n_maps ? *a.maps : MlpArgs{}, grid)
    __half *out = a.out != nullptr ? (__half *)a.out + q : nullptr;
    // (maps, of all keys, ride with the first share: they need nothing of its digits)
    const unsigned n_maps = a.maps && u == 0 ? mlp_psi_blocks(*a.maps, kPsiTiles) : 0;
    if (a.masked) {
      if (out != nullptr) LESSDEC_ROWS(true, true, false); else LESSDEC_ROWS(false, true, false);
    } else if (n_maps) {
      if (out != nullptr) LESSDEC_ROWS(true, false, true); else LESSDEC_ROWS(false, false, true);
    } else {
      if (out != nullptr) LESSDEC_ROWS(true, false, false); else LESSDEC_ROWS(false, false, false);
    }
#undef LESSDEC_ROWS
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Whether psi rides along: it needs nothing of the row pass and is bound by other instructions, so it fills what the longest
// sweeps leave idle, and a launch is saved; but it reads a head's weights again for every 64 rows, where a launch of its own keeps them
// in registers.  So it rides up to a number of workgroups of maps that grows with the sweeps' length, and that is smaller where the launch
// of its own has less to lose: narrower weights, and ranks whose blocks of eight features hold padding.  How many query heads share the
// unit makes no difference to that number.  Gain in percent of a whole prompt phase with psi riding along over psi in a launch of its own, by
// workgroups of 64 rows in a sweep; "|": the line.
//   D = 128, R' = 512, rank 8 and 16, 2048 + 256 a workgroup of the sweep:
//     1   2048 1.3 | 3072 -1.7, 4096 -2.8, 8192 -5.3            rank 16: 2048 2.1 | 2560 0.3, 3072 -1.5, 4096 -2.8
//     2   2048 2.7, 2560 0.1 | 3072 -0.7, 4096 -2.8             rank 16: 2048 3.0 | 4096 -1.9
//     4   2048 3.4, 3072 0.1 | 4096 -1.6, 8192 -3.5             rank 16: 2048 3.8, 3072 0.1 | 4096 -1.3
//     8   2048 7.8, 3072 3.7, 4096 1.1 | 6144 -0.6, 8192 -2.0   rank 16: 2048 7.6, 4096 1.4 | 8192 -2.4
//     16  2048 10.0, 4096 2.6, 6144 0.7 to 1.6 | 8192 -0.5, 12288 -2.2
//     32  2048 10.6, 4096 4.2, 8192 0.8, 10240 0.1 | 12288 -0.6        rank 16: 4096 4.5, 8192 0.7
//     64  8192 1.5 | 12288 -0.5          128  8192 0.6 | 12288 -1.0, 16384 0.2
//   others of D = 128, 1536 + 256 (R' = 256; rank 4; R' = 128):
//     1   | 2048 -1.6; -1.5; -0.6, 3072 -3.4; -4.5; -2.5        2   2048 0.0; -0.2; 0.9 | 2560 -2.6; -2.7
//     4   2048 2.1; 1.0; 2.4, 2560 0.0; -0.9; 1.0 | 3072 -1.8; -2.6; -0.6
//     8   2048 6.6; 5.5; 7.5 | 4096 0.0; -1.2; 1.6, 8192 -2.9; -4.8; -0.9
//     16  | 6144 0.6; -0.4, 10240 -1.3; -3.1                    32  2048 7.0; 10.5; 5.5, 8192 0.8; -0.1; 1.5 | 10240 -0.1; -0.7
//   D = 64, R' = 512, rank 8 and 16, 6144 + 512:
//     1   2048 5.7, 4096 1.6 | 8192 -0.4, 12288 -1.1 (rank 16: 8.0, 5.2 | 2.9)     4   2048 6.6, 8192 0.6 | 12288 -0.1
//     8   2048 10.8, 8192 2.0 | 12288 1.0                       32  8192 3.2, 12288 1.9
//   others of D = 64, 2560 + 512 (R' = 256; rank 4; R' = 128):
//     1   2048 3.2; 2.7; 2.1 | 4096 -1.4; -1.0; -1.5            4   2048 4.2; 4.7; 2.7, 4096 0.1; 0.5; -0.4 | 8192 -2.8; -2.4; -3.2
//     8   4096 3.8; 3.9; 3.9 | 8192 -0.8; -0.3; -0.6            16  8192 1.2 | 12288 -0.2      32  8192 2.4; 2.1; 2.7, 12288 2.2
// With 2, 4 and 8 query heads, D = 128: 4096 in sweeps of 32 2.5, 2.2, -; 2048 in sweeps of 8 5.3, 2.9, 1.9; 8192 in sweeps of 16 -0.2, 0.3.
// Other hidden widths, and few rows of a head, have no such form: riding is faster at every number with D = 128 (R' = 96, 320, 1024: 2.7 to
// 5.6 at 4096 and 8192, 1.1 to 3.0 at 16384 and 24576), with D = 64 up to 8192 (16384: R' = 96 -1.1, R' = 1024 -2.4).
bool rows_f16_take_maps(const MlpArgs &maps)
{
  const unsigned blocks = mlp_psi_blocks(maps, kPsiTiles);
  if (!mlp_weights_in_registers(maps)) return maps.D == 128 || blocks <= 8192;
  const unsigned sweep = (unsigned)((maps.rpu + 16 * kPrefillWaves - 1) / (16 * kPrefillWaves));
  const bool whole = maps.Rp > 384 && maps.R % 8 == 0;     // the widest weights, no padding among a block's features
  const unsigned most = maps.D == 128 ? (whole ? 2048 : 1536) + 256 * sweep : (whole ? 6144 : 2560) + 512 * sweep;
  const unsigned measured = maps.D == 128 ? 10240 : 12288;
  return blocks <= (most < measured ? most : measured);
}

hipError_t launch_rows_f16(const RowArgs &a, int D, hipStream_t st)
{
  return D == 128 ? launch_rows_t<128>(a, st) : launch_rows_t<64>(a, st);
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
// (Digits scaled per tile as in the row pass, nine products for sixteen, lose: <2, 8> 662 -> 732 us for 128 units x 8192
// tokens, where the branches for the lowest digits cost more than the products; <8, 4> spills.)
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
  // block of 16 digits [(kc, g)][key], the key's place turned by the block, so that the writes of one key meet different banks
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
  // Fewest of all: a tile to a workgroup, as long as that does not make more workgroups than the chip takes at once (a whole prompt
  // phase, <1, 8> against <2, 8>: 32 units x 500 tokens, 142 kept or in doubt, 93.7 against 97.8; 12 x 777, 210: 114.5 against
  // 118.7; 64 x 256, 82: 74.6 against 70.1; 32 x 777, 210: 133.7 against 130.5).
  if ((size_t)U * tiles <= 320) LESSDEC_COLUMNS(1, 8);
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
