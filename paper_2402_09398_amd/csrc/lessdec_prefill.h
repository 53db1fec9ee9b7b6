// What the prompt phase's kernel files share.
#pragma once

#include "lessdec_common.h"
#include "lessdec_internal.h"

namespace lessdec {

constexpr int kPrefillWaves = 4;   // waves per block of the prompt phase's passes
constexpr int kXcds = 8;           // workgroups go to the chip's 8 dies round-robin by index

// Workgroup -> (unit, group of tiles).  Causal sweeps have very different
// lengths, so every die gets the same sequence of groups: die x works through units x, x + 8,
// ..., each unit's groups in order.  The dies stay balanced and a unit's rows stay in one L2.
// grid = ceil(U / 8) * 8 * ngrp.
struct PrefillBlock { unsigned u; int grp; };
__device__ inline PrefillBlock prefill_block(unsigned b, int ngrp)
{
  const unsigned xcd = b % kXcds, r = b / kXcds;
  return PrefillBlock{(r / (unsigned)ngrp) * kXcds + xcd, (int)(r % (unsigned)ngrp)};
}
inline unsigned prefill_grid(unsigned U, unsigned ngrp) { return (U + kXcds - 1) / kXcds * kXcds * ngrp; }

// fp16 storage, scores from digit products (lessdec_rows.hip)
// Lambda-masking taken through the prompt: what the masked rows need besides
constexpr int kPrefixKeys = 64;
struct MaskedArgs {
  const float *phi, *psi;      // [U G, P, R], [U, P, R]
  const float *psimax;         // [U, R]
  const float *hpre, *zpre;    // [U, P / 64 + 1, R, D], [U, P / 64 + 1, R]
  int R, Nh, Nr, sparse_den;
  // first key that queries from q on meet one by one as a discarded pair: those before the last prefix state older than q's
  // window come with that state
  __host__ __device__ int first_low(int q) const
  {
    const int kb = q > Nr ? (q - Nr) / kPrefixKeys * kPrefixKeys : 0;
    return kb > Nh ? kb : Nh;
  }
  MaskedArgs from_unit(size_t u, int G, int P, int D) const
  {
    MaskedArgs m = *this;
    const size_t nkb = P / kPrefixKeys + 1;
    m.phi += u * G * P * R; m.psi += u * P * R; m.psimax += u * R;
    m.hpre += u * nkb * R * D; m.zpre += u * nkb * R;
    return m;
  }
};
struct RowArgs {
  const void *Q, *K, *V;
  unsigned U;
  int G, P;
  void *digits;              // digit_bytes(U, P, D)
  double *lse;
  void *out;                 // or NULL
  unsigned *zero0, *zero1;   // a word per unit that a later kernel takes a maximum into
  unsigned *fill;            // words to be set to kMlpEmpty
  size_t fill_count;
  const MaskedArgs *masked;  // or NULL: all causal pairs
  const MlpArgs *maps;       // psi of the keys in the same launch (rows_f16_take_maps), or NULL
};
bool rows_f16_take_maps(const MlpArgs &maps);
hipError_t launch_rows_f16(const RowArgs &a, int D, hipStream_t st);
// list == nullptr: every column
hipError_t launch_columns_f16(const void *Q, const void *K, unsigned U, int G, int P, int D, const double *lse,
                              const int32_t *list, const int32_t *count, int C, double *colsum, hipStream_t st);

}  // namespace lessdec
