// psi (Eq. 2), or phi (Eq. 1) when no third matrix is given, of many rows on the matrix cores:
// used by the prompt phase for every prompt key and by the multi-head decode step.
#include "lessdec_internal.h"
#include "lessdec_mlp.h"

namespace lessdec {

template <int D>
__global__ __launch_bounds__(256) void mlp_psi_kernel(const MlpArgs a)
{
  __shared__ __attribute__((aligned(16))) unsigned char s_lds[mlp_psi_lds(kPsiTiles)];
  mlp_psi_block<D, kPsiTiles>(a, blockIdx.x, s_lds);
}
// two maps in one launch (phi of the queries and psi of the keys of a multi-head decode step):
// the first na blocks work on a, the rest on b
template <int D>
__global__ __launch_bounds__(256) void mlp_pair_kernel(const MlpArgs a, const MlpArgs b, unsigned na)
{
  __shared__ __attribute__((aligned(16))) unsigned char s_lds[mlp_psi_lds(kPairTiles)];
  if (blockIdx.x < na) mlp_psi_block<D, kPairTiles>(a, blockIdx.x, s_lds);
  else mlp_psi_block<D, kPairTiles>(b, blockIdx.x - na, s_lds);
}

// Many rows per head (the prompt phase): a workgroup keeps its head's weights in registers and
// streams rows through them.  Wave w holds the groups of 32 hidden units w, w + 4, ... (NGW of
// them: R' = 128 NGW) for the whole kernel; per chunk of 16 rows it loads the rows and applies its
// groups; after two chunks the block adds the four layer-2 sums through the LDS and finishes the
// outputs as above (same arithmetic in the same order as mlp_psi_block: identical results).  The
// next chunk's rows are requested before the current chunk's arithmetic.
// Bound by vector instructions (15.5 per activation, one of them transcendental, where there were 17 and two) and the clock that
// the card lowers under them (2.1 GHz).  With one max, one mixed-precision fma per low half, one barrier per 32 rows in place of
// three per 16, and layer 1 of the next group issued between the activations of this one: 920 -> 756 us for 2048 units x 1024
// tokens, 460 -> 391 for 128 x 8192 (R' = 512, R = 8).  Then (808 and 418 on another card) an activation without a reciprocal, the
// finish without divisions and with W3's products requested together, and a row's unit found by a multiplication: 751 and 381.
// (With an activation of three instructions less, which is not as accurate: 676 and 343.  Four waves a SIMD, eight waves of two groups
// each, rows by DMA through the LDS, the polynomial's constants as literals, which makes a multiply-add 2.7 cycles there: 4 % fewer
// cycles at a clock 4 % lower, no gain.)
// grid = Hh * parts (head fastest), every block a contiguous share of the head's chunks.
template <int D, int NGW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void mlp_rows_kernel(const MlpArgs a,
                                                                                                  int parts, unsigned rpu_mul, int rpu_shift)
{
  __shared__ float s_red[2][4][16][32 + 1];                // [pair of chunks, in turn][wave][r][row]
  __shared__ double s_h2[32][17];                          // [row][r], each row written and read by one wave
  const int tid = threadIdx.x, wave = tid / 64, l = tid % 64, g = l / 16, c = l % 16;
  const int Hh = a.Hh, Rp = a.Rp, R = a.R;
  const int h = (int)blockIdx.x % Hh, part = (int)blockIdx.x / Hh;
  const __half *W1 = a.W1 + (size_t)h * Rp * D;
  const __half *W2 = a.W2 + (size_t)h * R * Rp;
  // 32-bit row arithmetic (the launcher checks that a head's rows fit) and a division by multiplication: rpu_mul = floor(2^(31 + s) /
  // rpu) + 1 with s = rpu_shift = ceil(log2 rpu) gives i / rpu = i rpu_mul 2^-(31 + s) for every i below 2^31
  const unsigned rows_head = (unsigned)a.B * (unsigned)a.rpu, rpu = (unsigned)a.rpu;
  const unsigned nchunk = (rows_head + 15) / 16;
  const unsigned ch0 = (unsigned)((unsigned long)nchunk * part / parts);
  const unsigned ch1 = (unsigned)((unsigned long)nchunk * (part + 1) / parts);
  auto global_row = [&](unsigned i) -> size_t {
    const unsigned bb = __umulhi(2 * i, rpu_mul) >> rpu_shift, p = i - bb * rpu;   // bb = i / rpu
    return ((size_t)bb * Hh + h) * rpu + p;
  };
  MlpTiles<D> w[NGW];
#pragma unroll
  for (int k = 0; k < NGW; ++k) w[k] = mlp_load_tiles<D>(W1, W2, Rp, R, 32 * (wave + 4 * k), g, c);
  __shared__ double s_w3[16][17];                          // W3 of the head, widened once; W3 == nullptr: phi (Eq. 1)
  {
    const int r = tid % 16, j = tid / 16;
    s_w3[r][j] = (a.W3 != nullptr && r < R && j < R) ? (double)__half2float(a.W3[((size_t)h * R + r) * R + j]) : 0.0;
  }
  // the lanes that finish a row: 8 where the outputs fit (all lanes have work for 32 rows), else 16
  const int nr = R <= 8 ? 8 : 16, r = tid % nr, row_first = tid / nr, row_step = 256 / nr;

  auto load_chunk = [&](unsigned ch, v8h (&bx)[D / 32]) {
    const unsigned i = ch * 16 + c;
    mlp_load_row<D>(a.x + (i < rows_head ? global_row(i) : 0) * D, g, bx);   // padding: any row
  };
  v8h bx_next[D / 32];
  if (ch0 < ch1) load_chunk(ch0, bx_next);
  for (unsigned ch = ch0; ch < ch1; ++ch) {
    v8h bx[D / 32];
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) bx[ks] = bx_next[ks];
    load_chunk(ch + 1 < ch1 ? ch + 1 : ch, bx_next);
    v4f c2 = {0.f, 0.f, 0.f, 0.f};
    // layer 1 of the next group beside the activations of this one
    v4f h0 = {0.f, 0.f, 0.f, 0.f}, h1 = {0.f, 0.f, 0.f, 0.f};
    mlp_hidden<D>(w[0], bx, h0, h1);
#pragma unroll
    for (int k = 0; k < NGW; ++k) {
      v4f n0 = {0.f, 0.f, 0.f, 0.f}, n1 = {0.f, 0.f, 0.f, 0.f};
      if (k + 1 < NGW) mlp_hidden<D>(w[k + 1], bx, n0, n1);
      v8h bhi, blo;
      mlp_activate(h0, h1, bhi, blo);
      c2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[k].a2, bhi, c2, 0, 0, 0);
      c2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[k].a2, blo, c2, 0, 0, 0);
      if (k + 1 < NGW) {
#pragma unroll
        for (int i = 0; i < 2 * (D / 32); ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 14, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      h0 = n0;
      h1 = n1;
    }
    const unsigned n = ch - ch0, half = n & 1;
    float(*red)[16][32 + 1] = s_red[(n / 2) & 1];
#pragma unroll
    for (int q = 0; q < 4; ++q) red[wave][4 * g + q][16 * half + c] = c2[q];
    if (!half && ch + 1 < ch1) continue;
    // one barrier per pair: a wave that reaches the next pair's barrier has read this pair's sums, and the pair
    // after that is the first to write over them
    __syncthreads();
    const unsigned rows_first = (ch - half) * 16;
    const int rows = half ? 32 : 16;
    for (int row = row_first; row < rows; row += row_step) {
      const float sum = ((red[0][r][row] + red[1][r][row]) + red[2][r][row]) + red[3][r][row];
      s_h2[row][r] = (r < R) ? gelu_poly_f64((double)sum) : 0.0;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int row = row_first; row < rows; row += row_step) {
      const unsigned i = rows_first + row;
      if (r < R && i < rows_head) {
        double acc3 = 0.0;
        if (a.W3 != nullptr) {
          // (eight at a time, all requested before the first is used; past R both are zero)
          for (int j = 0; j < nr; j += 8)
#pragma unroll
            for (int i = 0; i < 8; ++i) acc3 = fma(s_h2[row][j + i], s_w3[r][j + i], acc3);
        } else {
          acc3 = s_h2[row][r];
        }
        a.out[(size_t)global_row(i) * R + r] = (float)fabs(acc3);
      }
    }
  }
}

// Decode step: both maps for every unit, by parts of 64 hidden units, one job of mlp_parts_job
// per block.
template <int D>
__global__ __launch_bounds__(256) void mlp_parts_kernel(const __half *q, const __half *k, const __half *Wq1,
                                                        const __half *Wk1, const __half *Wq2, const __half *Wk2,
                                                        int Hh, int rrp, int x_stride, int B, float *out)
{
  // Plain scalar arguments, the ones the loads need first: the launch can preload the first
  // sixteen dwords into registers (the compile flag asks for it),
  // which takes the argument fetch out of a kernel that is one chain of latencies.  rrp = R | R' << 8.
  __shared__ __attribute__((aligned(16))) unsigned char s_slabs[2 * mlp_slab_bytes(D)];
  mlp_parts_block<D, false>(q, k, Wq1, Wk1, Wq2, Wk2, Hh, rrp >> 8, rrp & 0xff, B, x_stride, out, (int)blockIdx.x,
                            s_slabs, (int)threadIdx.x / 64, (int)threadIdx.x % 64);
}

// Decode step with G query heads per key head: phi of every query row and psi of every key row by
// parts, one job of mlp_parts_gq_job per block.  hg = Hk | G << 16, rrp = R | R' << 8.
template <int D>
__global__ __launch_bounds__(256) void mlp_parts_gq_kernel(const __half *q, const __half *k, const __half *Wq1,
                                                           const __half *Wk1, const __half *Wq2, const __half *Wk2,
                                                           int hg, int rrp, int B, float *out)
{
  __shared__ __attribute__((aligned(16))) unsigned char s_slab[mlp_slab_bytes(D)];
  mlp_parts_gq_job<D, false>(q, k, Wq1, Wk1, Wq2, Wk2, hg & 0xffff, hg >> 16, rrp >> 8, rrp & 0xff, B, out,
                             (int)blockIdx.x, s_slab, (int)threadIdx.x / 64, (int)threadIdx.x % 64);
}

bool mlp_mfma_supported(int dtype, int D, int Rp, int R)
{
  return dtype == LESSDEC_DTYPE_F16 && (D == 64 || D == 128) && Rp % 32 == 0 && Rp >= 32 && R <= 16;
}

// many rows per head and R' = 128, 256, 384 or 512: weights stay in registers, rows stream through
bool mlp_weights_in_registers(const MlpArgs &a)
{
  const long rows_head = (long)a.B * a.rpu;
  return a.Rp % 128 == 0 && a.Rp <= 512 && rows_head > 63 * 16 && rows_head < (1L << 31) - 64;
}

hipError_t launch_mlp(const MlpArgs &a, hipStream_t st)
{
  if (mlp_weights_in_registers(a)) {
    const int ngw = a.Rp / 128;
    const long nchunk = ((long)a.B * a.rpu + 15) / 16;
    long parts = 1024 / a.Hh;                              // about four workgroups per compute unit
    if (parts < 1) parts = 1;
    if (parts > nchunk / 8) parts = nchunk / 8;            // at least 8 chunks behind every weight load
    const unsigned grid = (unsigned)(a.Hh * parts);
    int shift = 0;
    while ((1L << shift) < a.rpu) ++shift;
    const unsigned mul = (unsigned)((1UL << (31 + shift)) / (unsigned long)a.rpu + 1);
#define LESSDEC_MLP_ROWS(DD, NG) mlp_rows_kernel<DD, NG><<<grid, 256, 0, st>>>(a, (int)parts, mul, shift)
    if (a.D == 128) {
      if (ngw == 1) LESSDEC_MLP_ROWS(128, 1); else if (ngw == 2) LESSDEC_MLP_ROWS(128, 2);
      else if (ngw == 3) LESSDEC_MLP_ROWS(128, 3); else LESSDEC_MLP_ROWS(128, 4);
    } else {
      if (ngw == 1) LESSDEC_MLP_ROWS(64, 1); else if (ngw == 2) LESSDEC_MLP_ROWS(64, 2);
      else if (ngw == 3) LESSDEC_MLP_ROWS(64, 3); else LESSDEC_MLP_ROWS(64, 4);
    }
#undef LESSDEC_MLP_ROWS
    return hipGetLastError();
  }
  const unsigned grid = mlp_psi_blocks(a, kPsiTiles);
  if (a.D == 128) mlp_psi_kernel<128><<<grid, 256, 0, st>>>(a);
  else mlp_psi_kernel<64><<<grid, 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_mlp_pair(const MlpArgs &a, const MlpArgs &b, hipStream_t st)
{
  const unsigned na = mlp_psi_blocks(a, kPairTiles), nb = mlp_psi_blocks(b, kPairTiles);
  if (a.D == 128) mlp_pair_kernel<128><<<na + nb, 256, 0, st>>>(a, b, na);
  else mlp_pair_kernel<64><<<na + nb, 256, 0, st>>>(a, b, na);
  return hipGetLastError();
}

hipError_t launch_mlp_parts(const MlpPartsArgs &a, hipStream_t st)
{
  const unsigned grid = (unsigned)mlp_parts_blocks(a.Hh, a.Rp, a.B);
  const int rrp = a.R | (a.Rp << 8), xs = a.x_stride ? a.x_stride : a.D;
  if (a.D == 128)
    mlp_parts_kernel<128><<<grid, 256, 0, st>>>(a.q, a.k, a.Wq1, a.Wk1, a.Wq2, a.Wk2, a.Hh, rrp, xs, a.B, a.out);
  else
    mlp_parts_kernel<64><<<grid, 256, 0, st>>>(a.q, a.k, a.Wq1, a.Wk1, a.Wq2, a.Wk2, a.Hh, rrp, xs, a.B, a.out);
  return hipGetLastError();
}

// a.Hh: key heads; G query heads each (q rows [B, Hh, G, D], Wq per query head)
hipError_t launch_mlp_parts_gq(const MlpPartsArgs &a, int G, hipStream_t st)
{
  const unsigned grid = (unsigned)mlp_parts_gq_jobs(a.Hh, G, a.Rp, a.B);
  const int rrp = a.R | (a.Rp << 8), hg = a.Hh | (G << 16);
  if (a.D == 128)
    mlp_parts_gq_kernel<128><<<grid, 256, 0, st>>>(a.q, a.k, a.Wq1, a.Wk1, a.Wq2, a.Wk2, hg, rrp, a.B, a.out);
  else
    mlp_parts_gq_kernel<64><<<grid, 256, 0, st>>>(a.q, a.k, a.Wq1, a.Wk1, a.Wq2, a.Wk2, hg, rrp, a.B, a.out);
  return hipGetLastError();
}

}  // namespace lessdec
