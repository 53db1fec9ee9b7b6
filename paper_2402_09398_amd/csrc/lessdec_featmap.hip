// Generic feature-map kernel (Eq. 1, Eq. 2) for any shape and storage type, and the state
// reset.  Weights are stored output-major: W1 [R'][D], W2 [R][R'], W3 [R][R] per head.
#include "lessdec_common.h"
#include "lessdec_internal.h"

namespace lessdec {

typedef double v4d __attribute__((ext_vector_type(4)));

// =====================================================================================
// Feature maps, generic path: any R', R, either storage type, fp64 throughout, on the fp64 matrix
// cores (v_mfma_f64_16x16x4_f64; lane = 16 g + c: A[i][k] from lane i + 16 k, B[k][j] from lane
// j + 16 k, result register v of lane (g, c) is element [g + 4 v][c]).
//   x    : rows of D values; row (u * rpu + p) belongs to unit u = b * Hh + h
//   out  : [rows, R] as double (out_f64) or float
//   W3   : NULL for phi (Eq. 1), the R x R matrix for psi (Eq. 2)
// A block of four waves evaluates 16 rows that share a head, over one of `parts` parts of the hidden
// units.  Layer 1 is H1 = W1 X^T, a tile of 16 hidden units at a time, tiles dealt to the waves; lane group g
// supplies the D / 4 elements from g D / 4 on, so a lane's operands are one run of its row.  Register v of the
// activated tile is then directly the B operand of layer 2 (hidden units g + 4 v).  The waves' layer-2
// sums meet in the LDS in wave order.  With one part the block finishes the map; a decode step, which has few
// (head, 16 rows) pairs, spreads the hidden units over blocks that leave their sums (fp64) in the workspace, and
// the step's own kernel adds them (one query head per unit, ranks up to 16), or featmap_finish_kernel in part order.
// Bound by the chain of requests, fp64 matrix products (66 cycles each) and activations of a wave.
// 8 x 32 units, D = 128, R' = 512, fp32 storage: 9.7 us for both maps; 10.4 + 4.1 with the library's erfc in the activations and the
// finishing launch, which the step has taken over (11.5 + 4.8 with the weights of the second layer
// requested after the first's products, a branch around every activation and divisions ahead of the first request), against 82 with a hidden unit per
// thread on the vector units and a block per (head, 8 rows).
// =====================================================================================
constexpr int kFmWaves = 4;

// gelu, the third matrix and the absolute value of one row's outputs: sum[r] -> f
template <typename T>
__device__ inline void featmap_store(const FeatmapArgs &a, int h, long row, int r, const double *h2)
{
  double f;
  if (a.W3 == nullptr) {
    f = fabs(h2[r]);
  } else {
    const T *W3 = reinterpret_cast<const T *>(a.W3) + ((size_t)h * a.R + r) * a.R;
    double s = 0.0;
#pragma unroll 8
    for (int j = 0; j < a.R; ++j) s = fma(h2[j], (double)Store<T>::to_float(W3[j]), s);
    f = fabs(s);
  }
  const size_t at = (size_t)row * a.R + r;
  if (a.out_f64) reinterpret_cast<double *>(a.out)[at] = f;
  else reinterpret_cast<float *>(a.out)[at] = (float)f;
}

// sums: [rows of a][parts][R], then b's; not used with one part.  grid = (blocks of a + blocks of b), block b of
// a map = ((chunk * parts) + part) * Hh + head
template <typename T, int D, int RT>
__global__ __launch_bounds__(64 * kFmWaves) void featmap_generic_kernel(const FeatmapArgs a_, const FeatmapArgs b_,
                                                                        unsigned na, int parts, double *__restrict__ sums)
{
  constexpr int CH = D / 4, EPV = Store<T>::kPerVec, NV = CH / EPV;
  __shared__ double s_red[kFmWaves][16][17];               // a wave's sums of 16 outputs x 16 rows
  __shared__ double s_h2[16][LESSDEC_MAX_RANK + 1];
  const bool first = blockIdx.x < na;
  const FeatmapArgs &a = first ? a_ : b_;
  const int Hh = a.Hh, Rp = a.Rp, R = a.R, rpu = a.rpu;
  unsigned bid = first ? blockIdx.x : blockIdx.x - na;
  const int h = (int)(bid % (unsigned)Hh);
  bid /= (unsigned)Hh;
  const int part = (int)(bid % (unsigned)parts);
  const long rows_head = (long)a.B * rpu, i0 = (long)(bid / (unsigned)parts) * 16;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64, g = l / 16, c = l % 16;
  auto global_row = [&](long i) -> long {                  // i-th row of this head -> row in x / out
    if (rpu == 1) return i * Hh + h;                       // (a decode step: without the division)
    const long b = i / rpu, p = i % rpu;
    return (b * Hh + h) * rpu + p;
  };
  typename Store<T>::Vec xr[NV];
  {
    const long i = i0 + c < rows_head ? i0 + c : rows_head - 1;          // padding: any row
    const T *x = reinterpret_cast<const T *>(a.x) + global_row(i) * D + g * CH;
#pragma unroll
    for (int k = 0; k < NV; ++k) xr[k] = load_vec<T>(x + k * EPV);
  }
  const T *W1 = reinterpret_cast<const T *>(a.W1) + (size_t)h * D * Rp;
  const T *W2 = reinterpret_cast<const T *>(a.W2) + (size_t)h * Rp * R;
  const int tiles = (Rp + 15) / 16, t0 = (int)((long)tiles * part / parts), t1 = (int)((long)tiles * (part + 1) / parts);
  v4d c2[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) c2[t] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int tile = t0 + wave; tile < t1; tile += kFmWaves) {
    const int hid = 16 * tile;
    const T *w1 = W1 + (size_t)(hid + c < Rp ? hid + c : Rp - 1) * D + g * CH;
    // all of the tile's weights are requested ahead of the products, the second layer's behind the first's
    typename Store<T>::Vec w[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) w[k] = load_vec<T>(w1 + k * EPV);
    T w2[4][RT];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int r = 16 * t + c, j = hid + g + 4 * v;
        w2[v][t] = W2[(size_t)(r < R ? r : R - 1) * Rp + (j < Rp ? j : Rp - 1)];
      }
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
      for (int e = 0; e < EPV; ++e)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Store<T>::get(w[k], e), (double)Store<T>::get(xr[k], e), acc, 0, 0, 0);
    double act[4];                                         // (four chains side by side: no branch around one)
#pragma unroll
    for (int v = 0; v < 4; ++v) act[v] = gelu_f64(acc[v]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = hid + g + 4 * v;
      if (j >= Rp) act[v] = 0.0;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        // (past the last unit a zero on both sides: the weight read in its place may be an infinity)
        c2[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(j < Rp ? (double)Store<T>::to_float(w2[v][t]) : 0.0, act[v], c2[t], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (t > 0) __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) s_red[wave][g + 4 * v][c] = c2[t][v];
    __syncthreads();
    const int r = tid % 16, row = tid / 16;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kFmWaves; ++w) sum += s_red[w][r][row];
    if (16 * t + r < R) {
      if (parts == 1) {
        s_h2[row][16 * t + r] = gelu_f64(sum);
      } else if (i0 + row < rows_head) {
        const size_t at = (first ? 0 : (size_t)a_.B * a_.Hh * a_.rpu) + (size_t)global_row(i0 + row);
        sums[(at * parts + part) * R + 16 * t + r] = sum;
      }
    }
  }
  if (parts > 1) return;
  __syncthreads();
  for (int o = tid; o < 16 * R; o += 64 * kFmWaves) {
    const int row = o / R, r = o % R;
    if (i0 + row >= rows_head) break;
    featmap_store<T>(a, h, global_row(i0 + row), r, s_h2[row]);
  }
}

// The parts' sums of a decode step's rows (rpu = 1) added in part order, and the rest of the maps.  A wave per row,
// a lane per output.  grid = ceil((rows of a + rows of b) / 4), block = 256.
template <typename T>
__global__ __launch_bounds__(256) void featmap_finish_kernel(const FeatmapArgs a_, const FeatmapArgs b_, int parts,
                                                             const double *__restrict__ sums)
{
  __shared__ double s_h2[4][LESSDEC_MAX_RANK];
  const long na = (long)a_.B * a_.Hh, nb = (long)b_.B * b_.Hh;
  const int wave = threadIdx.x / 64, r = threadIdx.x % 64, R = a_.R;
  const long i = (long)blockIdx.x * 4 + wave;
  const bool live = i < na + nb && r < R;
  if (live) {
    double sum = 0.0;
#pragma unroll 8
    for (int p = 0; p < parts; ++p) sum += sums[((size_t)i * parts + p) * R + r];
    s_h2[wave][r] = gelu_f64(sum);
  }
  __syncthreads();
  if (!live) return;
  if (i < na) featmap_store<T>(a_, (int)(i % a_.Hh), i, r, s_h2[wave]);
  else featmap_store<T>(b_, (int)((i - na) % b_.Hh), i - na, r, s_h2[wave]);
}

template <typename T, int D>
static void featmap_launch(const FeatmapArgs &a, const FeatmapArgs &b, bool both, int parts, double *sums, hipStream_t st)
{
  auto blocks = [&](const FeatmapArgs &x) { return (unsigned)(x.Hh * parts * (((long)x.B * x.rpu + 15) / 16)); };
  const unsigned na = blocks(a), grid = na + (both ? blocks(b) : 0u);
  if (a.R <= 16) featmap_generic_kernel<T, D, 1><<<grid, 64 * kFmWaves, 0, st>>>(a, b, na, parts, sums);
  else featmap_generic_kernel<T, D, LESSDEC_MAX_RANK / 16><<<grid, 64 * kFmWaves, 0, st>>>(a, b, na, parts, sums);
}
static void featmap_launch(const FeatmapArgs &a, const FeatmapArgs &b, bool both, int dtype, int parts, double *sums,
                           hipStream_t st)
{
  if (dtype == LESSDEC_DTYPE_F16) {
    if (a.D == 128) featmap_launch<__half, 128>(a, b, both, parts, sums, st);
    else featmap_launch<__half, 64>(a, b, both, parts, sums, st);
  } else {
    if (a.D == 128) featmap_launch<float, 128>(a, b, both, parts, sums, st);
    else featmap_launch<float, 64>(a, b, both, parts, sums, st);
  }
}

hipError_t launch_featmap_generic(const FeatmapArgs &a, int dtype, hipStream_t st)
{
  featmap_launch(a, a, false, dtype, 1, nullptr, st);
  return hipGetLastError();
}

int featmap_step_parts(int B, int heads, int Rp, int R, size_t bytes)
{
  // Parts of 64 hidden units (a tile per wave) as far as their sums fit the scratch and until there are 512 blocks.
  const size_t per = (size_t)B * heads * R * sizeof(double);
  const long chunks = (long)heads * ((B + 15) / 16);
  long parts = (Rp + 63) / 64;
  if (parts > (long)(bytes / per)) parts = (long)(bytes / per);
  if (parts > (512 + chunks - 1) / chunks) parts = (512 + chunks - 1) / chunks;
  return (int)parts;
}

hipError_t launch_featmap_step(const FeatmapArgs &a, const FeatmapArgs &b, int dtype, double *sums, size_t bytes, bool finish,
                               hipStream_t st)
{
  const size_t rows = (size_t)a.B * (a.Hh + b.Hh);
  const int parts = featmap_step_parts(a.B, a.Hh + b.Hh, a.Rp, a.R, bytes);
  hipError_t e;
  if (parts < 2) {                                         // a launch per map
    if ((e = launch_featmap_generic(a, dtype, st)) != hipSuccess) return e;
    return launch_featmap_generic(b, dtype, st);
  }
  featmap_launch(a, b, true, dtype, parts, sums, st);
  if ((e = hipGetLastError()) != hipSuccess || !finish) return e;
  const unsigned grid = (unsigned)((rows + 3) / 4);
  if (dtype == LESSDEC_DTYPE_F16) featmap_finish_kernel<__half><<<grid, 256, 0, st>>>(a, b, parts, sums);
  else featmap_finish_kernel<float><<<grid, 256, 0, st>>>(a, b, parts, sums);
  return hipGetLastError();
}

// =====================================================================================
// Reset: H = 0, z = 0, acc = 0, psi = 0, pos = -1, n_seen = 0, nothing pending (a fill kernel,
// so the call can be recorded into a HIP graph).
// =====================================================================================
__global__ void reset_kernel(float *H, size_t nH, double *z, size_t nz, double *acc, size_t nacc,
                             int32_t *pos, size_t npos, float *psi, size_t npsi, int32_t *n_seen,
                             int32_t *pend_slot, size_t nn)
{
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t i = t0; i < nH; i += stride) H[i] = 0.f;
  for (size_t i = t0; i < nz; i += stride) z[i] = 0.0;
  for (size_t i = t0; i < nacc; i += stride) acc[i] = 0.0;
  for (size_t i = t0; i < npos; i += stride) pos[i] = -1;
  for (size_t i = t0; i < npsi; i += stride) psi[i] = 0.f;
  for (size_t i = t0; i < nn; i += stride) {
    n_seen[i] = 0;
    pend_slot[i] = -1;
  }
}

hipError_t launch_reset(const lessdec_desc *d, hipStream_t st)
{
  const size_t U = (size_t)d->batch * d->heads, C = (size_t)d->n_heavy + d->n_recent;
  const size_t R = d->rank, D = d->head_dim;
  reset_kernel<<<1024, 256, 0, st>>>(d->H, U * R * D, d->z, U * R, d->acc, U * C, d->pos, U * C,
                                     d->psi, U * C * R, d->n_seen, d->pend_slot, U);
  return hipGetLastError();
}

}  // namespace lessdec
