// Prompt phase: regular causal attention (remark after Eq. 3), H2O scores of the prompt
// tokens (column sums of the attention matrix), one-shot cut to the budget, and the
// low-rank state of everything cut away (Eq. 6).
//
// The scores decide which tokens are kept, so Q K^T is needed to fp64 precision: with fp16 storage
// as integer products of digit planes (lessdec_rows.hip), with fp32 storage
// in fp64 on the matrix cores (v_mfma_f64_16x16x4_f64).  Operand layout of that instruction, wave64, lane = 16 * g + c:
//   A[i][k] is taken from lane i + 16 k, B[k][j] from lane j + 16 k,
//   result register v of lane (g, c) holds D[g + 4 v][c].
// Both passes compute transposed tiles S^T[key][query] = K Q^T, so a lane always owns one
// query column (c) and four keys (g + 4 v); a head row of D values is split into four
// contiguous chunks of D / 4, chunk g supplying the k index of the instruction.
#include <type_traits>

#include "lessdec_common.h"
#include "lessdec_internal.h"
#include "lessdec_lds.h"
#include "lessdec_prefill.h"

namespace lessdec {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <typename T, int D>
struct Chunk {
  static constexpr int CH = D / 4;                       // values per lane group
  static constexpr int EPV = Store<T>::kPerVec;
  static constexpr int NV = CH / EPV;                    // 16-byte loads per lane
  typename Store<T>::Vec v[NV];
  __device__ inline void load(const T *row, int g)
  {
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = load_vec<T>(row + g * CH + i * EPV);
  }
  __device__ inline double get(int s) const { return (double)Store<T>::get(v[s / EPV], s % EPV); }
};

// S^T tile: acc[v] = sum_d K[key g+4v][d] * Q[query c][d] of the lane's key chunk, already widened to fp64 by the
// caller, and its query chunk.
template <typename T, int D>
__device__ inline v4d tile_kq(const double (&kd)[D / 4], const Chunk<T, D> &qraw)
{
  v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < D / 4; ++s)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(kd[s], qraw.get(s), acc, 0, 0, 0);
  return acc;
}

// p V^T for one tile of 16 keys, fp32 storage: v_mfma_f32_16x16x4_f32, one key group per
// instruction (result register w of lane (g, c) holds D[4 g + w][c]); O[b][w] is output
// element d = 16 b + 4 g + w of query c.
template <int D>
__device__ inline void tile_pv(const float *Vu, int P, int j0, int g, int c, const double (&e)[4],
                               v4f (&O)[D / 16])
{
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int kj = j0 + g + 4 * v;
    const float *vrow = Vu + (size_t)(kj < P ? kj : P - 1) * D;
    const float pf = (float)e[v];
#pragma unroll
    for (int b = 0; b < D / 16; ++b)
      O[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(vrow[b * 16 + c], pf, O[b], 0, 0, 0);
  }
}
template <int D>
__device__ inline void store_out(float *orow, int g, const v4f (&O)[D / 16], float inv)
{
#pragma unroll
  for (int b = 0; b < D / 16; ++b)
#pragma unroll
    for (int w = 0; w < 4; ++w) orow[b * 16 + 4 * g + w] = O[b][w] * inv;
}

// -------------------------------------------------------------------------------------
// Row pass, fp32 storage (fp16: lessdec_rows.hip): one wave per block of 16 queries, kPrefillWaves consecutive query blocks per
// workgroup.  The workgroup sweeps the key tiles up to its last diagonal; every key tile is
// fetched and widened to fp64 once, by all 256 threads, into the LDS (two buffers, one
// barrier per tile) in the order the matrix instruction wants its operand, and each wave
// whose diagonal is not yet passed multiplies it with its own queries (kept in registers).
// A wave keeps the running row maximum m_i and sum L_i = sum_j e^{s_ij - m_i} (fp64) and, if
// an output is wanted, the flash-style running numerator in fp32, rescaled only in tiles
// where some row's maximum moved.  Leaves lse_i = m_i + ln L_i.
// LDS layout of a tile: lane (g, c) reads its operand values s = 2 i, 2 i + 1 (key row c,
// element g D/4 + s) as one 16-byte piece at index (4 i + g) 16 + c: conflict-free.
// -------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(64 * kPrefillWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void prefill_rowpass_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, unsigned U, int G, int P,
    double *__restrict__ lse, T *__restrict__ out)
{
  // U counts query rows here: unit u's G query heads are rows u G .. u G + G - 1 of Q, out and
  // lse, and attend over unit u's keys and values
  constexpr int CH = D / 4, DB = D / 16;
  constexpr int EPT = 16 * D / (64 * kPrefillWaves);      // tile elements widened per thread
  static_assert(EPT % 2 == 0 && CH % EPT == 0, "a thread's elements stay within one lane group");
  __shared__ double2 s_k[2][16 * D / 2];
  const int nblk = (P + 15) / 16;
  const int ngrp = (nblk + kPrefillWaves - 1) / kPrefillWaves;
  const PrefillBlock pb = prefill_block(blockIdx.x, ngrp);
  if (pb.u >= U) return;                                  // uniform over the workgroup
  const int grp = ngrp - 1 - pb.grp;                      // long rows first
  const size_t u = pb.u;
  const int l = threadIdx.x % 64, g = l / 16, c = l % 16;
  const int it = grp * kPrefillWaves + (int)(threadIdx.x / 64);
  const bool active = it < nblk;                          // wave-uniform
  const int it_last = (grp + 1) * kPrefillWaves - 1 < nblk - 1 ? (grp + 1) * kPrefillWaves - 1 : nblk - 1;
  const int qi = it * 16 + c;
  const int qrow = qi < P ? qi : P - 1;
  const size_t ukv = u / (unsigned)G;
  const T *Qu = Q + u * (size_t)P * D, *Ku = K + ukv * (size_t)P * D, *Vu = V + ukv * (size_t)P * D;
  const double scale = 1.0 / sqrt((double)D);

  double qd[CH];
  {
    Chunk<T, D> qraw;
    qraw.load(Qu + (size_t)qrow * D, g);
#pragma unroll
    for (int s = 0; s < CH; ++s) qd[s] = qraw.get(s);
  }
  double m_run = -__builtin_inf(), L = 0.0;
  v4f O[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) O[b] = v4f{0.f, 0.f, 0.f, 0.f};

  // this thread's share of a key tile: EPT consecutive elements of row wc
  const int wc = threadIdx.x % 16, we = EPT * (int)(threadIdx.x / 16);
  const int wg = we / CH, wi = (we % CH) / 2;             // lane group and first piece of those elements
  T raw[EPT];
  auto fetch = [&](int jt) {
    const int kr = jt * 16 + wc;
    const T *src = Ku + (size_t)(kr < P ? kr : P - 1) * D + we;
    if constexpr (EPT * sizeof(T) == 32) {
      reinterpret_cast<uint4 *>(raw)[0] = reinterpret_cast<const uint4 *>(src)[0];
      reinterpret_cast<uint4 *>(raw)[1] = reinterpret_cast<const uint4 *>(src)[1];
    } else {
      reinterpret_cast<uint4 *>(raw)[0] = reinterpret_cast<const uint4 *>(src)[0];
    }
  };
  fetch(0);
  for (int jt = 0; jt <= it_last; ++jt) {
    const int j0 = jt * 16;
    double2 *buf = s_k[jt & 1];
#pragma unroll
    for (int p = 0; p < EPT / 2; ++p)
      buf[((wi + p) * 4 + wg) * 16 + wc] =
          double2{(double)Store<T>::to_float(raw[2 * p]), (double)Store<T>::to_float(raw[2 * p + 1])};
    fetch(jt < it_last ? jt + 1 : jt);
    // tile jt is complete, and nobody still reads the buffer that tile jt + 1 will go into
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    if (!active || jt > it) continue;                     // wave-uniform
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < CH / 2; ++i) {
      const double2 kk = buf[(i * 4 + g) * 16 + c];
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(kk.x, qd[2 * i], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(kk.y, qd[2 * i + 1], acc, 0, 0, 0);
    }
    double s[4], tmax = -__builtin_inf();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int kj = j0 + g + 4 * v;
      s[v] = (kj <= qi && kj < P) ? acc[v] * scale : -__builtin_inf();
      tmax = fmax(tmax, s[v]);
    }
    tmax = fmax(tmax, __shfl_xor(tmax, 16));
    tmax = fmax(tmax, __shfl_xor(tmax, 32));
    // key j0 <= qi always holds for jt <= it, so tmax is finite for every query with qi >= j0;
    // queries past the prompt end (qi >= P) still see key j0 < P.
    if (__any(tmax > m_run)) {
      const double m_new = fmax(m_run, tmax);
      const double alpha = exp(m_run - m_new);            // 1 where the maximum stayed
      L *= alpha;
      m_run = m_new;
      if (out != nullptr) {
        const float af = (float)alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b) O[b] *= af;
      }
    }
    double e[4], esum = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      e[v] = exp_softmax_f64(s[v] - m_run);
      esum += e[v];
    }
    L += esum;
    if (out != nullptr) {
      tile_pv<D>(reinterpret_cast<const float *>(Vu), P, j0, g, c, e, O);
    }
  }
  L += __shfl_xor(L, 16);
  L += __shfl_xor(L, 32);
  if (active && qi < P) {
    if (g == 0) lse[u * (size_t)P + qi] = m_run + log(L);
    if (out != nullptr) store_out<D>(out + (u * (size_t)P + qi) * D, g, O, (float)(1.0 / L));
  }
}

// -------------------------------------------------------------------------------------
// Feature-wise maximum of psi over a unit's prompt keys: psimax[u][r] = max_j psi_all[u][j][r].
// The values are >= 0 (Eq. 2 ends in an absolute value), so they order like their bit patterns
// and an integer LDS maximum does.  A thread keeps to one feature and 256 / R keys apart, eight of them in flight: bound
// by memory (an LDS maximum per value took 49 us for 320 units x 2048 tokens at rank 16).   grid = U, block = 256.
// -------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prefill_psimax_kernel(const float *__restrict__ psi_all, int P, int R,
                                                             float *__restrict__ psimax)
{
  __shared__ int s_max[LESSDEC_MAX_RANK];
  const size_t u = blockIdx.x;
  const int tid = threadIdx.x, rows = 256 / R, r = tid % R, first = tid / R;
  if (tid < R) s_max[tid] = 0;
  __syncthreads();
  if (first < rows) {
    const float *pa = psi_all + u * (size_t)P * R + r;
    int top = 0;
#pragma unroll 8
    for (int j = first; j < P; j += rows) top = max(top, __float_as_int(pa[(size_t)j * R]));
    atomicMax(&s_max[r], top);
  }
  __syncthreads();
  if (tid < R) psimax[u * R + tid] = __int_as_float(s_max[tid]);
}

// -------------------------------------------------------------------------------------
// Prefix states for the masked row pass: hpre[u][kb] = sum of psi(k_j)^T v_j and zpre[u][kb] =
// sum of psi(k_j) over the pairs Nh <= j < 64 kb (Eq. 6 restricted to a prefix), kb = 0 ..
// P / 64: what the low-rank part of Eq. 3 needs for a query whose discarded pairs reach at least
// to 64 kb.  fp32 sums (they only enter attention outputs and their normalisation, never a
// score; the state itself is built in fp64 by the finalize kernel).
// First every block of 64 keys by itself (a workgroup each, psi through the LDS; thread (d, rg)
// owns column d of rows rg, rg + 256 / D, ... of H, RC of them), its sum left where the prefix
// after it belongs; then a running sum over the blocks, a thread per entry.  One workgroup per unit walking all keys
// took 1010 us for 320 units x 2048 tokens at rank 16; 88 + 36 now.
// grid = U * (P / 64), block = 256;  scan: grid = U * ceil((R D + R) / 256), block = 256.
// -------------------------------------------------------------------------------------
template <typename T, int D, int RC>
__global__ __launch_bounds__(256) void prefill_prefix_kernel(const T *__restrict__ V,
                                                             const float *__restrict__ psi_all, int P, int R,
                                                             int Nh, float *__restrict__ hpre,
                                                             float *__restrict__ zpre)
{
  constexpr int NG = 256 / D;                               // row groups
  __shared__ float s_psi[kPrefixKeys][LESSDEC_MAX_RANK + 1];
  const int nblk = P / kPrefixKeys, kb = (int)(blockIdx.x % nblk), j0 = kb * kPrefixKeys;   // whole blocks only
  const size_t u = blockIdx.x / nblk;
  const int tid = threadIdx.x, d = tid % D, rg = tid / D;
  const T *Vu = V + (u * (size_t)P + j0) * D;
  const float *pa = psi_all + (u * (size_t)P + j0) * R;
  for (int i = tid; i < kPrefixKeys * R; i += 256) {
    const int jj = i / R, r = i % R;
    s_psi[jj][r] = j0 + jj >= Nh ? pa[i] : 0.f;             // the first Nh pairs are never discarded
  }
  __syncthreads();
  float acc[RC];
#pragma unroll
  for (int i = 0; i < RC; ++i) acc[i] = 0.f;
#pragma unroll 8
  for (int jj = 0; jj < kPrefixKeys; ++jj) {
    const float v = Store<T>::to_float(Vu[(size_t)jj * D + d]);
#pragma unroll
    for (int i = 0; i < RC; ++i) acc[i] = fmaf(s_psi[jj][(rg + NG * i) % (LESSDEC_MAX_RANK + 1)], v, acc[i]);
  }
  float *hu = hpre + (u * (nblk + 1) + kb + 1) * R * D;
#pragma unroll
  for (int i = 0; i < RC; ++i) {
    const int r = rg + NG * i;
    if (r < R) hu[(size_t)r * D + d] = acc[i];
  }
  if (tid < R) {
    float zacc = 0.f;
    for (int jj = 0; jj < kPrefixKeys; ++jj) zacc += s_psi[jj][tid];
    zpre[(u * (nblk + 1) + kb + 1) * R + tid] = zacc;
  }
}
__global__ __launch_bounds__(256) void prefill_prefix_scan_kernel(int nblk, int RD, int R, float *__restrict__ hpre,
                                                                  float *__restrict__ zpre)
{
  const int per = (RD + R + 255) / 256;
  const size_t u = blockIdx.x / per;
  const int e = (int)(blockIdx.x % per) * 256 + (int)threadIdx.x;
  if (e >= RD + R) return;
  const int stride = e < RD ? RD : R;
  float *p = e < RD ? hpre + u * (nblk + 1) * (size_t)RD + e : zpre + u * (nblk + 1) * (size_t)R + (e - RD);
  float run = 0.f;
  p[0] = 0.f;
#pragma unroll 8
  for (int kb = 1; kb <= nblk; ++kb) {
    run += p[(size_t)kb * stride];
    p[(size_t)kb * stride] = run;
  }
}

// -------------------------------------------------------------------------------------
// Masked row pass, fp32 storage (fp16: lessdec_rows.hip): Lambda-masking taken through the prompt token by token (Sec. 4, "Setup";
// Sec. 3.2 builds the same matrix for training), all rows at once.  Under that policy the cache
// that token t meets is known beforehand: the first Nh tokens and the Nr tokens before it, the
// pairs discarded by then are Nh .. t - Nr - 1.  Row t of the attention matrix therefore has
// e^{q_t k_j / sqrt(D)} where pair j is cached (or is t itself) and phi(q_t) psi(k_j)^T where
// it was discarded, and out_t = (row t) V / (row t) 1 is Eq. 3 with H, z of Eq. 6.
// Same tiling as the row pass.  A workgroup first sweeps the key tiles that can hold cached
// pairs of any of its queries (the first ceil(Nh / 16) tiles and those from the window of its
// first query on), staged through the LDS as there, all other entries masked out.  Then every
// wave sweeps, on its own, the tiles that hold pairs discarded before its queries: the 16 x 16
// tile psi(K) phi(Q)^T is R / 4 matrix instructions instead of D / 4, nothing is staged.
// Online normalisation as in the row pass, the low-rank entries entering as w e^{-m}; before the
// second sweep m rises to ln of an upper bound of the query's weights (phi(q) . max_j psi(k_j),
// psimax [U, R] from prefill_psimax_kernel), so every weight handed to p V stays in [0, 1].
// Leaves lse_t = m_t + ln(sum of the entries that H2O's scores are normalised by): all of them,
// or with the sparse-denominator flag the exponentials only.
// -------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(64 * kPrefillWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void prefill_maskedrows_kernel(
    const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ V, unsigned U, int G, int P,
    const MaskedArgs mk, double *__restrict__ lse, float *__restrict__ out)
{
  using T = float;
  const float *phi = mk.phi, *psi = mk.psi, *psimax = mk.psimax, *hpre = mk.hpre, *zpre = mk.zpre;
  const int R = mk.R, Nh = mk.Nh, Nr = mk.Nr, sparse_den = mk.sparse_den;
  constexpr int CH = D / 4, DB = D / 16;
  constexpr int EPT = 16 * D / (64 * kPrefillWaves);
  static_assert(EPT % 2 == 0 && CH % EPT == 0, "a thread's elements stay within one lane group");
  __shared__ double2 s_k[2][16 * D / 2];
  const int nblk = (P + 15) / 16;
  const int ngrp = (nblk + kPrefillWaves - 1) / kPrefillWaves;
  const PrefillBlock pb = prefill_block(blockIdx.x, ngrp);
  if (pb.u >= U) return;                                  // uniform over the workgroup
  const int grp = ngrp - 1 - pb.grp;                      // long rows first
  const size_t u = pb.u;
  const int l = threadIdx.x % 64, g = l / 16, c = l % 16;
  const int it = grp * kPrefillWaves + (int)(threadIdx.x / 64);
  const bool active = it < nblk;                          // wave-uniform
  const int it_last = (grp + 1) * kPrefillWaves - 1 < nblk - 1 ? (grp + 1) * kPrefillWaves - 1 : nblk - 1;
  const int qi = it * 16 + c;
  const int qrow = qi < P ? qi : P - 1;
  const size_t ukv = u / (unsigned)G;
  const T *Qu = Q + u * (size_t)P * D, *Ku = K + ukv * (size_t)P * D, *Vu = V + ukv * (size_t)P * D;
  const float *psi_u = psi + ukv * (size_t)P * R;
  const float *phi_q = phi + (u * (size_t)P + qrow) * R;
  const double scale = 1.0 / sqrt((double)D);

  // key tiles [0, nfirst) and [band0, it_last] can hold cached pairs of the workgroup's queries
  const int q0b = grp * kPrefillWaves * 16;
  int nfirst = (Nh + 15) / 16;
  if (nfirst > it_last + 1) nfirst = it_last + 1;
  int band0 = q0b - Nr >= 0 ? (q0b - Nr) / 16 : 0;
  if (band0 < nfirst) band0 = nfirst;
  if (band0 > it_last + 1) band0 = it_last + 1;
  const int ndense = nfirst + (it_last + 1 - band0);
  auto tile_of = [&](int idx) { return idx < nfirst ? idx : band0 + (idx - nfirst); };

  double qd[CH];
  {
    Chunk<T, D> qraw;
    qraw.load(Qu + (size_t)qrow * D, g);
#pragma unroll
    for (int s = 0; s < CH; ++s) qd[s] = qraw.get(s);
  }
  double m_run = -__builtin_inf(), L = 0.0;               // L: sum of the exponentials
  v4f O[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) O[b] = v4f{0.f, 0.f, 0.f, 0.f};

  // this thread's share of a key tile: EPT consecutive elements of row wc
  const int wc = threadIdx.x % 16, we = EPT * (int)(threadIdx.x / 16);
  const int wg = we / CH, wi = (we % CH) / 2;
  T raw[EPT];
  auto fetch = [&](int jt) {
    const int kr = jt * 16 + wc;
    const T *src = Ku + (size_t)(kr < P ? kr : P - 1) * D + we;
    reinterpret_cast<uint4 *>(raw)[0] = reinterpret_cast<const uint4 *>(src)[0];
    if constexpr (EPT == 8) reinterpret_cast<uint4 *>(raw)[1] = reinterpret_cast<const uint4 *>(src)[1];
  };
  // 1) the cached pairs: the row pass over the tiles that can hold any, other entries masked out
  if (ndense > 0) fetch(tile_of(0));
  for (int idx = 0; idx < ndense; ++idx) {
    const int jt = tile_of(idx), j0 = jt * 16;
    double2 *buf = s_k[idx & 1];
#pragma unroll
    for (int p = 0; p < EPT / 2; ++p)
      buf[((wi + p) * 4 + wg) * 16 + wc] =
          double2{(double)Store<T>::to_float(raw[2 * p]), (double)Store<T>::to_float(raw[2 * p + 1])};
    fetch(tile_of(idx + 1 < ndense ? idx + 1 : idx));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    // no cached pair of this wave's queries in the tile? (wave-uniform)
    if (!active || jt > it || (j0 >= Nh && j0 + 15 < it * 16 - Nr)) continue;
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < CH / 2; ++i) {
      const double2 kk = buf[(i * 4 + g) * 16 + c];
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(kk.x, qd[2 * i], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(kk.y, qd[2 * i + 1], acc, 0, 0, 0);
    }
    double sc[4], tmax = -__builtin_inf();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int kj = j0 + g + 4 * v;
      const bool cached = kj <= qi && kj < P && (kj < Nh || kj >= qi - Nr);
      sc[v] = cached ? acc[v] * scale : -__builtin_inf();
      tmax = fmax(tmax, sc[v]);
    }
    tmax = fmax(tmax, __shfl_xor(tmax, 16));
    tmax = fmax(tmax, __shfl_xor(tmax, 32));
    if (__any(tmax > m_run)) {
      const double m_new = fmax(m_run, tmax);
      const double alpha = m_new > m_run ? exp(m_run - m_new) : 1.0;   // 0 when nothing was summed before
      L *= alpha;
      m_run = m_new;
      if (out != nullptr) {
        const float af = (float)alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b) O[b] *= af;
      }
    }
    double e[4], esum = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      e[v] = sc[v] > -__builtin_inf() ? exp_softmax_f64(sc[v] - m_run) : 0.0;
      esum += e[v];
    }
    L += esum;
    if (out != nullptr) tile_pv<D>(Vu, P, j0, g, c, e, O);
  }

  // 2) the discarded pairs, every wave on its own: key tiles from Nh's tile to the last one that
  // holds a pair older than the window of the wave's last query.  The tile psi(K) phi(Q)^T is
  // R / 4 matrix instructions; entries of pairs that are cached for the lane's query are masked
  // out.  The next tile's psi operands are requested before this tile's arithmetic.
  double Lw = 0.0;                                         // sum of the low-rank entries, times e^{-m_run}
  int jt_lo = Nh / 16;
  const int jt_hi = (it * 16 + 14 - Nr) >= 0 ? (it * 16 + 14 - Nr) / 16 : -1;
  if (active && jt_lo <= jt_hi) {
    // m_run is finite for every query of the prompt: the diagonal tile held the query itself
    double em_run = m_run > -__builtin_inf() ? exp(-m_run) : 0.0;
    // phi of the lane's query: feature 4 s + g is this lane's operand of step s
    double fq[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r = 4 * s + g;
      const float x = phi_q[r < R ? r : R - 1];
      fq[s] = r < R ? (double)x : 0.0;
    }
    // No weight of this query can exceed wb = phi(q) . max_j psi(k_j) (all features are >= 0), so
    // m rises to ln(wb) once, here, and every w e^{-m} handed to p V below stays in [0, 1]
    // without the sweep tracking a maximum.
    {
      const float *pm = psimax + ukv * (size_t)R;
      double wb = 0.0;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = 4 * s + g;
        wb = fma(fq[s], (double)pm[r < R ? r : R - 1], wb);  // fq is 0 past R
      }
      for (int r = 16 + g; r < R; r += 4) wb = fma((double)phi_q[r], (double)pm[r], wb);
      wb += __shfl_xor(wb, 16);
      wb += __shfl_xor(wb, 32);
      const double m_new = wb > 0.0 ? fmax(m_run, log(wb)) : m_run;
      if (m_new > m_run) {
        const double alpha = exp(m_run - m_new);
        L *= alpha;
        m_run = m_new;
        em_run = exp(-m_new);
        if (out != nullptr) {
          const float af = (float)alpha;
#pragma unroll
          for (int b = 0; b < DB; ++b) O[b] *= af;
        }
      }
    }
    // Pairs before 64 kbq were discarded before every query of this wave (and the first Nh are
    // left out of the prefix states): their share of Eq. 3 is phi(q) hpre[kbq] e^{-m} in the
    // numerator, on fp32 matrix tiles in the output layout of p V, and phi(q) zpre[kbq] e^{-m} in
    // the denominator.  Only the tiles from 64 kbq on are swept entry by entry.
    const int kbq = it * 16 - Nr > 0 ? (it * 16 - Nr) / kPrefixKeys : 0;
    if (kbq * kPrefixKeys > Nh) {
      const int nkb = P / kPrefixKeys + 1;
      const float *hk = hpre + (ukv * (size_t)nkb + kbq) * R * D;
      const float *zk = zpre + (ukv * (size_t)nkb + kbq) * R;
      double zsum = 0.0;
      // one step = features 4 s + g: f the lane's phi entry (0 past R), rc its clamped row
      auto prefix_step = [&](double f, int rc) {
        zsum = fma(f, (double)zk[rc], zsum);
        if (out != nullptr) {
          const float bf = (float)(f * em_run);
#pragma unroll
          for (int b = 0; b < DB; ++b) {
            const float a = hk[(size_t)rc * D + 16 * b + c];
            O[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bf, O[b], 0, 0, 0);
          }
        }
      };
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (4 * s < R) prefix_step(fq[s], 4 * s + g < R ? 4 * s + g : R - 1);
      for (int s = 4; 4 * s < R; ++s) {
        const int r = 4 * s + g, rc = r < R ? r : R - 1;
        prefix_step(r < R ? (double)phi_q[rc] : 0.0, rc);
      }
      Lw += zsum * em_run;                                    // this lane group's features; the groups are added at the end
      if (jt_lo < kbq * (kPrefixKeys / 16)) jt_lo = kbq * (kPrefixKeys / 16);
    }
    auto psi_operands = [&](int j0, float (&a)[4]) {
      const int kr = j0 + c;                                  // a tile of the last, ragged query block can pass the prompt end
      const float *prow = psi_u + (size_t)(kr < P ? kr : P - 1) * R;
#pragma unroll
      for (int s = 0; s < 4; ++s) {                           // unconditional loads, features past R zeroed after
        const int r = 4 * s + g;
        const float x = prow[r < R ? r : R - 1];
        a[s] = r < R ? x : 0.f;
      }
    };
    float pa_next[4];
    psi_operands(jt_lo * 16, pa_next);
    for (int jt = jt_lo; jt <= jt_hi; ++jt) {
      const int j0 = jt * 16;
      float pa[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) pa[s] = pa_next[s];
      const int jn = jt < jt_hi ? j0 + 16 : j0;
      psi_operands(jn, pa_next);
      v4d wt = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (4 * s < R) wt = __builtin_amdgcn_mfma_f64_16x16x4f64((double)pa[s], fq[s], wt, 0, 0, 0);
      for (int s = 4; 4 * s < R; ++s) {
        const int r = 4 * s + g;
        const int kr = j0 + c < P ? j0 + c : P - 1;
        const double a = r < R ? (double)psi_u[(size_t)kr * R + r] : 0.0, b = r < R ? (double)phi_q[r] : 0.0;
        wt = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, wt, 0, 0, 0);
      }
      double e[4], wsum = 0.0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int kj = j0 + g + 4 * v;
        e[v] = (kj >= Nh && kj < qi - Nr) ? fmin(wt[v] * em_run, 1.0) : 0.0;
        wsum += e[v];
      }
      Lw += wsum;
      if (out != nullptr) tile_pv<D>(Vu, P, j0, g, c, e, O);
    }
  }
  double Ls = L;                                           // exponentials only
  L += Lw;
  L += __shfl_xor(L, 16);
  L += __shfl_xor(L, 32);
  Ls += __shfl_xor(Ls, 16);
  Ls += __shfl_xor(Ls, 32);
  if (active && qi < P) {
    if (g == 0) lse[u * (size_t)P + qi] = m_run + log(sparse_den ? Ls : L);
    if (out != nullptr) store_out<D>(out + (u * (size_t)P + qi) * D, g, O, (float)(1.0 / L));
  }
}

// -------------------------------------------------------------------------------------
// Column pass, fp32 storage (fp16: lessdec_rows.hip): one wave per block of 16 keys.  Sweeps the query tiles from the diagonal
// down and sums a_ij = e^{s_ij - lse_i} over the queries: the accumulated attention
// probability of each prompt token (H2O's score, Sec. 2.1).  No atomics: every column is
// owned by one wave and reduced in a fixed order.
// -------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(64 * kPrefillWaves) void prefill_colpass_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, unsigned U, int P,
    const double *__restrict__ lse, int G, double *__restrict__ colsum)
{
  constexpr int CH = D / 4;
  const int nblk = (P + 15) / 16;
  const int ngrp = (nblk + kPrefillWaves - 1) / kPrefillWaves;
  const PrefillBlock pb = prefill_block(blockIdx.x, ngrp);
  const int grp = pb.grp;                                 // early columns have the longest sweeps
  const size_t u = pb.u;
  const int l = threadIdx.x % 64, g = l / 16, c = l % 16;
  const int jt = grp * kPrefillWaves + (int)(threadIdx.x / 64);
  if (jt >= nblk || pb.u >= U) return;                    // wave-uniform; the waves share nothing
  const int j0 = jt * 16;
  const T *Ku = K + u * (size_t)P * D;
  const double scale = 1.0 / sqrt((double)D);

  double kd[CH];
  {
    Chunk<T, D> kraw;
    const int kr = j0 + c;
    kraw.load(Ku + (size_t)(kr < P ? kr : P - 1) * D, g);
#pragma unroll
    for (int s = 0; s < CH; ++s) kd[s] = kraw.get(s);
  }
  double cs[4] = {0.0, 0.0, 0.0, 0.0};
  for (int h = 0; h < G; ++h) {                           // the unit's query heads, one sweep each
  const T *Qu = Q + (u * G + h) * (size_t)P * D;
  const double *lse_u = lse + (u * G + h) * (size_t)P;
  Chunk<T, D> qraw;
  double lq;
  {
    const int qr = j0 + c < P ? j0 + c : P - 1;
    qraw.load(Qu + (size_t)qr * D, g);
    lq = lse_u[qr];
  }
  auto tile = [&](int it, const Chunk<T, D> &cur, double lcur, Chunk<T, D> &nxt, double &lnxt) {
    const int qi = it * 16 + c;
    {
      const int qn = (it + 1 < nblk ? qi + 16 : qi);
      const int qr = qn < P ? qn : P - 1;
      nxt.load(Qu + (size_t)qr * D, g);
      lnxt = lse_u[qr];
    }
    const v4d acc = tile_kq<T, D>(kd, cur);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double a = exp_softmax_f64(fma(acc[v], scale, -lcur));
      cs[v] += (qi < P && (j0 + g + 4 * v) <= qi) ? a : 0.0;
    }
  };
  Chunk<T, D> qother;
  double lother;
  for (int it = jt; it < nblk; it += 2) {
    tile(it, qraw, lq, qother, lother);
    if (it + 1 < nblk) tile(it + 1, qother, lother, qraw, lq);
  }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) cs[v] += __shfl_xor(cs[v], o);
    const int kj = j0 + g + 4 * v;
    if (c == 0 && kj < P) colsum[u * (size_t)P + kj] = cs[v];
  }
}

// -------------------------------------------------------------------------------------
// Cheap column sums, fp16 storage only: the same sweep as the column pass on
// v_mfma_f32_16x16x32_f16 with fp32 accumulation and the fast fp32 exponential.  Their only
// use is to tell which tokens can possibly matter for the selection (prefill_select_kernel);
// every value that decides or is stored comes from the exact pass over those tokens.
// Lane (g, c) supplies elements 32 ks + 8 g .. + 7 of key row c (A) and of query row c (B);
// result register w holds S^T[key 4 g + w][query c].
// On the way: the largest squared norms of a unit's query and key rows (qmax, kmax, as bits of
// floats >= 0, zeroed before), whose product bounds every score and with it the rounding error of these
// sums; a wave takes the query rows at its keys' positions.
// The four waves of a workgroup take 16 KT consecutive keys each (in registers) and sweep the same queries, 64
// at a time through the LDS, so that a query row crosses the L2 once per workgroup; the next query tile's
// products stand beside this one's exponentials.  The chunks go straight into the LDS, two ahead of their use: with one ahead,
// through registers, the sweep waited for memory wherever a chunk's work was shorter than a round trip, and the
// registers held it to two waves a SIMD (three now, for which the form of four key tiles and D = 128 keeps four registers in scratch
// memory, 20 bytes a lane; without them, at two waves, 729, 1445 and 615 us).  717 -> 582 us for 2048 units x 1024 tokens,
// 1334 -> 1270 for 128 x 8192, 601 -> 511 for 128 x 4 heads x 2048.  Bound by issue (an instruction in 83 % of the cycles: exponentials take
// two slots, a matrix instruction blocks about two) and by the clock that the card lowers meanwhile (2.1 GHz).
// -------------------------------------------------------------------------------------
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
constexpr int kApproxQueries = 64; // queries per chunk
template <int D, int KT>
__global__ __launch_bounds__(64 * kPrefillWaves) __attribute__((amdgpu_waves_per_eu(3, 3))) void prefill_colapprox_kernel(
    const __half *__restrict__ Q, const __half *__restrict__ K, unsigned U, int P,
    const double *__restrict__ lse, int G, float *__restrict__ approx, unsigned *__restrict__ qmax,
    unsigned *__restrict__ kmax)
{
  constexpr int KS = D / 32, QC = kApproxQueries, RB = 2 * D, CH = D / 8;    // bytes and 16-byte chunks of a row
  constexpr int LOADS = QC * RB / 1024 / kPrefillWaves + 1;             // a wave's loads per chunk of queries
  constexpr double kLog2e = 1.44269504088896340736;
  // rows as they are, their 16-byte chunks turned by the row: 16 rows' reads of the same piece meet every bank once
  __shared__ __attribute__((aligned(16))) unsigned char s_q[3][QC * RB];
  __shared__ __attribute__((aligned(16))) double s_l[3][QC];
  auto turned = [](unsigned row, unsigned chunk) { return chunk ^ (D == 128 ? row % 16 : row / 2 % 8); };
  const int nch = (P + QC - 1) / QC, nkb = (P + 16 * KT - 1) / (16 * KT);
  const int ngrp = (nkb + kPrefillWaves - 1) / kPrefillWaves;
  const PrefillBlock pb = prefill_block(blockIdx.x, ngrp);
  if (pb.u >= U) return;                                  // uniform over the workgroup
  const size_t u = pb.u;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64, g = l / 16, c = l % 16;
  const int jt0 = (pb.grp * kPrefillWaves + wave) * KT, j0 = jt0 * 16;  // the wave's keys; past the prompt: none
  const __half *Ku = K + u * (size_t)P * D;
  const float scale = (float)(kLog2e / sqrt((double)D));                // base-2 units: the exponential is one instruction
  v8h ka[KT][KS];
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    const int kr = j0 + 16 * t + c;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      ka[t][ks] = *reinterpret_cast<const v8h *>(Ku + (size_t)(kr < P ? kr : P - 1) * D + 32 * ks + 8 * g);
  }
  // step by step the chunks from that of the workgroup's first key on, head after head
  const int c0 = pb.grp * kPrefillWaves * KT * 16 / QC, per = nch - c0, steps = G * per;
  int h = 0, q0 = c0 * QC;                                // the chunk to load next
  auto load = [&](int buf) __attribute__((always_inline)) {
    const int last = P - 1 - q0;                          // rows past the prompt: the last one
    const size_t first = (u * G + h) * (size_t)P + q0;
    unsigned l = tid % 64;
    asm("" : "+v"(l));                                    // else the addresses stay in registers between the chunks
#pragma unroll
    for (int k = 0; k < LOADS - 1; ++k) {
      const int piece = wave * (LOADS - 1) + k, row = piece * (1024 / RB) + (int)(l / CH);
      const int from = (row < last ? row : last) * RB + (int)turned(row, l % CH) * 16;
      lds_load<16>(Q + first * D, QC * RB, from, s_q[buf] + piece * 1024);
    }
    const int row = wave * (QC / kPrefillWaves) + (int)(l / 2), from = (row < last ? row : last) * 8 + (int)(l % 2) * 4;
    if (l < 2 * (QC / kPrefillWaves))
      lds_load<4>(lse + first, QC * 8, from, reinterpret_cast<unsigned char *>(s_l[buf] + wave * (QC / kPrefillWaves)));
    if ((q0 += QC) >= P) {                                // the next head's first chunk
      q0 = c0 * QC;
      ++h;
    }
  };
  // squared norm of a row that lies over the four lane groups, the largest of the wave's rows into `to`
  auto norm2 = [&](const v8h (&row)[KS]) {
    typedef _Float16 v2h __attribute__((ext_vector_type(2)));
    float ss = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const v2h x = {row[ks][2 * i], row[ks][2 * i + 1]};
        ss = __builtin_amdgcn_fdot2(x, x, ss, false);
      }
    ss += __shfl_xor(ss, 16);
    return ss + __shfl_xor(ss, 32);
  };
  auto leave_max = [&](float mx, unsigned *to) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if (l == 0) atomicMax(to, __float_as_uint(mx));
  };
  load(0);
  if (steps > 1) load(1);
  float mk = 0.f, mq = 0.f, cs[KT][4];
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    mk = fmaxf(mk, norm2(ka[t]));
#pragma unroll
    for (int w = 0; w < 4; ++w) cs[t][w] = 0.f;
  }
  for (int i = 0, b = 0, qc = c0; i < steps; ++i, b = b < 2 ? b + 1 : 0, qc = qc + 1 < nch ? qc + 1 : c0) {
    if (i + 1 < steps) lds_arrived<LOADS>(); else lds_arrived<0>();
    lds_barrier();                                        // the chunk is complete, and nobody still reads the one before it
    if (i + 2 < steps) load(b ? b - 1 : 2);
    if (j0 >= P || qc * QC + QC - 1 < j0) continue;       // wave-uniform: every query before the wave's keys
    auto query_tile = [&](int qt, v8h (&qa)[KS], float &lq) __attribute__((always_inline)) {
      int c = l % 16;
      asm("" : "+v"(c));                                  // (as above)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        qa[ks] = *reinterpret_cast<const v8h *>(s_q[b] + (16 * qt + c) * RB + turned(c, 4 * ks + g) * 16);
      lq = (float)(s_l[b][16 * qt + c] * kLog2e);
    };
    auto products = [&](const v8h (&qa)[KS], v4f (&acc)[KT]) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < KT; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < KT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka[t][ks], qa[ks], acc[t], 0, 0, 0);
    };
    if (qc * QC >= j0 + 16 * KT && qc * QC + QC <= P) {   // wave-uniform: every query after every key
      // the products of a query tile stand beside the exponentials of the one before
      v8h qa[2][KS];
      v4f acc[2][KT];
      float lq[2];
      query_tile(0, qa[0], lq[0]);
      products(qa[0], acc[0]);
#pragma unroll
      for (int qt = 0; qt < QC / 16; ++qt) {
        if (qt + 1 < QC / 16) {
          query_tile(qt + 1, qa[(qt + 1) & 1], lq[(qt + 1) & 1]);
          products(qa[(qt + 1) & 1], acc[(qt + 1) & 1]);
        }
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
          for (int w = 0; w < 4; ++w) cs[t][w] += __builtin_amdgcn_exp2f(fmaf(acc[qt & 1][t][w], scale, -lq[qt & 1]));
      }
      continue;
    }
#pragma unroll 1
    for (int qt = 0; qt < QC / 16; ++qt) {
      const int it = qc * (QC / 16) + qt, qi = it * 16 + c;
      if (it < jt0 || it * 16 >= P) continue;             // wave-uniform
      v8h qa[KS];
      v4f acc[KT];
      float lq;
      query_tile(qt, qa, lq);
      if (it < jt0 + KT) mq = fmaxf(mq, norm2(qa));       // the query rows at the wave's own positions
      products(qa, acc);
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int kj = j0 + 16 * t + 4 * g + w;
          const float a = __builtin_amdgcn_exp2f(fmaf(acc[t][w], scale, -lq));
          cs[t][w] += (qi < P && kj <= qi) ? a : 0.f;
        }
    }
  }
  if (j0 >= P) return;
  leave_max(mk, kmax + u);
  leave_max(mq, qmax + u);
#pragma unroll
  for (int t = 0; t < KT; ++t)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) cs[t][w] += __shfl_xor(cs[t][w], o);
      const int kj = j0 + 16 * t + 4 * g + w;
      if (c == 0 && kj < P) approx[u * (size_t)P + kj] = cs[t][w];
    }
}

// -------------------------------------------------------------------------------------
// Which tokens can matter, from the cheap column sums.  A cheap sum a~ and the exact one a
// satisfy |a~ - a| <= eps a + tau with
//   eps = 2^-24 ((D + 6) M + 3 ln P + G P / 16 + 6),   M = the unit's score bound (above):
// D M for the fp32 accumulation of the D exact fp16 products of a score, 5 M + 3 ln P for the
// rounded log2(e) / sqrt(D), the row's log-sum rounded to fp32 (|lse| <= M + ln P) and the fused
// multiply-add (|s - lse| <= 2 M + ln P), twice over, 2
// for the exponential itself, G P / 16 + 4 for a lane's running sum and the four lane exchanges;
// tau = 2^-100 covers terms flushed to zero.  The band used is twice that, and at least kBand
// (at the benchmark shapes eps is a tenth of kBand; the band only grows for prompts with far
// larger queries and keys).  With every cheap value within the band of the exact one, a token
// is surely a heavy hitter if fewer than Nh others could possibly be larger, surely discarded
// if at least Nh others are surely larger, and in doubt otherwise.
// Both counts are compared with the rank of j among the candidates, and hi(a) = a (1 + band) + tau,
// lo(a) = a (1 - band) - tau grow with a, so two order statistics decide: "fewer than Nh others could be larger"
// is hi(the (Nh + 1)-th largest) < lo(a_j), "at least Nh others surely are" is lo(the Nh-th largest) > hi(a_j).
// The Nh-th largest comes from a radix selection over the bits of the values (three passes of 11, 11 and 10
// bits; a sum that is not a number ranks last and is itself kept), the next one from one more pass; up to 256
// candidates, both by counting.
// flag[j] = 1 kept for sure (heavy or recent), 0 discarded for sure, 2 in doubt.  list, count: the tokens
// whose exact column sum is wanted (flag != 0), ascending.  With Lambda-masking (lambda) the first Nh and
// the last Nr tokens are kept, nothing is in doubt and approx is not looked at.
// One block per unit.  Counting every pair of candidates took 350 us for 2048 units x 1024 tokens and 1450 us
// for 128 x 8192; 26 and 56 now, the list included.   grid = U, block = 256.  qmax: see the cheap pass; kmax shares
// the place of count.
// -------------------------------------------------------------------------------------
constexpr float kBand = 1.0f / 256.0f;
__host__ __device__ inline float colapprox_error_bound(float M, int D, int P, int G)
{
  return 5.9604645e-08f * ((float)(D + 6) * M + 3.f * logf((float)P) + (float)G * (float)P / 16.f + 6.f);
}
// exclusive sum over the threads of a block of W waves; total: the sum of all.  s_wave: W ints
template <int W>
__device__ inline int block_scan(int x, int *s_wave, int &total)
{
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  int v = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(v, o);
    if (lane >= o) v += y;
  }
  __syncthreads();                                        // the scan before is done with s_wave
  if (lane == 63) s_wave[wave] = v;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    before += w < wave ? s_wave[w] : 0;
    total += s_wave[w];
  }
  return before + v - x;
}
__global__ __launch_bounds__(256) void prefill_select_kernel(const float *__restrict__ approx,
                                                             const unsigned *__restrict__ qmax, int D, int G, int P,
                                                             int Nh, int Nr, int lambda, int32_t *__restrict__ flag,
                                                             int32_t *__restrict__ list, int32_t *__restrict__ count)
{
  constexpr int kBins = 2048, kPer = kBins / 256;
  __shared__ int s_hist[kBins];
  __shared__ int s_wave[4], s_bin, s_rank, s_more;
  __shared__ unsigned s_next;
  const size_t u = blockIdx.x;
  const int tid = threadIdx.x, ncand = P - Nr;
  const float *a = approx + u * (size_t)P;
  float t1 = -1.f, t2 = -1.f, band = 0.f;                 // the Nh-th and (Nh + 1)-th largest; -1: there is none
  const float tau = 7.8886091e-31f;                       // 2^-100
  if (!lambda) {
    // the largest score magnitude: max_i |q_i| max_j |k_j| / sqrt(D), rounded up a little: the squared
    // norms carry fp32 rounding themselves
    const float M = sqrtf(__uint_as_float(qmax[u])) * sqrtf(__uint_as_float((unsigned)count[u])) *
                    (float)(1.0 / sqrt((double)D)) * 1.001f;
    band = fmaxf(kBand, 2.f * colapprox_error_bound(M, D, P, G));
    if (ncand <= 256) {
      // a value per thread: its rank by counting (equal ones by position)
      float *s_val = reinterpret_cast<float *>(s_hist), *s_t = s_val + 256;
      const float x = tid < ncand ? a[tid] : -1.f;
      s_val[tid] = x;
      if (tid < 2) s_t[tid] = -1.f;
      __syncthreads();
      int above = 0;
      for (int j = 0; j < ncand; ++j) above += (s_val[j] > x || (s_val[j] == x && j < tid)) ? 1 : 0;
      if (x >= 0.f && above == Nh - 1) s_t[0] = x;
      if (x >= 0.f && above == Nh) s_t[1] = x;
      __syncthreads();
      t1 = s_t[0];
      t2 = s_t[1];
    } else {
      unsigned prefix = 0, mask = 0;                        // bits of the Nh-th largest known so far
      int rank = Nh;                                        // its rank among the values with those bits, from 1
      bool found = Nh > 0;
      for (int pass = 0; pass < 3 && found; ++pass) {
        const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0, bins = pass == 2 ? 1024 : kBins;
        for (int i = tid; i < kBins; i += 256) s_hist[i] = 0;
        if (tid == 0) s_bin = -1;
        __syncthreads();
        for (int j = tid; j < ncand; j += 256) {
          const unsigned x = __float_as_uint(a[j]);
          if (x <= 0x7f800000u && (x & mask) == prefix) atomicAdd(&s_hist[(x >> shift) & (bins - 1)], 1);
        }
        __syncthreads();
        // thread t takes the bins from the top down: kPer of them, above them the threads before
        int mine = 0, total;
#pragma unroll
        for (int i = 0; i < kPer; ++i) mine += s_hist[kBins - 1 - (tid * kPer + i)];
        int above = block_scan<4>(mine, s_wave, total);
        if (above < rank && above + mine >= rank) {
#pragma unroll
          for (int i = 0; i < kPer; ++i) {
            const int bin = kBins - 1 - (tid * kPer + i), n = s_hist[bin];
            if (above < rank && above + n >= rank) {
              s_bin = bin;
              s_rank = rank - above;
            }
            above += n;
          }
        }
        __syncthreads();
        found = s_bin >= 0;                                 // not: fewer than Nh values that are numbers
        if (found) {
          prefix |= (unsigned)s_bin << shift;
          mask |= (unsigned)(bins - 1) << shift;
          rank = s_rank;
        }
        __syncthreads();
      }
      // the next one: the same value if it is there once more, else the largest below it
      if (tid == 0) {
        s_more = 0;
        s_next = 0;
      }
      __syncthreads();
      if (found || Nh == 0) {
        int same = 0;
        unsigned next = 0;
        for (int j = tid; j < ncand; j += 256) {
          const unsigned x = __float_as_uint(a[j]);
          if (x > 0x7f800000u) continue;
          if (found && x == prefix) ++same;
          else if ((Nh == 0 || x < prefix) && x + 1u > next) next = x + 1u;   // + 1: 0 stands for none
        }
        if (same) atomicAdd(&s_more, same);
        if (next) atomicMax(&s_next, next);
        __syncthreads();
        if (found) t1 = __uint_as_float(prefix);
        if (found && s_more > rank) t2 = t1;
        else if (s_next) t2 = __uint_as_float(s_next - 1u);
      }
      __syncthreads();
    }
  }
  const float keep_above = t2 * (1.f + band) + tau, drop_below = t1 * (1.f - band) - tau;
  int32_t *f = flag + u * (size_t)P, *out = list + u * (size_t)P;
  auto flag_of = [&](int j) {
    if (j >= ncand) return 1;                             // recent
    if (lambda) return j < Nh ? 1 : 0;
    const float x = a[j], lo = x * (1.f - band) - tau, hi = x * (1.f + band) + tau;
    if (!(x == x) || keep_above < lo) return 1;
    return Nh == 0 || drop_below > hi ? 0 : 2;
  };
  const int chunk = (P + 255) / 256;
  const int j0 = tid * chunk < P ? tid * chunk : P, j1 = j0 + chunk < P ? j0 + chunk : P;
  int cnt = 0;
  for (int j = j0; j < j1; ++j) {
    const int x = flag_of(j);
    f[j] = x;
    cnt += x != 0 ? 1 : 0;
  }
  int total, base = block_scan<4>(cnt, s_wave, total);
  for (int j = j0; j < j1; ++j)
    if (flag_of(j) != 0) out[base++] = j;
  if (tid == 0) count[u] = total;
}

// -------------------------------------------------------------------------------------
// Exact column sums of listed tokens only, fp32 storage: the column pass with 16 listed keys per wave in
// place of 16 consecutive ones.  The sweep starts at the query tile of the wave's earliest
// key; a key takes part from its own position on.  The length of the list is only known on
// the device: a unit gets enough blocks for a list a little longer than the budget, and its
// waves loop should the list be longer.   grid = ceil(U / 8) * 8 * blocks_per_unit.
// -------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(64 * kPrefillWaves) void prefill_colexact_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, unsigned U, int P, const double *__restrict__ lse,
    const int32_t *__restrict__ list, const int32_t *__restrict__ count, int blocks_per_unit, int G,
    double *__restrict__ colsum)
{
  constexpr int CH = D / 4;
  const int nblk = (P + 15) / 16;
  const PrefillBlock pb = prefill_block(blockIdx.x, blocks_per_unit);
  const size_t u = pb.u;
  const int l = threadIdx.x % 64, g = l / 16, c = l % 16;
  if (pb.u >= U) return;
  const int n = count[u];
  const T *Ku = K + u * (size_t)P * D;
  const double scale = 1.0 / sqrt((double)D);
  // tiles of 16 listed keys, dealt to the unit's waves in turn (the list is ascending, so
  // the long sweeps come first); wave-uniform, the waves share nothing
  for (int lt = pb.grp * kPrefillWaves + (int)(threadIdx.x / 64); lt * 16 < n;
       lt += blocks_per_unit * kPrefillWaves) {
    const int32_t *li = list + u * (size_t)P + lt * 16;
    const int nk = n - lt * 16 < 16 ? n - lt * 16 : 16;   // listed keys of this tile
    double kd[CH];
    {
      Chunk<T, D> kraw;
      kraw.load(Ku + (size_t)li[c < nk ? c : 0] * D, g);
#pragma unroll
      for (int s = 0; s < CH; ++s) kd[s] = kraw.get(s);
    }
    int kjv[4];                                           // positions of the lane's four keys
#pragma unroll
    for (int v = 0; v < 4; ++v) kjv[v] = g + 4 * v < nk ? li[g + 4 * v] : INT_MAX;
    const int it0 = li[0] / 16;
    double cs[4] = {0.0, 0.0, 0.0, 0.0};
    for (int h = 0; h < G; ++h) {                         // the unit's query heads, one sweep each
    const T *Qu = Q + (u * G + h) * (size_t)P * D;
    const double *lse_u = lse + (u * G + h) * (size_t)P;
    Chunk<T, D> qraw;
    double lq;
    {
      const int qr = it0 * 16 + c < P ? it0 * 16 + c : P - 1;
      qraw.load(Qu + (size_t)qr * D, g);
      lq = lse_u[qr];
    }
    auto tile = [&](int it, const Chunk<T, D> &cur, double lcur, Chunk<T, D> &nxt, double &lnxt) {
      const int qi = it * 16 + c;
      {
        const int qn = (it + 1 < nblk ? qi + 16 : qi);
        const int qr = qn < P ? qn : P - 1;
        nxt.load(Qu + (size_t)qr * D, g);
        lnxt = lse_u[qr];
      }
      const v4d acc = tile_kq<T, D>(kd, cur);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double a = exp_softmax_f64(fma(acc[v], scale, -lcur));
        cs[v] += (qi < P && kjv[v] <= qi) ? a : 0.0;
      }
    };
    Chunk<T, D> qother;
    double lother;
    for (int it = it0; it < nblk; it += 2) {
      tile(it, qraw, lq, qother, lother);
      if (it + 1 < nblk) tile(it + 1, qother, lother, qraw, lq);
    }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) cs[v] += __shfl_xor(cs[v], o);
      if (c == 0 && kjv[v] != INT_MAX) colsum[u * (size_t)P + kjv[v]] = cs[v];
    }
  }
}

// -------------------------------------------------------------------------------------
// Settles the tokens in doubt with their exact column sums: the heavy set is the tokens kept
// for sure plus the best of those in doubt, by (column sum, position) as in the rank kernel.
// keep[j] = 1 / 0.   grid = U, block = 256.
// -------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prefill_refine_kernel(const double *__restrict__ colsum,
                                                             const int32_t *__restrict__ flag, int P, int Nh,
                                                             int Nr, int32_t *__restrict__ keep)
{
  constexpr int kCap = 1024;                    // tokens in doubt held in the LDS (a handful in practice)
  __shared__ int s_sure, s_nd;
  __shared__ int s_idx[kCap];
  __shared__ double s_val[kCap];
  const size_t u = blockIdx.x;
  const int tid = threadIdx.x;
  const double *cs = colsum + u * (size_t)P;
  const int32_t *f = flag + u * (size_t)P;
  int32_t *out = keep + u * (size_t)P;
  const int ncand = P - Nr;
  if (tid == 0) s_sure = s_nd = 0;
  __syncthreads();
  int mine = 0;
  for (int j = tid; j < P; j += 256) {
    const int fj = f[j];
    mine += (fj == 1 && j < ncand) ? 1 : 0;
    if (fj == 2) {
      const int k = atomicAdd(&s_nd, 1);
      if (k < kCap) {
        s_idx[k] = j;
        s_val[k] = cs[j];
      }
    }
    out[j] = fj == 1 ? 1 : 0;
  }
  if (mine) atomicAdd(&s_sure, mine);
  __syncthreads();
  const int need = Nh - s_sure;                 // heavy slots left for the tokens in doubt
  const int nd = s_nd;
  if (nd <= kCap) {
    for (int k = tid; k < nd; k += 256) {
      const double a = s_val[k];
      const int j = s_idx[k];
      int larger = 0;
      for (int i = 0; i < nd; ++i) larger += (s_val[i] > a || (s_val[i] == a && s_idx[i] > j)) ? 1 : 0;
      out[j] = larger < need ? 1 : 0;
    }
  } else {
    for (int j = tid; j < ncand; j += 256) {
      if (f[j] != 2) continue;
      const double a = cs[j];
      int larger = 0;
      for (int i = 0; i < ncand; ++i) {
        if (f[i] != 2) continue;
        const double b = cs[i];
        larger += (b > a || (b == a && i > j)) ? 1 : 0;
      }
      out[j] = larger < need ? 1 : 0;
    }
  }
}

// -------------------------------------------------------------------------------------
// Selection: the last Nr tokens are recent; among the others the Nh largest (column sum,
// position) pairs are heavy hitters; everything else is discarded.  Exact rank counting,
// no sort: token j is heavy iff fewer than Nh candidates are larger.  (Lambda-masking past the budget:
// prefill_select_kernel.)
// One thread per token: keep[j] = 1 / 0.   grid = U * ceil(P / 256), block = 256.
// -------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prefill_rank_kernel(const double *__restrict__ colsum, int P,
                                                           int Nh, int Nr, int32_t *__restrict__ keep_of)
{
  const int nb = (P + 255) / 256;
  const size_t u = blockIdx.x / nb;
  const int j = (int)(blockIdx.x % nb) * 256 + (int)threadIdx.x;
  if (j >= P) return;
  const double *cs = colsum + u * (size_t)P;
  const int C = Nh + Nr;
  const int ncand = P - Nr;                     // positions < P - Nr compete for the heavy slots
  int keep = 1;
  if (P > C && j < ncand) {
    const double a = cs[j];
    int larger = 0;
    for (int i = 0; i < ncand; ++i) {
      const double b = cs[i];
      larger += (b > a || (b == a && i > j)) ? 1 : 0;
    }
    keep = larger < Nh ? 1 : 0;
  }
  keep_of[u * (size_t)P + j] = keep;
}

// -------------------------------------------------------------------------------------
// State of the discarded pairs, H = sum psi(k)^T v and z = sum psi(k) (Eq. 6) in fp64, of a share of a unit's tokens.
// A wave takes 256 / D tokens at a time, D / 4 lanes per token with four columns each, in chunks of eight rows of H: a
// value of psi is widened once for four columns and a value of V once for eight rows, and z is one lane's work.  Four
// columns and not eight: with 64 sums a lane the registers allow two waves a SIMD, too few to cover the loads.
// A unit's tokens are cut into `shares`, a workgroup each, whose sums the finalize kernel adds in order (part); one
// share stores H and z itself.  The lane groups meet by a reduce-scatter over the rows of H, the waves in the LDS.
// keep: 1 / 0 (kept / discarded).   grid = U shares, block = 256.
// One workgroup of eight waves per unit with eight columns a lane, slots and cache in the same kernel, took 282 us for
// 2048 units x 1024 tokens, 211 for 128 x 8192, 200 for 320 x 2048 at rank 16, 22 for 32 x 777; this kernel and the next:
// 192 + 48 (the cache's rows: bound by memory), 104 + 33, 131 + 28, 7 + 9.  fp32, a whole prompt phase, one workgroup per unit as
// above and in shares: 12 units x 2000 tokens at rank 32 1267 and 1168 us, 32 x 777 466 and 436.
// -------------------------------------------------------------------------------------

// four stored elements, all zero unless mask is ~0, as doubles
__device__ inline void load_four(const __half *p, unsigned mask, double (&v)[4])
{
  const uint2 x = *reinterpret_cast<const uint2 *>(p);
  const unsigned w[2] = {x.x & mask, x.y & mask};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const __half2 h = __builtin_bit_cast(__half2, w[i]);
    v[2 * i] = (double)__low2float(h);
    v[2 * i + 1] = (double)__high2float(h);
  }
}
__device__ inline void load_four(const float *p, unsigned mask, double (&v)[4])
{
  const uint4 x = *reinterpret_cast<const uint4 *>(p);
  const unsigned w[4] = {x.x & mask, x.y & mask, x.z & mask, x.w & mask};
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = (double)__uint_as_float(w[i]);
}

constexpr int kStateWaves = 4;
template <typename T, int D>
__device__ inline void discarded_state(size_t u, int share, int shares, const T *__restrict__ V, int P,
                                       const int32_t *__restrict__ keep, const float *__restrict__ psi_all, int R,
                                       float *__restrict__ H, double *__restrict__ z, double *__restrict__ part)
{
  constexpr int W = kStateWaves, RC = 8, LPT = D / 4, TPW = 64 / LPT;   // lanes per token, tokens per wave at a time
  __shared__ double s_part[W][RC][D], s_z[W][RC];
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, dl = lane % LPT, tp = lane / LPT;
  const int lo = (int)((long)P * share / shares), hi = (int)((long)P * (share + 1) / shares);
  const T *Vu = V + u * (size_t)P * D;
  const int32_t *ku = keep + u * (size_t)P;
  const float *pa = psi_all + u * (size_t)P * R;
  const bool vec4 = R % 4 == 0;                            // psi rows readable as 16-byte vectors
  for (int r0 = 0; r0 < R; r0 += RC) {
    const int rn = R - r0 < RC ? R - r0 : RC;
    const int rz = r0 + (dl < rn ? dl : 0);                // the lane's row of z (lanes dl < rn)
    double h[RC][4], zs;
    // Kept tokens go through the same arithmetic with values and psi of z zeroed, so that no load stands under a
    // condition.  CLEAN: psi of kept tokens zeroed too; without it a kept token adds psi times zero, which is zero
    // unless its psi is not finite
    auto sweep = [&](auto clean) __attribute__((always_inline)) {
      zs = 0.0;
#pragma unroll
      for (int r = 0; r < RC; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) h[r][i] = 0.0;
#pragma unroll 4
      for (int j0 = lo + wave * TPW; j0 < hi; j0 += W * TPW) {
        const int j = j0 + tp < hi ? j0 + tp : hi - 1;
        const unsigned mask = (ku[j] == 0 && j0 + tp < hi) ? ~0u : 0u;   // ~0: discarded
        const float *pj = pa + (size_t)j * R + r0;
        float gj[RC];
        // rows past R repeat earlier ones; their sums are never stored
        if (vec4) {
#pragma unroll
          for (int r4 = 0; r4 < RC / 4; ++r4) {
            const float4 x = *reinterpret_cast<const float4 *>(pj + (4 * r4 < rn ? 4 * r4 : 0));
            gj[4 * r4] = x.x; gj[4 * r4 + 1] = x.y; gj[4 * r4 + 2] = x.z; gj[4 * r4 + 3] = x.w;
          }
        } else {
#pragma unroll
          for (int r = 0; r < RC; ++r) gj[r] = pj[r < rn ? r : 0];
        }
        if constexpr (clean.value) {
#pragma unroll
          for (int r = 0; r < RC; ++r) gj[r] = __uint_as_float(__float_as_uint(gj[r]) & mask);
        }
        const unsigned gz = __float_as_uint(pa[(size_t)j * R + rz]) & mask;
        double v[4];
        load_four(Vu + (size_t)j * D + 4 * dl, mask, v);
        zs += (double)__uint_as_float(gz);
#pragma unroll
        for (int r = 0; r < RC; ++r) {
          const double g = (double)gj[r];
#pragma unroll
          for (int i = 0; i < 4; ++i) h[r][i] = fma(g, v[i], h[r][i]);
        }
      }
    };
    sweep(std::false_type{});
    bool lost = false;                                     // such a psi shows in every column of its row
#pragma unroll
    for (int r = 0; r < RC; ++r) lost |= !(h[r][0] == h[r][0]);
    if (__any(lost)) sweep(std::true_type{});
    // the wave's token groups: a lane keeps half of its rows at each distance; row of h[k] is then row0 + k
    int row0 = 0;
    auto halve = [&](auto distance, auto rows) __attribute__((always_inline)) {
      constexpr int o = distance.value, n = rows.value;
      const bool up = lane & o;
#pragma unroll
      for (int k = 0; k < n; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double send = up ? h[k][i] : h[k + n][i], mine = up ? h[k + n][i] : h[k][i];
          h[k][i] = mine + __shfl_xor(send, o);
        }
      row0 += up ? n : 0;
      zs += __shfl_xor(zs, o);
    };
    halve(std::integral_constant<int, 32>{}, std::integral_constant<int, RC / 2>{});
    if constexpr (TPW == 4) halve(std::integral_constant<int, 16>{}, std::integral_constant<int, RC / 4>{});
    constexpr int KEEP = RC / TPW;                         // rows a lane ends with
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) s_part[wave][row0 + k][4 * dl + i] = h[k][i];
    if (tp == 0 && dl < RC) s_z[wave][dl] = zs;
    __syncthreads();
    double *pu = part + (u * shares + share) * (size_t)(R * D + R);
    for (int x = tid; x < rn * D; x += 64 * W) {
      const int r = x / D, d = x % D;
      double sum = s_part[0][r][d];
#pragma unroll
      for (int w = 1; w < W; ++w) sum += s_part[w][r][d];
      if (shares > 1) pu[(r0 + r) * D + d] = sum;
      else H[(u * R + r0 + r) * D + d] = (float)sum;
    }
    if (tid < rn) {
      double sum = s_z[0][tid];
#pragma unroll
      for (int w = 1; w < W; ++w) sum += s_z[w][tid];
      if (shares > 1) pu[R * D + r0 + tid] = sum;
      else z[u * R + r0 + tid] = sum;
    }
    if (r0 + RC < R) __syncthreads();                      // s_part, s_z are written again
  }
}
template <typename T, int D>
__global__ __launch_bounds__(64 * kStateWaves) void prefill_state_kernel(
    const T *__restrict__ V, int P, const int32_t *__restrict__ keep, const float *__restrict__ psi_all, int R, int shares,
    float *__restrict__ H, double *__restrict__ z, double *__restrict__ part)
{
  discarded_state<T, D>(blockIdx.x / (unsigned)shares, (int)(blockIdx.x % (unsigned)shares), shares, V, P, keep, psi_all, R, H, z, part);
}

// -------------------------------------------------------------------------------------
// Slots and cache: the kept tokens get slots in order (ring_nh >= 0: as in-place replacement leaves them) and their
// rows are gathered into the cache (acc = column sum, pos, psi), unused slots cleared; the shares of H and z (more than
// one; none: nothing was discarded, both are zero) are added up.  slot_of: 1 / 0 (kept / discarded).  STATE: the state
// too, in one share (short prompts of few units, where a launch costs more than it spreads).
// grid = U, block = 64 W, dynamic LDS = C ints.
// -------------------------------------------------------------------------------------
template <typename T, int D, int W, bool STATE>
__global__ __launch_bounds__(64 * W) void prefill_finalize_kernel(
    const T *__restrict__ K, const T *__restrict__ V, int P, const double *__restrict__ colsum,
    const int32_t *__restrict__ slot_of, const float *__restrict__ psi_all, int C, int R,
    T *__restrict__ k_cache, T *__restrict__ v_cache, double *__restrict__ acc,
    int32_t *__restrict__ pos, float *__restrict__ psi, float *__restrict__ H,
    double *__restrict__ z, int32_t *__restrict__ n_seen, int32_t *__restrict__ pend_slot, int ring_nh,
    const double *__restrict__ part, int shares)
{
  constexpr int THREADS = 64 * W;
  extern __shared__ int s_tok[];                           // [C] token held by each slot
  __shared__ int s_wave[W];
  const size_t u = blockIdx.x;
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  const T *Ku = K + u * (size_t)P * D, *Vu = V + u * (size_t)P * D;
  const int32_t *so = slot_of + u * (size_t)P;
  const float *pa = psi_all + u * (size_t)P * R;
  const int kept = P < C ? P : C;

  // 1) slot = number of kept tokens before j: per-thread contiguous chunk + the threads before
  {
    const int chunk = (P + THREADS - 1) / THREADS;
    const int lo = tid * chunk < P ? tid * chunk : P, hi = (lo + chunk < P) ? lo + chunk : P;
    int cnt = 0, total;
    for (int j = lo; j < hi; ++j) cnt += so[j];
    int base = block_scan<W>(cnt, s_wave, total);
    for (int j = lo; j < hi; ++j) {
      const int keep = so[j];
      // ring_nh >= 0: the slots as in-place replacement leaves them when the first ring_nh tokens
      // stay and the others pass through the remaining slots in turn (Sec. 3.2)
      const int slot = (ring_nh < 0 || j < ring_nh || P <= C || C <= ring_nh) ? base : ring_nh + (j - ring_nh) % (C - ring_nh);
      if (keep && slot < C) s_tok[slot] = j;
      base += keep;
    }
  }
  // 2) the shares of the state, in order
  if (!STATE && shares != 1) {
    const double *pu = part + u * shares * (size_t)(R * D + R);
    for (int x = tid; x < R * D + R; x += THREADS) {
      double sum = 0.0;
#pragma unroll 4
      for (int i = 0; i < shares; ++i) sum += pu[(size_t)i * (R * D + R) + x];
      if (x < R * D) H[u * R * D + x] = (float)sum;
      else z[u * R + x - R * D] = sum;
    }
  }
  __syncthreads();

  // 3) gather: rows moved as 16-byte vectors, 64 / kVecs slots per wave at a time
  constexpr int kVecs = D * (int)sizeof(T) / 16;           // per row: 8, 16 or 32
  constexpr int kSlotsPerWave = 64 / kVecs;
  for (int s = wave * kSlotsPerWave + lane / kVecs; s < C; s += W * kSlotsPerWave) {
    const size_t slot = u * C + s;
    const int i = lane % kVecs;
    if (s < kept) {
      const int j = s_tok[s];
      reinterpret_cast<uint4 *>(k_cache + slot * D)[i] = reinterpret_cast<const uint4 *>(Ku + (size_t)j * D)[i];
      reinterpret_cast<uint4 *>(v_cache + slot * D)[i] = reinterpret_cast<const uint4 *>(Vu + (size_t)j * D)[i];
      if (i == 0) {
        acc[slot] = colsum[u * (size_t)P + j];
        pos[slot] = j;
      }
      for (int r = i; r < R; r += kVecs) psi[slot * R + r] = pa[(size_t)j * R + r];
    } else {
      if (i == 0) {
        acc[slot] = 0.0;
        pos[slot] = -1;
      }
      for (int r = i; r < R; r += kVecs) psi[slot * R + r] = 0.f;
    }
  }
  if (tid == 0) {
    n_seen[u] = P;
    pend_slot[u] = -1;
  }
  if constexpr (STATE) {
    static_assert(W == kStateWaves, "one state block per workgroup");
    discarded_state<T, D>(u, 0, 1, V, P, slot_of, psi_all, R, H, z, nullptr);
  }
}

template <typename T, int D>
static hipError_t launch_prefill_t(const PrefillArgs &a, hipStream_t st)
{
  const lessdec_desc *d = a.d;
  const int P = a.P, C = d->n_heavy + d->n_recent;
  const unsigned U = (unsigned)d->batch * d->heads;
  const int G = d->q_per_kv > 1 ? d->q_per_kv : 1;          // query heads per unit
  const unsigned tiles = (unsigned)(((P + 15) / 16 + kPrefillWaves - 1) / kPrefillWaves);
  const unsigned grid = (U + kXcds - 1) / kXcds * kXcds * tiles;
  const bool lambda = (d->flags & LESSDEC_FLAG_LAMBDA) != 0;
  // the prompt taken token by token under Lambda-masking, all rows at once (needs P > C: inside
  // the budget nothing is discarded and the regular rows are the same)
  const bool masked = a.masked && lambda && P > C;
  const int ring_nh = masked ? d->n_heavy : -1;
  hipError_t e;
  MlpArgs fm;                                             // psi of every key on the matrix cores
  fm.B = d->batch; fm.Hh = d->heads; fm.rpu = P; fm.D = d->head_dim; fm.Rp = d->hidden; fm.R = d->rank;
  fm.x = (const __half *)a.K; fm.W1 = (const __half *)d->Wk1; fm.W2 = (const __half *)d->Wk2;
  fm.W3 = (const __half *)d->Wk3; fm.out = a.psi_all;
  const bool matrix_maps = mlp_mfma_supported(d->dtype, d->head_dim, d->hidden, d->rank);
  const bool maps_ride = matrix_maps && !masked && rows_f16_take_maps(fm);
  auto key_features = [&]() -> hipError_t {
    if (matrix_maps) return launch_mlp(fm, st);
    FeatmapArgs fa;
    fa.x = a.K; fa.W1 = d->Wk1; fa.W2 = d->Wk2; fa.W3 = d->Wk3; fa.out = a.psi_all; fa.out_f64 = 0;
    fa.B = d->batch; fa.Hh = d->heads; fa.rpu = P; fa.D = d->head_dim; fa.Rp = d->hidden; fa.R = d->rank;
    return launch_featmap_generic(fa, d->dtype, st);
  };
  // the key digits' kernel empties the exchange array on its way
  if (sizeof(T) != 2 && (e = launch_fill_empty(a.empty, a.empty_count, st)) != hipSuccess) return e;
  if (masked) {
    // psi of every prompt key, phi of every prompt query (Eq. 1, Eq. 2), then the masked rows
    if ((e = key_features()) != hipSuccess) return e;
    if (mlp_mfma_supported(d->dtype, d->head_dim, d->hidden, d->rank)) {
      MlpArgs fm;
      fm.B = d->batch; fm.Hh = d->heads * G; fm.rpu = P; fm.D = d->head_dim; fm.Rp = d->hidden; fm.R = d->rank;
      fm.x = (const __half *)a.Q; fm.W1 = (const __half *)d->Wq1; fm.W2 = (const __half *)d->Wq2;
      fm.W3 = nullptr; fm.out = a.phi_all;
      e = launch_mlp(fm, st);
    } else {
      FeatmapArgs fa;
      fa.x = a.Q; fa.W1 = d->Wq1; fa.W2 = d->Wq2; fa.W3 = nullptr; fa.out = a.phi_all; fa.out_f64 = 0;
      fa.B = d->batch; fa.Hh = d->heads * G; fa.rpu = P; fa.D = d->head_dim; fa.Rp = d->hidden; fa.R = d->rank;
      e = launch_featmap_generic(fa, d->dtype, st);
    }
    if (e != hipSuccess) return e;
    prefill_psimax_kernel<<<U, 256, 0, st>>>(a.psi_all, P, d->rank, a.psimax);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    {
      const int rc = (d->rank + 256 / D - 1) / (256 / D);   // rows of H per thread
      const int nblk = P / kPrefixKeys;
#define LESSDEC_PREFIX(RC) prefill_prefix_kernel<T, D, RC><<<U * nblk, 256, 0, st>>>((const T *)a.V, a.psi_all, P, d->rank, \
                                                                                     d->n_heavy, a.hpre, a.zpre)
      if (nblk == 0) {}
      else if (rc <= 4) LESSDEC_PREFIX(4); else if (rc <= 8) LESSDEC_PREFIX(8);
      else if (rc <= 16) LESSDEC_PREFIX(16); else LESSDEC_PREFIX(32);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      prefill_prefix_scan_kernel<<<U * (unsigned)((d->rank * D + d->rank + 255) / 256), 256, 0, st>>>(
          nblk, d->rank * D, d->rank, a.hpre, a.zpre);
#undef LESSDEC_PREFIX
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const MaskedArgs mk = {a.phi_all, a.psi_all, a.psimax, a.hpre, a.zpre, d->rank, d->n_heavy, d->n_recent,
                         (d->flags & LESSDEC_FLAG_SPARSE_DENOM) ? 1 : 0};
  if constexpr (sizeof(T) == 2) {
    const RowArgs r = {a.Q, a.K, a.V, U, G, P, a.digits, a.lse, a.out, (unsigned *)a.bound, (unsigned *)a.count,
                       (unsigned *)a.empty, a.empty_count, masked ? &mk : nullptr, maps_ride ? &fm : nullptr};
    if ((e = launch_rows_f16(r, D, st)) != hipSuccess) return e;
  } else {
    const unsigned rows = prefill_grid(U * G, tiles);
    if (masked)
      prefill_maskedrows_kernel<D><<<rows, 64 * kPrefillWaves, 0, st>>>((const float *)a.Q, (const float *)a.K, (const float *)a.V,
                                                                       U * G, G, P, mk, a.lse, (float *)a.out);
    else
      prefill_rowpass_kernel<T, D><<<rows, 64 * kPrefillWaves, 0, st>>>((const T *)a.Q, (const T *)a.K, (const T *)a.V, U * G, G, P,
                                                                       a.lse, (T *)a.out);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // Column sums and selection.  Exact sums are needed of the kept tokens (they become the
  // accumulated scores) and of those whose rank is in doubt; with fp16 storage the cheap pass
  // tells which those are, with Lambda-masking the kept set is known beforehand.  Otherwise
  // (fp32 storage, or a prompt inside the budget) every column is summed exactly.
  const unsigned rank_grid = U * (unsigned)((P + 255) / 256);
  int32_t *keep = a.slot_of;
  if (P > C && (lambda || sizeof(T) == 2)) {
    if constexpr (sizeof(T) == 2) {
      if (!lambda) {
        // 256 keys per workgroup; 128 where that leaves compute units idle, or most of a workgroup's waves
        // without keys (640 units x 70 tokens: 13 against 18 us; 512 units x 150, D = 64: 17 against 13); 64 where even that
        // is one round (a whole prompt phase: 32 units x 500 94.5 against 97.8, 128 x 128 58.4 / 59.7; 64 x 500 114.4 / 113.9)
        const unsigned wide = prefill_grid(U, (unsigned)((P + 255) / 256)), narrow = prefill_grid(U, (unsigned)((P + 127) / 128));
#define LESSDEC_APPROX(KT, GRID)                                                                                        \
  prefill_colapprox_kernel<D, KT><<<GRID, 64 * kPrefillWaves, 0, st>>>((const __half *)a.Q, (const __half *)a.K, U, P, a.lse, G, \
                                                                       a.approx, (unsigned *)a.bound, (unsigned *)a.count)
        const unsigned thin = (unsigned)((P + 63) / 64);
        if (P <= 64 || (size_t)U * thin <= 448) LESSDEC_APPROX(1, prefill_grid(U, thin));
        else if (wide >= 512 && P > 128) LESSDEC_APPROX(4, wide);
        else LESSDEC_APPROX(2, narrow);
#undef LESSDEC_APPROX
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
    }
    prefill_select_kernel<<<U, 256, 0, st>>>(a.approx, (const unsigned *)a.bound, D, G, P, d->n_heavy, d->n_recent,
                                             lambda ? 1 : 0, a.slot_of, a.list, a.count);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if constexpr (sizeof(T) == 2) {
      e = launch_columns_f16(a.Q, a.K, U, G, P, D, a.lse, a.list, a.count, C, a.colsum, st);
    } else {
      const int bpu = (C + 32 + 16 * kPrefillWaves - 1) / (16 * kPrefillWaves);
      prefill_colexact_kernel<T, D><<<(U + kXcds - 1) / kXcds * kXcds * (unsigned)bpu, 64 * kPrefillWaves, 0, st>>>(
          (const T *)a.Q, (const T *)a.K, U, P, a.lse, a.list, a.count, bpu, G, a.colsum);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    if (!lambda) {
      prefill_refine_kernel<<<U, 256, 0, st>>>(a.colsum, a.slot_of, P, d->n_heavy, d->n_recent, a.list);
      keep = a.list;
    }
  } else {
    if constexpr (sizeof(T) == 2) {
      e = launch_columns_f16(a.Q, a.K, U, G, P, D, a.lse, nullptr, nullptr, C, a.colsum, st);
    } else {
      prefill_colpass_kernel<T, D><<<grid, 64 * kPrefillWaves, 0, st>>>((const T *)a.Q, (const T *)a.K, U, P,
                                                                       a.lse, G, a.colsum);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    prefill_rank_kernel<<<rank_grid, 256, 0, st>>>(a.colsum, P, d->n_heavy, d->n_recent, a.slot_of);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (!masked && !maps_ride && (e = key_features()) != hipSuccess) return e;
  const int shares = P > C ? (int)state_shares(U, (size_t)P, (size_t)d->rank, D, a.part_bytes) : 0;
  const bool fused = P > C && P <= 64 && U <= 512;         // (32 units x 12 tokens: 40.7 us in all, 41.6 with two launches)
  if (shares > 0 && !fused) {
    prefill_state_kernel<T, D><<<U * shares, 64 * kStateWaves, 0, st>>>((const T *)a.V, P, keep, a.psi_all, d->rank, shares,
                                                                        d->H, d->z, a.part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
#define LESSDEC_FINALIZE(W, STATE)                                                                                         \
  prefill_finalize_kernel<T, D, W, STATE><<<U, 64 * W, (size_t)C * sizeof(int), st>>>(                                    \
      (const T *)a.K, (const T *)a.V, P, a.colsum, keep, a.psi_all, C, d->rank, (T *)d->k_cache, (T *)d->v_cache, d->acc, \
      d->pos, d->psi, d->H, d->z, d->n_seen, d->pend_slot, ring_nh, a.part, shares)
  if (fused) LESSDEC_FINALIZE(kStateWaves, true);
  else LESSDEC_FINALIZE(8, false);
#undef LESSDEC_FINALIZE
  return hipGetLastError();
}

// -------------------------------------------------------------------------------------
// Row staging for the prompt taken token by token: one 16-byte vector per thread.
// -------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prompt_rows_kernel(const uint4 *__restrict__ Q, const uint4 *__restrict__ K,
                                                          const uint4 *__restrict__ V, uint4 *__restrict__ out,
                                                          uint4 *__restrict__ qs, uint4 *__restrict__ ks,
                                                          uint4 *__restrict__ vs, const uint4 *__restrict__ outs,
                                                          unsigned U, int G, int P, int vecs, int gather,
                                                          int scatter)
{
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;   // vector index in [U * G, vecs]
  if (i >= (size_t)U * G * vecs) return;
  const size_t ug = i / vecs, c = i % vecs;                  // query row (unit, head)
  if (scatter >= 0) out[(ug * P + scatter) * vecs + c] = outs[i];
  if (gather >= 0) {
    qs[i] = Q[(ug * P + gather) * vecs + c];
    if (ug % G == 0) {                                       // the unit's key and value rows, once
      const size_t u = ug / G;
      ks[u * vecs + c] = K[(u * P + gather) * vecs + c];
      vs[u * vecs + c] = V[(u * P + gather) * vecs + c];
    }
  }
}

hipError_t launch_prompt_rows(const PromptRowsArgs &a, int gather, int scatter, hipStream_t st)
{
  const int vecs = a.D * (a.dtype == LESSDEC_DTYPE_F16 ? 2 : 4) / 16;
  const size_t n = (size_t)a.U * a.G * vecs;
  prompt_rows_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(
      (const uint4 *)a.Q, (const uint4 *)a.K, (const uint4 *)a.V, (uint4 *)a.out, (uint4 *)a.qs, (uint4 *)a.ks,
      (uint4 *)a.vs, (const uint4 *)a.outs, a.U, a.G, a.P, vecs, gather, scatter);
  return hipGetLastError();
}

hipError_t launch_prefill(const PrefillArgs &a, hipStream_t st)
{
  const int D = a.d->head_dim;
  if (a.d->dtype == LESSDEC_DTYPE_F16)
    return D == 128 ? launch_prefill_t<__half, 128>(a, st) : launch_prefill_t<__half, 64>(a, st);
  return D == 128 ? launch_prefill_t<float, 128>(a, st) : launch_prefill_t<float, 64>(a, st);
}

}  // namespace lessdec
