// Decode step (Algorithm 1) for several query heads per key/value head (multi-query and
// grouped-query attention; Sec. 3.2, "Inexpensive Training", extends H2O to the attention
// scores of all query heads).  The G query heads of a unit share its sparse cache and its state
// H, z (psi acts on keys); each has its own phi and its own Eq. 3; a pair's accumulated score
// grows by its probability under every head.
//
// One block of 256 threads per unit (or per share of a unit's heads), all arithmetic fp64 in the
// order of the equations, the heads four at a time; a block first copies its unit's rows into the
// LDS when they fit.  The discarded pair is folded into H, z within the step (nothing is left
// pending).
#include "lessdec_digits.h"
#include "lessdec_wave.h"

namespace lessdec {

namespace {

// four adjacent stored elements (8 or 16 bytes, aligned) as floats, and back
template <typename T> __device__ inline void load_four(const T *p, float (&v)[4]);
template <> __device__ inline void load_four<float>(const float *p, float (&v)[4])
{
  const float4 x = *reinterpret_cast<const float4 *>(p);
  v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
}
template <> __device__ inline void load_four<__half>(const __half *p, float (&v)[4])
{
  const uint2 x = *reinterpret_cast<const uint2 *>(p);
  const __half2 lo = *reinterpret_cast<const __half2 *>(&x.x), hi = *reinterpret_cast<const __half2 *>(&x.y);
  v[0] = __low2float(lo); v[1] = __high2float(lo); v[2] = __low2float(hi); v[3] = __high2float(hi);
}
template <typename T> __device__ inline void store_four(T *p, const float (&v)[4]);
template <> __device__ inline void store_four<float>(float *p, const float (&v)[4])
{
  *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
template <> __device__ inline void store_four<__half>(__half *p, const float (&v)[4])
{
  const __half2 lo = __halves2half2(__float2half(v[0]), __float2half(v[1]));
  const __half2 hi = __halves2half2(__float2half(v[2]), __float2half(v[3]));
  uint2 x;
  x.x = *reinterpret_cast<const unsigned *>(&lo);
  x.y = *reinterpret_cast<const unsigned *>(&hi);
  *reinterpret_cast<uint2 *>(p) = x;
}

}  // namespace

// Layouts of this file's kernels: q, out [U,G,D]; k, v [U,D]; f_phi [U,G,R] fp64 or f_phi32 in
// fp32; f_psi [U,R] fp32.

// LDS copies of a unit's rows as they were before the step (H before the fold), for
// gqa_finish_unit; every null member is read from memory instead.
template <typename T>
struct LdsCopies {
  const T *k = nullptr, *v = nullptr;      // [m+1, D] rows in slot order, the appended pair last
  const float *H = nullptr;                // [R, D]
  const double *acc = nullptr;             // [m]
  const int *pos = nullptr;                // [m]
};

// After the unit's last head, by the whole block: accumulated scores, eviction
// choice, fold of the discarded pair into H, z (Eq. 4, Eq. 5), in-place insert of the new pair
// (Sec. 3.2).  s_inc holds the step's probabilities per pair summed over the heads; s_e is
// scratch of the same size; s_cand THREADS entries.
// Bound by latency: the loads are one round before the choice and one behind it (the pair that leaves: value row,
// psi), and H's elements are spread over all threads.  In a launch of its own, 64 units x 204 slots, D = 64: 5.1 us,
// against 6.5 with the choice as a tree over the LDS (a barrier per halving), H by the first D threads and every load
// where it was used; a whole step of 71 heads 33.5 us, against 35.5.
template <typename T, int D, int THREADS = 256>
__device__ inline void gqa_finish_unit(const StepArgs &a, int u, int tid, double *s_e, const double *s_inc,
                                       Cand *s_cand, const LdsCopies<T> lds = LdsCopies<T>())
{
  const int C = a.C, R = a.R;
  const int n = sane_n_seen(a.n_seen[u]);
  const int m = n < C ? n : C;
  const int rows = m + 1;
  const bool full = (m == C);
  T *kc = reinterpret_cast<T *>(a.k_cache) + (size_t)u * C * D;
  T *vc = reinterpret_cast<T *>(a.v_cache) + (size_t)u * C * D;
  const T *kn = reinterpret_cast<const T *>(a.k) + (size_t)u * D;
  const T *vn = reinterpret_cast<const T *>(a.v) + (size_t)u * D;
  float *Hu = a.H + (size_t)u * R * D;
  double *zu = a.z + (size_t)u * R;
  // requested before the choice, and before n_seen is needed, on which they do not depend: this thread's
  // elements of H (a full unit folds the discarded pair into all of them), z, the scores and positions of the
  // first pass, and the new pair's rows
  constexpr int HB = 8;
  const float *Hs = lds.H ? lds.H : Hu;
  const int hn = R * D;
  float h[HB];
  double z_old = 0.0;
  if (hn > 0) {
#pragma unroll
    for (int j = 0; j < HB; ++j) h[j] = Hs[tid + j * THREADS < hn ? tid + j * THREADS : hn - 1];
    if (tid < R) z_old = zu[tid];
  }
  const int first = tid < C ? tid : C - 1;
  const double acc_first = lds.acc ? lds.acc[first] : a.acc[(size_t)u * C + first];
  const int pos_first = lds.pos ? lds.pos[first] : a.pos[(size_t)u * C + first];
  T k_new = T(0.f), v_new = T(0.f);
  float psi_new = 0.f;
  if (tid < D) {
    k_new = lds.k ? lds.k[(size_t)m * D + tid] : kn[tid];
    v_new = lds.v ? lds.v[(size_t)m * D + tid] : vn[tid];
  }
  if (tid < R) psi_new = a.f_psi[(size_t)u * R + tid];
  // accumulated scores; eviction candidate of this thread's rows
  const bool lambda = (a.flags & LESSDEC_FLAG_LAMBDA) != 0;
  Cand best = cand_none();
  for (int r = tid; r < rows; r += THREADS) {
    double na = s_inc[r];
    int pj = n;
    if (r < m) {
      na += r == tid ? acc_first : lds.acc ? lds.acc[r] : a.acc[(size_t)u * C + r];
      pj = r == tid ? pos_first : lds.pos ? lds.pos[r] : a.pos[(size_t)u * C + r];
    }
    s_e[r] = na;
    if (full) {
      const bool is_cand = (r < m) ? (pj <= n - a.Nr && (!lambda || pj >= a.Nh)) : (a.Nr == 0);
      const Cand cnd{lambda ? 0.0 : na, pj, r};
      if (is_cand && cand_less(cnd, best)) best = cnd;
    }
  }
  // the smallest score, then the oldest among equals: of a wave by lane exchanges, of the waves through the LDS
  constexpr int NW = THREADS / kWave;
  const double amin = wave_allreduce(best.acc, OpMin{});
  const int pmin = wave_allreduce(best.acc == amin ? best.pos : INT_MAX, OpMinI{});
  const unsigned long long who = __ballot(best.acc == amin && best.pos == pmin && best.slot >= 0);
  if ((tid & (kWave - 1)) == 0) s_cand[tid / kWave] = cand_none();
  if (who != 0ull && (tid & (kWave - 1)) == __ffsll((long long)who) - 1) s_cand[tid / kWave] = best;
  __syncthreads();
  Cand win = s_cand[0];
#pragma unroll
  for (int w = 1; w < NW; ++w)
    if (cand_less(s_cand[w], win)) win = s_cand[w];
  const int eslot = full ? win.slot : -1;                    // eslot == m: the new pair itself
  const bool evict = eslot >= 0;
  const int ins_slot = full ? ((evict && eslot < m) ? eslot : -1) : m;

  // fold of the discarded pair into H, z (Eq. 4, Eq. 5), before its row is overwritten; the
  // pair's value row and psi go through the LDS
  if (evict) {
    float *s_ve = reinterpret_cast<float *>(s_cand + NW);    // behind the waves' candidates: [D], then psi [R]
    float *s_pe = s_ve + D;
    if (tid < D)
      s_ve[tid] = Store<T>::to_float(
          lds.v ? lds.v[(size_t)eslot * D + tid] : (eslot < m ? vc[(size_t)eslot * D + tid] : v_new));
    if (tid < R) s_pe[tid] = eslot < m ? a.psi[((size_t)u * C + eslot) * R + tid] : psi_new;
    __syncthreads();
    for (int e0 = 0; e0 < hn; e0 += HB * THREADS) {
      if (e0 > 0) {
#pragma unroll
        for (int j = 0; j < HB; ++j) {
          const int e = e0 + tid + j * THREADS;
          h[j] = Hs[e < hn ? e : hn - 1];
        }
      }
#pragma unroll
      for (int j = 0; j < HB; ++j) {
        const int e = e0 + tid + j * THREADS;
        if (e < hn) Hu[e] = (float)fma((double)s_pe[e / D], (double)s_ve[e % D], (double)h[j]);
      }
    }
    if (tid < R) zu[tid] = z_old + (double)s_pe[tid];
  }
  __syncthreads();
  // scores of the pairs that stay, and the new pair into its slot (Sec. 3.2: in place)
  for (int r = tid; r < m; r += THREADS)
    if (r != ins_slot) a.acc[(size_t)u * C + r] = s_e[r];
  if (ins_slot >= 0) {
    if (tid < D) {
      kc[(size_t)ins_slot * D + tid] = k_new;
      vc[(size_t)ins_slot * D + tid] = v_new;
    }
    if (tid < R) a.psi[((size_t)u * C + ins_slot) * R + tid] = psi_new;
    if (tid == 0) {
      a.acc[(size_t)u * C + ins_slot] = s_e[m];
      a.pos[(size_t)u * C + ins_slot] = n;
    }
  }
  if (tid == 0) {
    a.n_seen[u] = n + 1;
    a.pend_slot[u] = -1;
    if (a.evicted_pos) a.evicted_pos[u] = evict ? win.pos : -1;
  }
}

// The heads of a unit (or of a block's share of them) are taken four at a time (kGqaChunk = the
// block's four waves).  Per chunk: every thread scores its 16-byte share of a key row against
// the four queries; wave w then does the softmax of head w by itself (maximum, Eq. 3's low-rank
// denominator term, exponentials, their sum) with lane exchanges only, and the head's output the
// same way.  Four barriers per chunk.
// STAGE: the unit's key and value rows, H, the scores and positions are copied into the LDS
// once and every chunk works from there.  Without it (rows too many for the LDS) they are read
// from memory where they are used, the first passes of a sweep requested together.
// Dynamic LDS: see gqa_chunk_lds.
constexpr int kGqaChunk = 4;

template <typename T, int D, bool STAGE>
__global__ __launch_bounds__(256) void gqa_chunk_kernel(const StepArgs a, int G, int nhb)
{
  extern __shared__ double dyn[];
  constexpr int GC = kGqaChunk;
  constexpr int EPL = Store<T>::kPerVec, LPR = D / EPL, RPB = 256 / LPR;   // lanes per row, rows per pass
  constexpr int NQ = GC * D / 256;                                         // query elements per thread and chunk
  static_assert(NQ >= 1 && GC == 256 / kWave, "head_dim 64 or 128; one wave per head of a chunk");
  using Vec = typename Store<T>::Vec;
  const int u = (int)blockIdx.x / nhb, hb = (int)blockIdx.x % nhb, tid = threadIdx.x;
  const int g_begin = (int)((long)G * hb / nhb), g_end = (int)((long)G * (hb + 1) / nhb);
  const int lr = tid % LPR, rb = tid / LPR, lane = tid % kWave, w = tid / kWave;
  const int C = a.C, R = a.R;
  const int rows_cap = C + 2;                        // stride of the partial sums in the workspace
  const int ecap = (C + 3) & ~1;                     // LDS stride of a head's scores: even, so that all arrays stay 16-byte aligned
  double *s_e = dyn;                                 // [GC][ecap] scores, then e^{s - m*}
  double *s_inc = s_e + GC * ecap;               // [ecap] this step's probabilities per pair, summed over the heads
  double *s_q = s_inc + ecap;                    // [GC][D] queries of the chunk
  double *s_f = s_q + GC * D;                        // [GC][64] phi(q) of the chunk
  double *s_z = s_f + GC * 64;                       // [64] z
  double *s_hd = s_z + 64;                           // [GC][4] per head: e^{-m*} (0 without a state term), 1/den, 1/dacc
  double *s_acc = s_hd + GC * 4;                     // [C rounded up to 2] accumulated scores before the step
  int *s_pos = reinterpret_cast<int *>(s_acc + (C + 1) / 2 * 2);   // [C rounded up to 4] positions; 16-byte steps
  float *s_H = reinterpret_cast<float *>(s_pos + (C + 3) / 4 * 4);   // [R,D]
  T *s_k = reinterpret_cast<T *>(s_H + R * D);                  // [C+1,D] keys, the appended one last
  T *s_v = s_k + (size_t)(C + 1) * D;                           // [C+1,D] values
  Cand *s_cand = reinterpret_cast<Cand *>(s_q);                 // after the last chunk (256 entries fit in s_q, s_f)
  static_assert(sizeof(Cand) * 256 <= (GC * D + GC * 64) * sizeof(double), "candidates overlay the query area");

  const int n = sane_n_seen(a.n_seen[u]);
  const int m = n < C ? n : C;             // live slots are 0..m-1 (slots fill in order)
  const int rows = m + 1;                  // + the appended pair (K', V' of Eq. 3)
  const T *kc = reinterpret_cast<const T *>(a.k_cache) + (size_t)u * C * D;
  const T *vc = reinterpret_cast<const T *>(a.v_cache) + (size_t)u * C * D;
  const T *kn = reinterpret_cast<const T *>(a.k) + (size_t)u * D;
  const T *vn = reinterpret_cast<const T *>(a.v) + (size_t)u * D;
  const float *Hu = a.H + (size_t)u * R * D;

  // a chunk's query elements and phi entry of this thread, requested one chunk ahead; heads past
  // the block's share repeat its last one (computed, never stored)
  auto head_of = [&](int g0, int i) { return g0 + i < g_end ? g0 + i : g_end - 1; };
  auto fetch_q = [&](int g0, int j) -> double {
    const int e = j * 256 + tid, g = head_of(g0, e / D);
    return (double)Store<T>::to_float(reinterpret_cast<const T *>(a.q)[((size_t)u * G + g) * D + e % D]);
  };
  auto fetch_f = [&](int g0) -> double {
    if (tid >= GC * R) return 0.0;
    const size_t i = ((size_t)u * G + head_of(g0, tid / R)) * R + tid % R;
    return a.f_phi32 ? (double)a.f_phi32[i] : a.f_phi[i];
  };
  double q_next[NQ], f_next;
#pragma unroll
  for (int j = 0; j < NQ; ++j) q_next[j] = fetch_q(g_begin, j);
  f_next = fetch_f(g_begin);

  for (int r = tid; r < rows; r += 256) s_inc[r] = 0.0;
  if (tid < R) s_z[tid] = a.z[(size_t)u * R + tid];
  if constexpr (STAGE) {
    for (int r = tid; r < m; r += 256) {
      s_acc[r] = a.acc[(size_t)u * C + r];
      s_pos[r] = a.pos[(size_t)u * C + r];
    }
    // all requests of a batch first, then the LDS stores (the staged sizes fit one batch)
    constexpr int VPR = D / EPL, NB = 8;                     // 16-byte vectors per row; vectors per thread and batch
    const int nvec = rows * VPR;
    for (int b0 = 0; b0 < nvec; b0 += NB * 256) {
      Vec kb[NB], vb[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int i = b0 + j * 256 + tid, ic = i < nvec ? i : nvec - 1;
        const int r = ic / VPR, c = ic % VPR;
        kb[j] = load_vec<T>((r < m ? kc + (size_t)r * D : kn) + c * EPL);
        vb[j] = load_vec<T>((r < m ? vc + (size_t)r * D : vn) + c * EPL);
      }
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int i = b0 + j * 256 + tid;
        if (i < nvec) {
          reinterpret_cast<Vec *>(s_k)[i] = kb[j];
          reinterpret_cast<Vec *>(s_v)[i] = vb[j];
        }
      }
    }
    const int nh4 = R * D / 4;
    for (int b0 = 0; b0 < nh4; b0 += 4 * 256) {
      float4 hb4[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = b0 + j * 256 + tid;
        hb4[j] = reinterpret_cast<const float4 *>(Hu)[i < nh4 ? i : nh4 - 1];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = b0 + j * 256 + tid;
        if (i < nh4) reinterpret_cast<float4 *>(s_H)[i] = hb4[j];
      }
    }
  }
  const double inv_sqrt_d = 1.0 / sqrt((double)D);
  const bool sparse_den = (a.flags & LESSDEC_FLAG_SPARSE_DENOM) != 0;

  for (int g0 = g_begin; g0 < g_end; g0 += GC) {
    __syncthreads();                                         // the previous chunk is done with s_q, s_f, s_e, s_hd
#pragma unroll
    for (int j = 0; j < NQ; ++j) s_q[j * 256 + tid] = q_next[j];
    if (tid < GC * R) s_f[(tid / R) * 64 + tid % R] = f_next;
    if (g0 + GC < g_end) {
#pragma unroll
      for (int j = 0; j < NQ; ++j) q_next[j] = fetch_q(g0 + GC, j);
      f_next = fetch_f(g0 + GC);
    }
    __syncthreads();
    // scores of the four heads against the cached keys and the appended key: LPR lanes of 16
    // bytes per row, RPB rows per pass
    {
      double qreg[GC][EPL];
#pragma unroll
      for (int g = 0; g < GC; ++g)
#pragma unroll
        for (int i = 0; i < EPL; ++i) qreg[g][i] = s_q[g * D + lr * EPL + i];
      auto row_vec = [&](int r) -> Vec {                     // this lane's 16 bytes of key row r (clamped: in range)
        const int rc = r < rows ? r : rows - 1;
        if constexpr (STAGE) return *reinterpret_cast<const Vec *>(s_k + (size_t)rc * D + lr * EPL);
        return load_vec<T>((rc < m ? kc + (size_t)rc * D : kn) + lr * EPL);
      };
      auto score = [&](int r, const Vec &kv) {
        double kd[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) kd[i] = (double)Store<T>::get(kv, i);
#pragma unroll
        for (int g = 0; g < GC; ++g) {
          double acc = 0.0;
#pragma unroll
          for (int i = 0; i < EPL; ++i) acc = fma(qreg[g][i], kd[i], acc);
          acc = row_sum<LPR>(acc);
          if (lr == 0 && r < rows) s_e[g * ecap + r] = acc * inv_sqrt_d;
        }
      };
      if constexpr (STAGE) {
        for (int r0 = 0; r0 < rows; r0 += RPB) score(r0 + rb, row_vec(r0 + rb));
      } else {
        // from memory: the rows of the first NP passes are requested together
        constexpr int NP = 8;
        Vec kvs[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) kvs[p] = row_vec(p * RPB + rb);
#pragma unroll
        for (int p = 0; p < NP; ++p)
          if (p * RPB < rows) score(p * RPB + rb, kvs[p]);
        for (int r0 = NP * RPB; r0 < rows; r0 += RPB) score(r0 + rb, row_vec(r0 + rb));
      }
    }
    __syncthreads();
    // wave w: softmax of head w.  m* = max(scores, ln(phi(q) z^T)) is the common shift (Eq. 3
    // times e^{-m*}); den = phi(q) z^T e^{-m*} + sum_j e^{s_j - m*}
    {
      double *e_w = s_e + w * ecap;
      double mx = -__builtin_inf();
      for (int r = lane; r < rows; r += kWave) mx = fmax(mx, e_w[r]);
      mx = wave_allreduce(mx, OpMax{});
      double fz = 0.0;
      for (int r = 0; r < R; ++r) fz = fma(s_f[w * 64 + r], s_z[r], fz);
      const double lfz = fz > 0.0 ? log(fz) : -__builtin_inf();
      const double mstar = fmax(mx, lfz);
      const double wl = fz > 0.0 ? exp(lfz - mstar) : 0.0;
      double part = 0.0;
      for (int r = lane; r < rows; r += kWave) {
        const double e = exp_softmax_f64(e_w[r] - mstar);
        e_w[r] = e;
        part += e;
      }
      const double sum = wave_allreduce(part, OpAdd{});
      const double den = wl + sum;
      if (lane == 0) {
        s_hd[w * 4 + 0] = fz > 0.0 ? exp(-mstar) : 0.0;
        s_hd[w * 4 + 1] = 1.0 / den;
        s_hd[w * 4 + 2] = g0 + w < g_end ? 1.0 / (sparse_den ? sum : den) : 0.0;   // heads past the share add nothing
      }
    }
    __syncthreads();
    // wave w: output of head w, (phi(q) H e^{-m*} + sum_j e_j V_j) / den.  A lane takes four
    // adjacent columns and every NRS-th row; the row shares then meet by lane exchange.
    {
      constexpr int NQD = D / 4, NRS = kWave / NQD;          // column quads; row shares per wave
      const int dq = lane % NQD, rs = lane / NQD;
      const double *e_w = s_e + w * ecap;
      const double hs = s_hd[w * 4 + 0];
      double num[4] = {0.0, 0.0, 0.0, 0.0};
      if (rs == 0 && hs > 0.0) {
#pragma unroll 8
        for (int r = 0; r < R; ++r) {
          const float4 h4 = *reinterpret_cast<const float4 *>((STAGE ? s_H : Hu) + r * D + 4 * dq);
          const double f = s_f[w * 64 + r];
          num[0] = fma(f, (double)h4.x, num[0]);
          num[1] = fma(f, (double)h4.y, num[1]);
          num[2] = fma(f, (double)h4.z, num[2]);
          num[3] = fma(f, (double)h4.w, num[3]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) num[i] *= hs;
      }
#pragma unroll 8
      for (int r = rs; r < rows; r += NRS) {
        const double e = e_w[r];
        float v4[4];
        if constexpr (STAGE) load_four<T>(s_v + (size_t)r * D + 4 * dq, v4);
        else load_four<T>((r < m ? vc + (size_t)r * D : vn) + 4 * dq, v4);
#pragma unroll
        for (int i = 0; i < 4; ++i) num[i] = fma(e, (double)v4[i], num[i]);
      }
#pragma unroll
      for (int o = NQD; o < kWave; o *= 2)
#pragma unroll
        for (int i = 0; i < 4; ++i) num[i] += __shfl_xor(num[i], o);
      if (rs == 0 && g0 + w < g_end) {
        const double inv_den = s_hd[w * 4 + 1];
        float o4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          o4[i] = (float)(num[i] * inv_den);
          asm volatile("" : "+v"(o4[i]));                  // fp64 -> fp16 in one step would be a software sequence
        }
        store_four<T>(reinterpret_cast<T *>(a.out) + ((size_t)u * G + g0 + w) * D + 4 * dq, o4);
      }
    }
    // the chunk's probabilities (H2O accumulates those of every head), in head order
    for (int r = tid; r < rows; r += 256) {
      double inc = s_inc[r];
#pragma unroll
      for (int g = 0; g < GC; ++g) inc = fma(s_e[g * ecap + r], s_hd[g * 4 + 2], inc);
      s_inc[r] = inc;
    }
  }
  __syncthreads();

  if (nhb > 1) {
    // the unit's heads are spread over nhb blocks: leave this block's sums for the finishing launch
    double *part = a.gqa_parts + ((size_t)u * nhb + hb) * rows_cap;
    for (int r = tid; r < rows; r += 256) part[r] = s_inc[r];
    return;
  }
  LdsCopies<T> lds;
  if constexpr (STAGE) {
    lds.k = s_k; lds.v = s_v; lds.H = s_H; lds.acc = s_acc; lds.pos = s_pos;
  }
  gqa_finish_unit<T, D>(a, u, tid, s_e, s_inc, s_cand, lds);
}

// Dynamic LDS of gqa_chunk_kernel, in bytes.
template <typename T, int D>
static size_t gqa_chunk_lds(int C, int R, bool stage)
{
  const size_t work = (size_t)((kGqaChunk + 1) * ((C + 3) & ~1) + kGqaChunk * (D + 64) + 64 + kGqaChunk * 4) * sizeof(double);
  if (!stage) return work;
  return work + (size_t)((C + 1) / 2 * 2) * sizeof(double) + (size_t)((C + 3) / 4 * 4) * sizeof(int) +
         (size_t)R * D * sizeof(float) + 2 * (size_t)(C + 1) * D * sizeof(T);
}

// Finishing launch when a unit's heads were spread over several blocks: adds their sums in
// block order and finishes the unit.   grid = U, block = 256, dynamic LDS = 2 (C + 2) doubles.
template <typename T, int D>
__global__ __launch_bounds__(256) void gqa_finish_kernel(const StepArgs a, int nhb)
{
  extern __shared__ double dyn[];
  __shared__ Cand s_cand[256];
  const int u = (int)blockIdx.x, tid = threadIdx.x;
  const int rows_cap = a.C + 2;
  double *s_e = dyn, *s_inc = dyn + rows_cap;
  // the first pass's sums are requested before n_seen says how many of them the blocks wrote
  double p[kGqaMaxHeadBlocks];
  auto request = [&](int r) __attribute__((always_inline)) {
#pragma unroll
    for (int hb = 0; hb < kGqaMaxHeadBlocks; ++hb)
      p[hb] = a.gqa_parts[((size_t)u * nhb + (hb < nhb ? hb : nhb - 1)) * rows_cap + r];
  };
  request(tid < rows_cap ? tid : rows_cap - 1);
  const int n = sane_n_seen(a.n_seen[u]);
  const int rows = (n < a.C ? n : a.C) + 1;
  for (int r = tid; r < rows; r += 256) {
    if (r != tid) request(r);
    double v = 0.0;
#pragma unroll
    for (int hb = 0; hb < kGqaMaxHeadBlocks; ++hb)
      if (hb < nhb) v += p[hb];
    s_inc[r] = v;
  }
  __syncthreads();
  gqa_finish_unit<T, D>(a, u, tid, s_e, s_inc, s_cand);
}

// -------------------------------------------------------------------------------------
// Many query heads per unit (multi-query attention), fp16 storage: the heads sixteen at a time as the
// columns of matrix tiles.  A block of eight waves per share of a unit's head groups; tile T of 16 cache
// rows belongs to wave T mod 8, which keeps its scores in registers (NTW tiles).  Scores are exact
// integer products of digit planes (lessdec_digits.h; fp64 matrix products where a value has no
// digits), lane (g, c) holding rows 4 g + w of head c; softmax in fp64, maximum and sum through the LDS; a
// pair's share of the accumulated scores is its row's sum over the lanes c; p V in fp64 on
// v_mfma_f64_16x16x4_f64, as the vector form accumulates it, a row's values straight from memory (element
// d = D / 16 i + b is operand row i of block b, so a lane reads one run per row), and the waves' partial
// outputs meet in the LDS in wave order.  The vector form above (other shapes) scores a row for four heads at a time
// on the fp64 vector units: 64 us a step for 64 units x 71 heads x 204 slots (D = 64), against 35 here.
// Bound by latency: the two launches beside it, then a chain of key rows, two exchanges of the softmax, p V and the
// exchange of the outputs.  (p V on fp32 tiles: the same time at D = 64, 7 % less at D = 128 with 400 slots.)
// Dynamic LDS: gqm_lds.
// -------------------------------------------------------------------------------------
constexpr int kGqmWaves = 8, kGqmHeads = 16, kGqmMaxRows = 1024;

template <int D, int NTW>
__global__ __launch_bounds__(64 * kGqmWaves, D == 64 && NTW <= 2 ? 4 : 2) void gqm_step_kernel(const StepArgs a, int G, int nhb, int finish)
{
  using T = __half;
  constexpr int KC = D / 64, DB = D / 16, NV = DB / 2, THREADS = 64 * kGqmWaves, OS = D + 2;   // (two doubles behind a head's outputs, against bank conflicts)
  extern __shared__ __attribute__((aligned(16))) double dyn[];
  __shared__ double s_mx[kGqmWaves][kGqmHeads], s_sum[kGqmWaves][kGqmHeads], s_hd[kGqmHeads][2];
  const int C = a.C, R = a.R, rows_cap = C + 2;
  double *s_inc = dyn;                               // [C+2, even] this step's probabilities per pair, summed over the heads
  double *s_z = s_inc + (rows_cap + 1) / 2 * 2;      // [R, even] z
  double *s_f = s_z + (R + 1) / 2 * 2;               // [16][R] phi(q) of the group
  double *s_o = s_f + kGqmHeads * R;                 // [8][16][OS] partial outputs
  double *s_e = s_o;                                 // [C+1] scratch of the finish, after the last group
  Cand *s_cand = reinterpret_cast<Cand *>(s_o + kGqmMaxRows);
  static_assert(sizeof(Cand) * THREADS + sizeof(double) * kGqmMaxRows <= sizeof(double) * kGqmWaves * kGqmHeads * OS,
                "scores and candidates overlay the partial outputs");
  const int u = (int)blockIdx.x / nhb, hb = (int)blockIdx.x % nhb;
  const int ngrp = (G + kGqmHeads - 1) / kGqmHeads;
  const int grp0 = ngrp * hb / nhb, grp1 = ngrp * (hb + 1) / nhb;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int n = sane_n_seen(a.n_seen[u]);
  const int m = n < C ? n : C;             // live slots are 0..m-1 (slots fill in order)
  const int rows = m + 1;                  // + the appended pair (K', V' of Eq. 3)
  const T *kc = reinterpret_cast<const T *>(a.k_cache) + (size_t)u * C * D;
  const T *vc = reinterpret_cast<const T *>(a.v_cache) + (size_t)u * C * D;
  const T *kn = reinterpret_cast<const T *>(a.k) + (size_t)u * D, *vn = reinterpret_cast<const T *>(a.v) + (size_t)u * D;
  const float *Hu = a.H + (size_t)u * R * D;
  const double cs = kLog2E / sqrt((double)D);        // q . k to base-2 units
  const bool sparse_den = (a.flags & LESSDEC_FLAG_SPARSE_DENOM) != 0;
  auto row_of = [&](const T *cache, const T *last, int r) { return r < m ? cache + (size_t)r * D : last; };   // rows past the appended one repeat it

  for (int r = tid; r < rows; r += THREADS) s_inc[r] = 0.0;
  if (tid < R) s_z[tid] = a.z[(size_t)u * R + tid];
  for (int grp = grp0; grp < grp1; ++grp) {
    // the lane's place is unknown to the compiler anew for every group, or it computes all addresses ahead of the
    // loop and spills them
    int g = tid % 64 / 16, c = tid % 16;
    asm volatile("" : "+v"(g), "+v"(c));
    const int h0 = grp * kGqmHeads;
    const int hc = h0 + c < G ? h0 + c : G - 1;      // heads past the last repeat it: computed, never kept
    const bool head = h0 + c < G;
    __syncthreads();                                 // the group before is done with the LDS
    for (int i = tid; i < kGqmHeads * R; i += THREADS) {
      const int h = h0 + i / R < G ? h0 + i / R : G - 1;
      const size_t at = ((size_t)u * G + h) * R + i % R;
      s_f[i] = a.f_phi32 ? (double)a.f_phi32[at] : a.f_phi[at];
    }
    // scores of this wave's tiles, base-2 units
    const T *qrow = reinterpret_cast<const T *>(a.q) + ((size_t)u * G + hc) * D;
    RowDigits<D> qd;
    const bool qbad = __any(!qd.load(qrow, g));
    double e[NTW][4], mx = -__builtin_inf();
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      const int r0 = 16 * (t * kGqmWaves + wave);
#pragma unroll
      for (int w = 0; w < 4; ++w) e[t][w] = -__builtin_inf();
      if (r0 >= rows) continue;                      // wave-uniform
      RowDigits<D> kd;
      const bool kbad = __any(!kd.load(row_of(kc, kn, r0 + c), g));
      if (!qbad && !kbad) {
        v4i s[7];
#pragma unroll
        for (int i = 0; i < 7; ++i) s[i] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < KC; ++k)
#pragma unroll
          for (int pa = 0; pa < 4; ++pa) dot_planes(kd.d[k][pa], qd.d[k], pa, s);
        const DotParts p = dot_join(s);
#pragma unroll
        for (int w = 0; w < 4; ++w) e[t][w] = dot_affine(p, w, cs, 0.0);
      } else {
        const v4d s = dot_tile_f64<D>([&](int i) { return row_of(kc, kn, r0 + i); }, qrow, g, c);
#pragma unroll
        for (int w = 0; w < 4; ++w) e[t][w] = s[w] * cs;
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (r0 + 4 * g + w >= rows) e[t][w] = -__builtin_inf();
        mx = fmax(mx, e[t][w]);
      }
    }
    // this wave's value rows are requested ahead of the exchange where the registers hold them
    constexpr bool kAhead = NTW <= 4;
    unsigned vraw[kAhead ? NTW : 1][4][NV];
    auto load_values = [&](int t, unsigned (&v)[4][NV]) __attribute__((always_inline)) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const T *src = row_of(vc, vn, 16 * (t * kGqmWaves + wave) + 4 * g + w) + DB * c;
        if constexpr (NV == 4) {
          const uint4 x = *reinterpret_cast<const uint4 *>(src);
          v[w][0] = x.x; v[w][1] = x.y; v[w][2] = x.z; v[w][3] = x.w;
        } else {
          const uint2 x = *reinterpret_cast<const uint2 *>(src);
          v[w][0] = x.x; v[w][1] = x.y;
        }
      }
    };
    if constexpr (kAhead) {
#pragma unroll
      for (int t = 0; t < NTW; ++t) load_values(t, vraw[t]);
    }
    mx = fmax(mx, __shfl_xor(mx, 16));
    mx = fmax(mx, __shfl_xor(mx, 32));
    if (g == 0) s_mx[wave][c] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kGqmWaves; ++w) mx = fmax(mx, s_mx[w][c]);
    // m* = max(scores, exponent of phi(q) z^T) is the common shift (Eq. 3 times 2^{-m*}); den = phi(q) z^T
    // 2^{-m*} + sum_j 2^{s_j - m*}
    double fz = 0.0;
    for (int r = 0; r < R; ++r) fz = fma(s_f[c * R + r], s_z[r], fz);
    // (an infinite phi(q) z^T leaves no number, as ln of it would)
    const double mstar = fz > 0.0 ? fmax(mx, fz < __builtin_inf() ? (double)__builtin_amdgcn_frexp_exp(fz) : fz) : mx;
    double down[1] = {-mstar}, hs[1];
    exp2_f64(down, hs);
    if (!(fz > 0.0)) hs[0] = 0.0;
    double part = 0.0;
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      double y[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {                  // no weight for rows past the last, -inf and what is not a number
        y[w] = e[t][w] - mstar;
        y[w] = y[w] > -5000.0 ? y[w] : -5000.0;
      }
      exp2_f64(y, e[t]);
      part += (e[t][0] + e[t][1]) + (e[t][2] + e[t][3]);
    }
    part += __shfl_xor(part, 16);
    part += __shfl_xor(part, 32);
    if (g == 0) s_sum[wave][c] = part;
    __syncthreads();
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kGqmWaves; ++w) sum += s_sum[w][c];
    const double den = (fz > 0.0 ? fz * hs[0] : 0.0) + sum;
    if (wave == 0 && g == 0) {
      s_hd[c][0] = hs[0];
      s_hd[c][1] = 1.0 / den;
    }
    const double ascale = head ? 1.0 / (sparse_den ? sum : den) : 0.0;
    v4d O[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) O[b] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      const int r0 = 16 * (t * kGqmWaves + wave);
      if (r0 >= rows) continue;                      // wave-uniform
      if constexpr (!kAhead) load_values(t, vraw[0]);
      if (r0 + 16 > rows) {                          // wave-uniform: rows past the last have no value either
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
          for (int i = 0; i < NV; ++i) vraw[kAhead ? t : 0][w][i] = r0 + 4 * g + w < rows ? vraw[kAhead ? t : 0][w][i] : 0u;
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const double inc = row16_allreduce(e[t][w] * ascale, OpAdd{});
        const int r = r0 + 4 * g + w;
        if (c == 0 && r < rows) s_inc[r] += inc;     // the row is this wave's alone
#pragma unroll
        for (int b = 0; b < DB; ++b) {
          const __half2 h = __builtin_bit_cast(__half2, vraw[kAhead ? t : 0][w][b / 2]);
          O[b] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(b % 2 ? __high2float(h) : __low2float(h)), e[t][w], O[b], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int b = 0; b < DB; b += 2)
        *reinterpret_cast<double2 *>(s_o + (wave * kGqmHeads + c) * OS + DB * (g + 4 * w) + b) = double2{O[b][w], O[b + 1][w]};
    __syncthreads();
    // outputs, two adjacent columns of a head per thread: (phi(q) H 2^{-m*} + sum_j 2^{s_j - m*} V_j) / den
    for (int i = tid; i < kGqmHeads * D / 2; i += THREADS) {
      const int h = i / (D / 2), d = i % (D / 2) * 2;
      if (h0 + h >= G) break;
      double n0 = 0.0, n1 = 0.0;
      if (s_hd[h][0] > 0.0) {
#pragma unroll 4
        for (int r = 0; r < R; ++r) {
          const float2 h2 = *reinterpret_cast<const float2 *>(Hu + r * D + d);
          n0 = fma(s_f[h * R + r], (double)h2.x, n0);
          n1 = fma(s_f[h * R + r], (double)h2.y, n1);
        }
        n0 *= s_hd[h][0];
        n1 *= s_hd[h][0];
      }
#pragma unroll
      for (int w = 0; w < kGqmWaves; ++w) {
        const double2 o = *reinterpret_cast<const double2 *>(s_o + (w * kGqmHeads + h) * OS + d);
        n0 += o.x;
        n1 += o.y;
      }
      float f0 = (float)(n0 * s_hd[h][1]), f1 = (float)(n1 * s_hd[h][1]);
      asm volatile("" : "+v"(f0), "+v"(f1));         // fp64 -> fp16 in one step would be a software sequence
      *reinterpret_cast<__half2 *>(reinterpret_cast<T *>(a.out) + ((size_t)u * G + h0 + h) * D + d) = __floats2half2_rn(f0, f1);
    }
  }
  __syncthreads();
  if (!finish) {
    // the unit is finished by a launch of its own: leave this block's sums for it
    double *sums = a.gqa_parts + ((size_t)u * nhb + hb) * rows_cap;
    for (int r = tid; r < rows; r += THREADS) sums[r] = s_inc[r];
    return;
  }
  gqa_finish_unit<T, D, THREADS>(a, u, tid, s_e, s_inc, s_cand);
}

// Dynamic LDS of gqm_step_kernel, in bytes.
static size_t gqm_lds(int C, int R, int D)
{
  return ((size_t)(C + 3) / 2 * 2 + (R + 1) / 2 * 2 + kGqmHeads * R + (size_t)kGqmWaves * kGqmHeads * (D + 2)) * sizeof(double);
}

// Sixteen heads to a matrix tile pay from nine heads on (up to eight the streaming kernel takes them), also where a unit's
// one group of heads leaves it one block and the vector form would have had up to eight: a step against the
// vector form, us, 204 slots, D = 64: 9 heads x 8 units 23.0 and 25.8, x 64 23.5 and 26.2, x 512 29.8 and 56.3; 16 x 128 24.3
// and 32.1; 17 x 32 25.5 and 26.6; 800 slots: 9 x 8 36.6 and 50.5; D = 128, 800 slots: 16 x 256 58.8 and 181.  The two are
// level (within 2 %) with 16 slots and up to 64 units.
static bool gqm_supported(int dtype, int C, int G)
{
  return dtype == LESSDEC_DTYPE_F16 && G > 8 && C + 1 <= kGqmMaxRows;
}

// Blocks per unit: one when the units alone fill the chip, else the heads are spread over up
// to kGqaMaxHeadBlocks blocks (the cache rows are then staged once per block).
int gqa_head_blocks(long units, int G)
{
  int nhb = (int)((512 + units - 1) / units);          // measured: 512 units x 8 heads lose with a split
  if (nhb > kGqaMaxHeadBlocks) nhb = kGqaMaxHeadBlocks;
  if (nhb > G) nhb = G;
  return nhb < 1 ? 1 : nhb;
}

// Most dynamic LDS the staged form may take: two blocks of it share a compute unit's 160 KB.
constexpr size_t kGqaStagedLds = 76 * 1024;

// LDS one block may take on this device (queried once; the devices of a process are alike).
static size_t block_lds_limit()
{
  static const size_t limit = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return (size_t)0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return (size_t)0;
    return (size_t)v;
  }();
  return limit;
}

template <int D>
static hipError_t launch_step_gqm_t(const StepArgs &a, int G, hipStream_t st)
{
  const int ngrp = (G + kGqmHeads - 1) / kGqmHeads, tiles = (a.C + 1 + 15) / 16, ntw = (tiles + kGqmWaves - 1) / kGqmWaves;
  int nhb = gqa_head_blocks(a.U, G);
  // Few units: the finish is a launch of its own, also where the heads are one group and the block could finish its
  // unit itself (2 us a step less: 21.1 against 23.0 for 8 units x 16 heads), as lessdec_step_launches answers for the shape.
  const bool split = nhb > 1;
  if (nhb > ngrp) nhb = ngrp;
  const size_t lds = gqm_lds(a.C, a.R, D);
  if (lds > block_lds_limit()) return hipErrorInvalidValue;
#define LESSDEC_GQM(NTW) gqm_step_kernel<D, NTW><<<a.U * nhb, 64 * kGqmWaves, lds, st>>>(a, G, nhb, split ? 0 : 1)
  if (ntw <= 1) LESSDEC_GQM(1); else if (ntw <= 2) LESSDEC_GQM(2); else if (ntw <= 4) LESSDEC_GQM(4); else LESSDEC_GQM(8);
#undef LESSDEC_GQM
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (split) gqa_finish_kernel<__half, D><<<a.U, 256, (size_t)2 * (a.C + 2) * sizeof(double), st>>>(a, nhb);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_step_gqa_t(const StepArgs &a, int G, hipStream_t st)
{
  int nhb = gqa_head_blocks(a.U, G);
  const int nchunk = (G + kGqaChunk - 1) / kGqaChunk;
  if (nhb > nchunk) nhb = nchunk;                           // whole chunks per block
  // the rows are staged whenever they fit: with a single chunk per block they are read once either
  // way, but the copy has all its requests in flight at once (measured: 25.6 against 26.5 us)
  const size_t staged = gqa_chunk_lds<T, D>(a.C, a.R, true), plain = gqa_chunk_lds<T, D>(a.C, a.R, false);
  const bool stage = staged <= kGqaStagedLds && staged <= block_lds_limit();
  if (!stage && plain > block_lds_limit()) return hipErrorInvalidValue;
  if (stage)
    gqa_chunk_kernel<T, D, true><<<a.U * nhb, 256, staged, st>>>(a, G, nhb);
  else
    gqa_chunk_kernel<T, D, false><<<a.U * nhb, 256, plain, st>>>(a, G, nhb);
  if (nhb > 1) gqa_finish_kernel<T, D><<<a.U, 256, (size_t)2 * (a.C + 2) * sizeof(double), st>>>(a, nhb);
  return hipGetLastError();
}

hipError_t launch_step_gqa(const StepArgs &a, int G, int dtype, int D, hipStream_t st)
{
  if (gqm_supported(dtype, a.C, G)) return D == 128 ? launch_step_gqm_t<128>(a, G, st) : launch_step_gqm_t<64>(a, G, st);
  if (dtype == LESSDEC_DTYPE_F16)
    return D == 128 ? launch_step_gqa_t<__half, 128>(a, G, st) : launch_step_gqa_t<__half, 64>(a, G, st);
  return D == 128 ? launch_step_gqa_t<float, 128>(a, G, st) : launch_step_gqa_t<float, 64>(a, G, st);
}

}  // namespace lessdec
