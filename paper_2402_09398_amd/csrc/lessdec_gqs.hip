// Decode step (Algorithm 1) with several query heads per key/value head (Sec. 3.2: H2O aggregates
// the scores of all query heads), streaming form: one block per unit.
//
// A wave takes GH query heads (two or four) and every GH-th load of the unit's K rows and then of its V rows, which pass through a
// register ring as in the single-head kernel (lessdec_wpu.hip): a row is fetched and widened once for GH heads, and a
// wave's stream is a part of the cache.  Behind the scores wave g works for head g (softmax, denominator, output), and what the
// heads share is worked off by one wave each:
//   phase 1    scores of the wave's heads and rows, in fp64, into the LDS;
//   barrier 1  scores complete;
//   phase 2    wave g: shift and exponentials of head g, which weight the value rows as they are (the
//              sum is scaled by 1 / den at the output);
//   barrier 2  weights complete;
//   phase 3    p . V of the wave's heads and rows in fp32, into the LDS; behind its first pass wave g: phi(q) from the
//              feature-map entries, Eq. 3's denominator, the head's share of every pair's score increment, phi(q) H; the
//              last wave: psi of the step's key;
//   barrier 3  partial outputs and increments complete, every load of the unit's state and rows back: from here on the state may
//              be stored;
//   phase 4    wave g: the partial sums of head g in wave order, its output; wave 1: the increments in head order onto the
//              accumulated scores, the eviction, the discarded row parked and the new pair put in its place (Sec. 3.2); wave
//              2: H and z with the pending pair folded in; the last wave: psi.  All stores go through the L2 to memory.
// The fold of the discarded pair into H, z is left to the next step (pend_slot, as on the
// single-head path).  phi(q) per head and psi(k) come from the feature-map launch before it,
// complete or as the parts of their layer-2 sums, or (FUSED) from jobs inside this launch.
//
// Bound by vector instructions in phase 1 (with two waves a SIMD an fp64 one every 4.5 cycles) and by the chain behind it.  With a
// wave per head, each streaming every row for itself, 512 units x 4 heads x 102 slots took 10.3 us to the end of the keys, 18.1 to
// the end of a block (21.2 the slowest), 21.1 a step; now 6.8, 13.5 (17.0) and 16.4.  Other shapes at launch_step_gqs_h.
#include "lessdec_mlp.h"
#include "lessdec_wave.h"

namespace lessdec {

constexpr int kGqsMaxHeads = 8;
constexpr int kGqsFourWaves = 1024; // (below, at the launch)
constexpr int kGqsMaxRows = 512;    // C + 1 at most
constexpr int kGqsParts = 8;        // feature maps taken as parts up to this many (R' <= 512)

// FUSED: the step's feature-map jobs (mlp_parts_gq_job) are the first n_mlp workgroups of the launch
// and hand their results to the attention waves through the exchange array, as in the one-wave-
// per-unit kernel (wpu_step_kernel): an entry no job has written yet holds kMlpEmpty, jobs write
// through with device-scope stores, waves read with device-scope loads, ask again while any entry
// is empty (bounded by poll_limit, then the NaNs of the empty entries show in the unit's
// outputs), and hand the entries back empty with their other stores.  Workgroups are dispatched in
// index order and a job waits for nothing, so no cycle of waits exists.  A job is four waves: a
// block of four query heads runs one job, a block of eight two.
// GH: query heads of a wave, and waves that share a unit's rows
template <int D, int NR2, int RM, int DEPTH, int GH, bool FUSED>
__global__ __launch_bounds__(kGqsMaxHeads * kWave, FUSED || DEPTH == 4 ? 4 : 1) void gqs_step_kernel(
    void *k_cache_, const void *q_, const void *k_, int C_, int G_, int n_mlp, const void *Wq1_, const void *Wk1_,
    const void *Wq2_, const StepArgs a)
{
  using T = __half;
  constexpr int EPL = 8;                   // elements per lane
  constexpr int LPR = D / EPL;             // lanes per row
  constexpr int RPI = kWave / LPR;         // rows per load instruction
  constexpr int RS = GH;
  using Vec = typename Store<T>::Vec;

  extern __shared__ __attribute__((aligned(16))) double dyn[];

  const int C = C_, R = a.R, G = G_;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if constexpr (FUSED) {
    if ((int)blockIdx.x < n_mlp) {
      mlp_parts_gq_job<D, true>(reinterpret_cast<const __half *>(q_), reinterpret_cast<const __half *>(k_),
                                reinterpret_cast<const __half *>(Wq1_), reinterpret_cast<const __half *>(Wk1_),
                                reinterpret_cast<const __half *>(Wq2_), reinterpret_cast<const __half *>(a.Wk2), a.Hh, G,
                                a.Rp, R, a.B, a.mlp_out, (int)blockIdx.x * (G / 4) + wave / 4,
                                reinterpret_cast<unsigned char *>(dyn) + (wave / 4) * mlp_slab_bytes(D), wave % 4, lane);
      return;
    }
  }
  const int lr = lane % LPR, rb = lane / LPR;
  const int u = FUSED ? (int)blockIdx.x - n_mlp : (int)blockIdx.x;
  const int HG = (G + GH - 1) / GH, NW = HG * RS;           // groups of heads, waves
  const int hg = wave / RS, share = wave % RS;
  const int g = wave < G ? wave : G - 1;                     // the head this wave works for behind the scores
  const bool head_wave = wave < G, book_wave = wave == 1;
  const bool fold_wave = wave == (NW > 2 ? 2 : 0), psi_wave = wave == (NW > 2 ? NW - 1 : 0);
  const int rows_cap = (C + 2) & ~1;
  double *s_sc = dyn;                                        // [G][C+1] scores, then a head's share of the score increments
  float *s_p = reinterpret_cast<float *>(dyn + (size_t)G * rows_cap);               // [HG][C+1][GH] weights
  float *s_o = s_p + (size_t)HG * rows_cap * GH;             // [NW][GH][D] partial outputs

  T *kc = reinterpret_cast<T *>(k_cache_) + (size_t)u * C * D;
  T *vc = reinterpret_cast<T *>(a.v_cache) + (size_t)u * C * D;
  const T *kn = reinterpret_cast<const T *>(k_) + (size_t)u * D;
  const T *vn = reinterpret_cast<const T *>(a.v) + (size_t)u * D;

  // ---- requests, in the order they are wanted back (all unconditional, clamped addresses) ----------
  Vec qv[GH];
#pragma unroll
  for (int h = 0; h < GH; ++h) {
    const int head = hg * GH + h < G ? hg * GH + h : G - 1;
    qv[h] = load_vec<T>(reinterpret_cast<const T *>(q_) + ((size_t)u * G + head) * D + lr * EPL);
  }
  const Vec knv = load_vec<T>(kn + lr * EPL);
  u4v buf[DEPTH];
  {
    const __amdgpu_buffer_rsrc_t rk =
        __builtin_amdgcn_make_buffer_rsrc(kc, 0, C * D * (int)sizeof(T), 0x00020000);
#pragma unroll
    for (int j = 0; j < DEPTH; ++j)
      buf[j] = __builtin_amdgcn_raw_buffer_load_b128(rk, lane * 16, (j * RS + share) * (kWave * 16), 2 /* nt */);
  }
  __builtin_amdgcn_sched_barrier(0);
  const int rl = (lane & 15) < R ? (lane & 15) : R - 1;
  // phi(q) of this wave's head and psi(k) of the step's key (lane r < R): complete from the feature-map
  // launch, or (a.mlp_parts) as the parts of their layer-2 sums
  constexpr int NP = kGqsParts;
  const bool parts = a.mlp_parts != nullptr;
  const int nparts = mlp_nparts(a.Rp), rp = mlp_entry_stride(R);
  const size_t fi = ((size_t)u * G + g) * R + rl;
  double f_lane = 0.0;
  float npsi_lane = 0.f;
  float pq[NP], pk[NP];
  __half w3[RM];
  const float *eq = a.mlp_parts + ((size_t)u * G + g) * nparts * rp + rl;
  const float *ek = a.mlp_parts + ((size_t)a.U * G + u) * nparts * rp + rl;
  auto request_parts = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int pc = p < nparts ? p : nparts - 1;
      if constexpr (FUSED) {
        pq[p] = __hip_atomic_load(eq + (size_t)pc * rp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        pk[p] = __hip_atomic_load(ek + (size_t)pc * rp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        pq[p] = eq[(size_t)pc * rp];
        pk[p] = ek[(size_t)pc * rp];
      }
    }
  };
  auto finish_phi = [&]() __attribute__((always_inline)) {
    double sq = 0.0;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (p < nparts) sq += (double)pq[p];
    f_lane = lane < R ? fabs(gelu_poly_f64(sq)) : 0.0;     // last activation of Eq. 1
  };
  auto finish_psi = [&]() __attribute__((always_inline)) {
    double sk = 0.0;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (p < nparts) sk += (double)pk[p];
    const double h2 = gelu_poly_f64(sk);                   // lane r < R; Eq. 2: |W3 gelu(.)|
    double acc3 = 0.0;
#pragma unroll
    for (int j = 0; j < RM; ++j)
      if (j < R) acc3 = fma(readlane_v(h2, j), (double)__half2float(w3[j]), acc3);
    npsi_lane = (float)fabs(acc3);
  };
  const int n = sane_n_seen(a.n_seen[u]);
  const Pending pend = decode_pending(a.pend_slot[u], C);
  const int m = n < C ? n : C;          // live slots are 0..m-1 (slots fill in order)
  const int rows = m + 1;               // + the appended pair (K', V' of Eq. 3)
  const bool full = (m == C);
  // The stream: position s < nitp is the wave's load s of K, position nitp + t its load t of V.
  const int nl = (rows + RPI - 1) / RPI;                     // load instructions per stream (>= 1)
  const int nit = nl > share ? (nl - share + RS - 1) / RS : 1;   // the wave's
  const int nitp = (nit + DEPTH - 1) / DEPTH * DEPTH;        // K part of the stream, padded
  const int live_bytes = m * D * (int)sizeof(T);
  auto issue = [&](int s) -> u4v {                           // s is wave-uniform
    const bool isk = s < nitp;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(isk ? kc : vc, 0, live_bytes, 0x00020000);
    return __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, ((isk ? s : s - nitp) * RS + share) * (kWave * 16), 2 /* nt */);
  };

  // ---- phase 1: scores as the key rows arrive -------------------------------------------------------
  {
    const double inv_sqrt_d = 1.0 / sqrt((double)D);
    double qd[GH][EPL];
#pragma unroll
    for (int h = 0; h < GH; ++h)
#pragma unroll
      for (int i = 0; i < EPL; ++i) qd[h][i] = (double)Store<T>::get(qv[h], i);
    u4v knu;                                               // (as a value: a choice between addresses would put the ring into scratch memory)
    __builtin_memcpy(&knu, &knv.raw, 16);
    const bool stores = lr < GH && hg * GH + lr < G;       // lane lr < GH of a row ends with the score of head lr
    double *s_mine = s_sc + (size_t)(stores ? hg * GH + lr : 0) * rows_cap;
    auto key_pass = [&](int base) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < DEPTH; ++j) {
        const int s = base + j;
        if (s < nit) {
          const int r = (s * RS + share) * RPI + rb;
          const u4v kraw = (r == m) ? knu : buf[j];          // r == m: the appended key
          Vec kv;
          __builtin_memcpy(&kv.raw, &kraw, 16);
          double sum[GH] = {};
#pragma unroll
          for (int i = 0; i < EPL; ++i) {
            const double k = (double)Store<T>::get(kv, i);
#pragma unroll
            for (int h = 0; h < GH; ++h) sum[h] = fma(qd[h][i], k, sum[h]);
          }
          double x;
          if constexpr (GH == 4) x = row_sum4<LPR>(sum, lane);
          else x = row_sum2<LPR>(sum[0], sum[1], lane);
          if (stores && r < rows) s_mine[r] = x * inv_sqrt_d;
        }
        buf[j] = issue(s + DEPTH);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    for (int base = 0; base < nitp; base += DEPTH) key_pass(base);
  }
  // ---- requests behind the keys, once the queries have given their registers back: feature maps and state --------------------
  if (parts) {
    request_parts();                                         // (FUSED: the jobs are done by now)
    const __half *w3row = reinterpret_cast<const __half *>(a.Wk3) + ((size_t)(u % a.Hh) * R + rl) * R;
#pragma unroll
    for (int j = 0; j < RM; ++j) w3[j] = w3row[j < R ? j : R - 1];
  } else {
    f_lane = a.f_phi32 ? (double)a.f_phi32[fi] : a.f_phi[fi];
    npsi_lane = a.f_psi[(size_t)u * R + rl];
  }
  double z_lane = a.z[(size_t)u * R + rl];                   // lane r < R
  const float ppsi_lane = a.pend_psi[(size_t)u * R + rl];
  float psie_lane = a.psi[((size_t)u * C + (pend.slot >= 0 && pend.slot < C ? pend.slot : 0)) * R + rl];
  __builtin_amdgcn_sched_barrier(0);
  // barrier 1: the scores
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");

  // ---- phase 2: shift and exponentials of the wave's head ------------------------------------------
  double sc[NR2];
  double M = -__builtin_inf();
  if (head_wave) {
#pragma unroll
    for (int i = 0; i < NR2; ++i) {
      const int j = lane + i * kWave;
      const double x = s_sc[(size_t)g * rows_cap + (j < rows ? j : 0)];
      sc[i] = j < rows ? x : -__builtin_inf();
      M = fmax(M, sc[i]);
    }
    M = wave_allreduce(M, OpMax{});
#pragma unroll
    for (int i = 0; i < NR2; ++i) sc[i] = exp_softmax_f64(sc[i] - M);
#pragma unroll
    for (int i = 0; i < NR2; ++i) {
      const int j = lane + i * kWave;
      if (j < rows) s_p[((size_t)(g / GH) * rows_cap + j) * GH + g % GH] = (float)sc[i];
    }
  }
  // barrier 2: the weights
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");

  // ---- phase 3: e^{s - M} . V as the value rows arrive ----------------------------------------------
  float o[GH][EPL];
#pragma unroll
  for (int h = 0; h < GH; ++h)
#pragma unroll
    for (int i = 0; i < EPL; ++i) o[h][i] = 0.f;
  struct alignas(4 * GH) Weights { float h[GH]; };
  const Weights *p_row = reinterpret_cast<const Weights *>(s_p) + (size_t)hg * rows_cap;
  auto add_row = [&](const Weights &p, const Vec &vv) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < EPL; ++i)
#pragma unroll
      for (int h = 0; h < GH; ++h) o[h][i] = fmaf(p.h[h], Store<T>::get(vv, i), o[h][i]);
  };
  auto value_pass = [&](int base) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) {
      const int s = base + j;
      if (s < nit) {
        const int r = (s * RS + share) * RPI + rb;
        Vec vv;
        __builtin_memcpy(&vv.raw, &buf[j], 16);
        if (r < m) add_row(p_row[r], vv);
      }
      buf[j] = issue(nitp + s + DEPTH);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // The first pass always runs, so that its loads sit under no condition; passes past the end of the stream consume nothing
  // and request rows outside the buffer's range, which fetches nothing.
  value_pass(0);

  // between the passes: the feature maps, Eq. 3's denominator, the head's share of the score increments, phi(q) H
  double lscale = 0.0, pscale = 0.0;
  float fh[4] = {0.f, 0.f, 0.f, 0.f};                        // phi(q) H, this lane's columns and rows
  if (parts) {
    if constexpr (FUSED) {
      // The first look stands outside the loop and looks at every entry: a look at the loop's head,
      // or one that leaves after the first empty entry, would make whoever uses the entries next
      // wait for everything in flight.
      auto have_all = [&]() {
        unsigned missing = 0;
#pragma unroll
        for (int p = 0; p < NP; ++p)
          missing |= (unsigned)(__float_as_uint(pq[p]) == kMlpEmpty) | (unsigned)(__float_as_uint(pk[p]) == kMlpEmpty);
        return __all(missing == 0u) != 0;
      };
      bool have = have_all();
      constexpr int kSleep = 4;
      for (int spin = 0; !have && spin < poll_limit(kSleep); ++spin) {
        __builtin_amdgcn_s_sleep(kSleep);
        request_parts();
        have = have_all();
      }
    }
    if (psi_wave) finish_psi();
    if (head_wave) finish_phi();
  }
  // requests that take the entries' place: what the output and the bookkeeping want
  const Vec vnv = load_vec<T>(vn + lr * EPL);
  constexpr int NHB = RPI / 2, HR = RM / NHB;
  const int col0 = lr * EPL + ((lane & LPR) ? 4 : 0);
  const int hb = lane / (2 * LPR);                           // which rows of H: r = NHB * i + hb
  float4 hreg[HR];
#pragma unroll
  for (int i = 0; i < HR; ++i) {
    const int r = NHB * i + hb;
    hreg[i] = *reinterpret_cast<const float4 *>(a.H + ((size_t)u * R + (r < R ? r : R - 1)) * D + col0);
  }
  const uint2 pend_v_h = *reinterpret_cast<const uint2 *>(reinterpret_cast<const T *>(a.pend_v) + (size_t)u * D + col0);
  double acc_pre[NR2];
  int pos_pre[NR2];
#pragma unroll
  for (int i = 0; i < NR2; ++i) {
    const int j = lane + i * kWave;
    const size_t idx = (size_t)u * C + (j < C ? j : C - 1);
    acc_pre[i] = a.acc[idx];
    pos_pre[i] = a.pos[idx];
  }
  // pending fold of z (Eq. 5)
  if (lane >= R) z_lane = 0.0;
  if (!pend.fold) psie_lane = 0.f;
  else if (pend.slot >= C) psie_lane = ppsi_lane;            // the previous step discarded its own pair
  if (lane < R && pend.fold) z_lane += (double)psie_lane;
  if (head_wave) {
    if (lane >= R) f_lane = 0.0;
    double S = 0.0;
#pragma unroll
    for (int i = 0; i < NR2; ++i) S += sc[i];
    S = wave_allreduce(S, OpAdd{});                          // sparse part of the denominator, shifted
    const double fz = wave_allreduce(f_lane * z_lane, OpAdd{});
    if (fz > 0.0 && M <= 0.0) {
      const double w = exp_softmax_f64(M);
      const double inv = 1.0 / (fz + w * S);
      pscale = w * inv;
      lscale = inv;
    } else {
      const double eM = (fz > 0.0) ? exp_softmax_f64(-M) : 0.0;
      const double inv = 1.0 / (fz * eM + S);
      pscale = inv;
      lscale = eM * inv;
    }
    double ascale = pscale;
    if (a.flags & LESSDEC_FLAG_SPARSE_DENOM) ascale = 1.0 / S;
#pragma unroll
    for (int i = 0; i < NR2; ++i) {
      const int j = lane + i * kWave;
      if (j < rows) s_sc[(size_t)g * rows_cap + j] = sc[i] * ascale;
    }
  }
  for (int base = DEPTH; base < nit; base += DEPTH) value_pass(base);
  if (head_wave || fold_wave) {
    // fold the pending pair into H (Eq. 4), then this head's phi(q) H
    const float f32 = (float)f_lane;
    const __half2 *pvh = reinterpret_cast<const __half2 *>(&pend_v_h);
    const float2 pv01 = __half22float2(pvh[0]), pv23 = __half22float2(pvh[1]);
#pragma unroll
    for (int i = 0; i < HR; ++i) {
      const int r = NHB * i + hb;
      const int rc = r < R ? r : R - 1;
      const float fr = r < R ? __shfl(f32, rc) : 0.f;
      const float pe = __shfl(psie_lane, rc);
      if (pend.fold) {
        hreg[i].x = fmaf(pe, pv01.x, hreg[i].x);
        hreg[i].y = fmaf(pe, pv01.y, hreg[i].y);
        hreg[i].z = fmaf(pe, pv23.x, hreg[i].z);
        hreg[i].w = fmaf(pe, pv23.y, hreg[i].w);
      }
      fh[0] = fmaf(fr, hreg[i].x, fh[0]);
      fh[1] = fmaf(fr, hreg[i].y, fh[1]);
      fh[2] = fmaf(fr, hreg[i].z, fh[2]);
      fh[3] = fmaf(fr, hreg[i].w, fh[3]);
    }
  }
  // the appended pair's value row
  if (share == 0 && rb == 0) add_row(p_row[m], vnv);
  {
    // the row groups' partial sums, spread over the heads
    if constexpr (GH == 4) {
      float part[EPL];
      combine_four_heads<LPR>(o, part);
      if (LPR == 16 || (lane & 8) == 0) {
        float4 *dst = reinterpret_cast<float4 *>(s_o + ((size_t)wave * GH + lane / 16) * D + lr * EPL);
        dst[0] = float4{part[0], part[1], part[2], part[3]};
        dst[1] = float4{part[4], part[5], part[6], part[7]};
      }
    } else {
      float part[4];
      combine_two_heads<LPR>(o, part, lane);
      if (LPR == 16 || (lane & 16) == 0)
        *reinterpret_cast<float4 *>(s_o + ((size_t)wave * GH + lane / 32) * D + col0) = float4{part[0], part[1], part[2], part[3]};
    }
  }
  // barrier 3: partial outputs and increments.  (The rows still in a ring are requests past the value stream, out of range:
  // every wave that arrives here has all the cache rows and state it will ever read, but for the discarded row.)
#pragma unroll
  for (int j = 0; j < DEPTH; ++j) asm volatile("" ::"v"(buf[j]));
#pragma unroll
  for (int i = 0; i < HR; ++i) asm volatile("" ::"v"(hreg[i].x), "v"(hreg[i].y), "v"(hreg[i].z), "v"(hreg[i].w));
#pragma unroll
  for (int i = 0; i < NR2; ++i) asm volatile("" ::"v"(acc_pre[i]), "v"(pos_pre[i]));
  asm volatile("" ::"v"(z_lane), "v"(ppsi_lane), "v"(psie_lane), "v"(pend_v_h.x), "v"(pend_v_h.y), "v"(npsi_lane), "v"(f_lane));
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");

  // ---- phase 4 --------------------------------------------------------------------------------------
  int eslot = -1, ins_slot = -1;
  u4v pv_row = {0u, 0u, 0u, 0u};                            // the discarded pair's value row
  if (book_wave) {
    // accumulated scores and the eviction
    const bool lambda = (a.flags & LESSDEC_FLAG_LAMBDA) != 0;
    int epos = -1;
    double na_[NR2];
    Cand best = cand_none();
#pragma unroll
    for (int i = 0; i < NR2; ++i) na_[i] = 0.0;
    // In head order, four at a time: eight of four rows a lane are more registers than anything else here needs, and left 129 to 256
    // rows two waves a SIMD where three fit (2048 units x 4 heads x 150 slots 62.5 us a step, now 54.5; D = 64 49.4 and 40.2).
#pragma unroll 4
    for (int h = 0; h < G; ++h) {
#pragma unroll
      for (int i = 0; i < NR2; ++i) {
        const int j = lane + i * kWave;
        na_[i] += s_sc[(size_t)h * rows_cap + (j < rows ? j : 0)];
      }
    }
#pragma unroll
    for (int i = 0; i < NR2; ++i) {
      const int j = lane + i * kWave;
      const double na = na_[i] + (j < m ? acc_pre[i] : 0.0);
      const int pj = j < m ? pos_pre[i] : n;
      na_[i] = na;
      const bool is_cand = (j < m) ? (pj <= n - a.Nr && (!lambda || pj >= a.Nh)) : (j == m && a.Nr == 0);
      const Cand cnd{lambda ? 0.0 : na, pj, j};
      const bool take = full && is_cand && cand_less(cnd, best);
      best.acc = take ? cnd.acc : best.acc;
      best.pos = take ? cnd.pos : best.pos;
      best.slot = take ? cnd.slot : best.slot;
    }
    if (full) {
      const double amin = wave_allreduce(best.acc, OpMin{});
      const int pmin = wave_allreduce(best.acc == amin ? best.pos : INT_MAX, OpMinI{});
      const unsigned long long win = __ballot(best.acc == amin && best.pos == pmin && best.slot >= 0);
      if (win != 0ull) {
        eslot = __builtin_amdgcn_readlane(best.slot, __ffsll((long long)win) - 1);
        epos = pmin;
      }
    }
    const bool evict = eslot >= 0;                           // eslot == m: the new pair itself
    ins_slot = full ? ((evict && eslot < m) ? eslot : -1) : m;
    // its value row once more, from row 0 where no cached pair leaves
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(vc, 0, C * D * (int)sizeof(T), 0x00020000);
    const int er = (evict && eslot < m) ? eslot : 0;
    pv_row = __builtin_amdgcn_raw_buffer_load_b128(rv, lr * 16, er * (D * (int)sizeof(T)), 0);
#pragma unroll
    for (int i = 0; i < NR2; ++i) {
      // (the new pair's, row m, goes where it is put)
      const int j = lane + i * kWave, to = j < m ? j : ins_slot;
      if (j < m ? j != ins_slot : j == m && ins_slot >= 0) store_wt(a.acc + (size_t)u * C + to, na_[i]);
    }
    if (lane == 0) {
      store_wt(a.pend_slot + u, eslot >= 0 ? (eslot < m ? eslot : C) : (m | kPendNoFold));
      if (a.evicted_pos) store_wt(a.evicted_pos + u, eslot >= 0 ? epos : -1);
      store_wt(a.n_seen + u, n + 1);
      if (ins_slot >= 0) store_wt(a.pos + (size_t)u * C + ins_slot, n);
    }
  }
  if (fold_wave && pend.fold) {                              // H and z with the pending pair folded in (Eq. 4, Eq. 5)
#pragma unroll
    for (int i = 0; i < HR; ++i) {
      const int r = NHB * i + hb;
      if (r < R) store_wt16(a.H + (size_t)u * R * D, (r * D + col0) * (int)sizeof(float), hreg[i]);
    }
    if (lane < R) store_wt(a.z + (size_t)u * R + lane, z_lane);
  }
  if (psi_wave && lane < R) {
    if (pend.slot >= 0 && pend.slot < C) store_wt(a.psi + ((size_t)u * C + pend.slot) * R + lane, ppsi_lane);
    store_wt(a.pend_psi + (size_t)u * R + lane, npsi_lane);
  }
  // the feature-map entries go back empty
  if (parts) {
    for (int e = lane; e < nparts * (rp / 4); e += kWave) {
      if (head_wave)
        store_wt16(a.mlp_out + ((size_t)u * G + g) * nparts * rp, e * 16, uint4{kMlpEmpty, kMlpEmpty, kMlpEmpty, kMlpEmpty});
      if (psi_wave)
        store_wt16(a.mlp_out + ((size_t)a.U * G + u) * nparts * rp, e * 16, uint4{kMlpEmpty, kMlpEmpty, kMlpEmpty, kMlpEmpty});
    }
  }
  if (head_wave) {
    // the head's output: the waves' partial sums in wave order, phi(q) H over the row subsets of H
    float4 part[RS];
#pragma unroll
    for (int s = 0; s < RS; ++s)
      part[s] = *reinterpret_cast<const float4 *>(s_o + ((size_t)((g / GH) * RS + s) * GH + g % GH) * D + col0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (LPR == 8) fh[i] = add_xor<16>(fh[i]);
      fh[i] = add_xor<32>(fh[i]);
    }
    float4 sum = part[0];
#pragma unroll
    for (int s = 1; s < RS; ++s) {
      sum.x += part[s].x; sum.y += part[s].y; sum.z += part[s].z; sum.w += part[s].w;
    }
    if (hb == 0) {
      // (written out so that the forms of this kernel round alike: one multiply-add, fp64 -> fp32 -> fp16)
      auto value = [&](float x, float f) {
        float y = (float)fma(pscale, (double)x, lscale * (double)f);
        asm("" : "+v"(y));
        return y;
      };
      __half2 res[2];
      res[0] = __floats2half2_rn(value(sum.x, fh[0]), value(sum.y, fh[1]));
      res[1] = __floats2half2_rn(value(sum.z, fh[2]), value(sum.w, fh[3]));
      store_wt8(reinterpret_cast<T *>(a.out) + ((size_t)u * G + g) * D + col0, *reinterpret_cast<const uint2 *>(res));
    }
  }
  if (book_wave) {
    // the discarded row, parked for the next step's fold, then the new pair in its place
    if (eslot >= 0 && rb == 0) {
      uint4 row = vnv.raw;
      if (eslot < m) __builtin_memcpy(&row, &pv_row, 16);
      store_wt16(reinterpret_cast<T *>(a.pend_v) + (size_t)u * D, lr * EPL * (int)sizeof(T), row);
    }
    if (ins_slot >= 0 && rb == 0) {
      store_wt16(kc + (size_t)ins_slot * D, lr * EPL * (int)sizeof(T), knv.raw);
      store_wt16(vc + (size_t)ins_slot * D, lr * EPL * (int)sizeof(T), vnv.raw);
    }
  }
}

bool gqs_supported(int dtype, int D, int C, int R, int G)
{
  return dtype == LESSDEC_DTYPE_F16 && (D == 64 || D == 128) && R <= 16 && C + 1 <= kGqsMaxRows && G >= 2 &&
         G <= kGqsMaxHeads;
}

bool gqs_takes_parts(int Rp) { return mlp_nparts(Rp) <= kGqsParts; }

// One launch for the whole step: four or eight query heads per unit (the block is then one or two
// feature-map jobs of four waves), parts that fit the registers kept for them, and the kernel form
// that stays within the 128 registers four resident waves per SIMD leave each.
bool gqs_fusable(int D, int C, int Rp, int R, int G)
{
  return (G == 4 || G == 8) && D == 128 && C + 1 <= 2 * kWave && R <= 8 && mlp_nparts(Rp) <= kGqsParts;
}

template <int D, int RM, int GH>
static hipError_t launch_step_gqs_t(const StepArgs &a, int G, hipStream_t st, const MlpPartsArgs *fm)
{
  constexpr int kDepth = 7;
  const int rows_cap = (a.C + 2) & ~1, groups = (G + GH - 1) / GH, waves = groups * GH;
  const size_t lds = (size_t)G * rows_cap * sizeof(double) + (size_t)groups * rows_cap * GH * sizeof(float) +
                     (size_t)waves * GH * D * sizeof(float);
  const unsigned block = (unsigned)(waves * kWave);
  const int rows = a.C + 1;
  if (fm) {
    if constexpr (D == 128 && RM == 8 && GH == 2) {
      const int per = G / 4;                               // feature-map jobs, of four waves each, a block
      const unsigned n_mlp = (unsigned)((mlp_parts_gq_jobs(a.Hh, G, a.Rp, a.B) + per - 1) / per);
      const size_t slabs = (size_t)per * mlp_slab_bytes(D), lds_f = lds < slabs ? slabs : lds;
      gqs_step_kernel<D, 2, RM, 5, GH, true><<<n_mlp + (unsigned)a.U, block, lds_f, st>>>(a.k_cache, a.q, a.k, a.C, G, (int)n_mlp,
                                                                                         fm->Wq1, fm->Wk1, fm->Wq2, a);
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;
    }
  }
  const unsigned grid = (unsigned)a.U;
  // (Ranks above 8 at D = 64, two heads a wave, few rows: a ring of four leaves the registers for four waves a SIMD, where seven deep three
  // are there and 880 units of three heads do not run at once.  x 41 slots 26.0 against 23.3 us a step; 2000 x 2 x 41 29.2 and 24.7, 4000 x
  // 2 x 120 55.8 and 50.9, 1200 x 6 x 120 67.9 and 51.6.)
  constexpr int kFewDepth = D == 64 && RM == 16 && GH == 2 ? 4 : kDepth;
#define LESSDEC_GQS_LAUNCH(NR2, DEPTH)                                                                            \
  gqs_step_kernel<D, NR2, RM, DEPTH, GH, false><<<grid, block, lds, st>>>(a.k_cache, a.q, a.k, a.C, G, 0, nullptr, nullptr, \
                                                                          nullptr, a)
  if (rows <= 2 * kWave) LESSDEC_GQS_LAUNCH(2, kFewDepth);
  else if (rows <= 4 * kWave) LESSDEC_GQS_LAUNCH(4, kDepth);
  else LESSDEC_GQS_LAUNCH(kGqsMaxRows / kWave, kDepth);
#undef LESSDEC_GQS_LAUNCH
  return hipGetLastError();
}

template <int D, int RM>
static hipError_t launch_step_gqs_h(const StepArgs &a, int G, hipStream_t st, const MlpPartsArgs *fm)
{
  // Four heads a wave (a row is widened once for them, a stream is a quarter of the rows) where that leaves none idle, or the
  // launch is small.  A step, four against two: 512 units x 4 heads x 400 slots 33.0 and 41.8, 16 x 4 x 204 17.3 and 20.6, 1024 x
  // 4 x 102 at rank 16 32.8 and 35.1, 512 x 8 x 150 33.1 and 36.7; of 3 heads 256 x 102 13.6 and 14.9, 1024 x 60 23.1 and 22.3;
  // 96 x 5 x 150 18.5 and 20.6, 512 x 6 x 102 27.2 and 24.5.  (The one launch has the registers for two, and its shapes
  // take two as two launches as well: the same bits either way.)
  const bool four = !gqs_fusable(D, a.C, a.Rp, a.R, G) && G > 2 && (G % 4 == 0 || (long)a.U * (G > 4 ? 8 : 4) <= kGqsFourWaves);
  return four ? launch_step_gqs_t<D, RM, 4>(a, G, st, fm) : launch_step_gqs_t<D, RM, 2>(a, G, st, fm);
}

hipError_t launch_step_gqs(const StepArgs &a, int G, int D, hipStream_t st, const MlpPartsArgs *fm)
{
  if (fm && !gqs_fusable(D, a.C, a.Rp, a.R, G)) return hipErrorInvalidValue;
  // (Up to rank 8 with that many rows of H and W3: at D = 64 the form for 16 of them holds three waves a SIMD, this one four, without which
  // 1024 units of three heads do not run at once; x 30 slots 19.6 against 15.8 us a step, x 60 20.8 against 17.2.)
  if (D == 64) return a.R <= 8 ? launch_step_gqs_h<64, 8>(a, G, st, fm) : launch_step_gqs_h<64, 16>(a, G, st, fm);
  return a.R <= 8 ? launch_step_gqs_h<128, 8>(a, G, st, fm) : launch_step_gqs_h<128, 16>(a, G, st, fm);
}

}  // namespace lessdec
