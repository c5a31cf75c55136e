// The adjoint by strips (FP32 I/O, K = 8, b0 factored): the training step of
// kernels_backward.hpp with one lane per strip of the time axis.
//
// Forward: the strips' start states (adj_strip_state_kernel: strip_state) and
// strip_filter with checkpoints, every section's state at the start of every
// 32 samples (2K doubles, 128 bytes, written like the signal's 128).
// Backward: the states mu_k at every strip's end come from dL/dy as the
// forward's do from x (adj_strip_rev_kernel: strip_state in reversed time), and
// strip_adjoint_kernel then takes the strip's lines from last to first, 16
// samples at a time:
//   * u_k and w_k of the samples from the checkpoint, by the plain recurrences
//     (four FMA per section), four sections' worth held in registers: the
//     lower four sections run once more for it, eleven section passes (and
//     eight over a line's first half, for its second half's states);
//   * per section mu (two FMA), the five sums of the coefficient gradients
//     (five) and lambda (two), the sums kept per lane over the whole strip.
// That is 133 FP64 instructions per sample and no scan over lanes; the tiles'
// adjoint issues 259 per sample, and a run-in per tile.  One wavefront per
// SIMD: 512 registers hold the four sections' signals (160), lambda (32), 40
// sums (80), 16 states (32) and three lines in flight (96).  Bound by FP64
// issue: 72% of a wavefront's cycles issue VALU, 12% wait for LDS and memory.
// Measured (MI355X, us, forward with checkpoints and backward of 64 x 2^18
// samples, r <= 0.95): tiles save 105, adjoint 233; strips start states 25,
// save 38, end states 25, adjoint 121.  One signal of 2^25 + 1001: tiles 127 +
// 520, strips 17 + 78 + 18 + 223.
#pragma once

#include "adjoint_types.hpp"
#include "kernels_strip.hpp"

namespace sosf {

struct AdjStripArgs {
  const AdjStrip *chans;         // batched: channel descriptors; null for a single signal
  const int32_t *item_chan;
  int64_t items;
  const int64_t *hdr;            // batched: the schedule's generation is hdr[1]
  int64_t gen;
  AdjStrip one;
};

__device__ __forceinline__ bool adj_strip_item(const AdjStripArgs &a, int64_t item, AdjStrip &d) {
  if (item >= a.items) return false;
  if (a.chans) {
    if (as_ctab(a.hdr)[1] != a.gen) return false;   // a replay from before a replan writes nothing
    load_desc(d, a.chans + as_ctab(a.item_chan)[item]);
  } else {
    d = a.one;
  }
  return true;
}

// Start states into the first samples of ys's strips (y, or gx as scratch).
template <typename TI>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void adj_strip_state_kernel(const TI *__restrict__ xs,
                                                                                 TI *__restrict__ ys,
                                                                                 AdjStripArgs a) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  AdjStrip d;
  const int64_t item = (int64_t)blockIdx.x * kWavesPerBlock + w;
  if (!adj_strip_item(a, item, d)) return;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kWavesPerBlock * kStripStateLds];
  const int s0 = (int)((item - d.c.first_item) * kStripLanes);
  if (d.c.terms > 1) strip_state<TI, 1, true>(xs, ys, d.c, s0, smem + w * kStripStateLds);
  else strip_state<TI, 1, false>(xs, ys, d.c, s0, smem + w * kStripStateLds);
}

// States at the strips' ends, from dL/dy, into the workspace.
template <typename TI>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void adj_strip_rev_kernel(const TI *__restrict__ gys,
                                                                               double *__restrict__ ws,
                                                                               AdjStripArgs a) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  AdjStrip d;
  const int64_t item = (int64_t)blockIdx.x * kWavesPerBlock + w;
  if (!adj_strip_item(a, item, d)) return;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kWavesPerBlock * kStripStateLds];
  const int s0 = (int)((item - d.c.first_item) * kStripLanes);
  double *rev = ws + d.rev_off;
  if (d.c.terms > 1) strip_state<TI, 1, true, true>(gys, nullptr, d.c, s0, smem + w * kStripStateLds, rev);
  else strip_state<TI, 1, false, true>(gys, nullptr, d.c, s0, smem + w * kStripStateLds, rev);
}

// The forward pass with checkpoints; STORE: y too.
template <typename TI, bool STORE>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void adj_strip_save_kernel(const TI *__restrict__ xs,
                                                                                TI *__restrict__ ys,
                                                                                double *__restrict__ ws,
                                                                                AdjStripArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  AdjStrip d;
  const int64_t item = (int64_t)blockIdx.x * kWavesPerBlock + w;
  if (!adj_strip_item(a, item, d)) return;
  strip_filter<TI, kAdjStripK, true, STORE>(xs, ys, d.c, (item - d.c.first_item) * kStripLanes,
                                            smem + (size_t)w * StripStage<TI>::BYTES,
                                            reinterpret_cast<TI *>(ws + d.ck_off));
}

// One section's adjoint on 16 samples, in place: L = lambda_k on entry and
// lambda_{k-1} on exit; n = (mu[16], mu[17]) on entry and (mu[0], mu[1]) on
// exit; U, W the section's input and output; the sums pair mu of the same
// sample and of one and two samples later with them, as in adjoint_rows.
// t = (b1, b2, a1, a2).
constexpr int kAdjC = 16;
__device__ __forceinline__ void strip_adjoint_section(double (&L)[kAdjC], const double (&t)[4], double (&n)[2],
                                                      const double (&U)[kAdjC], const double (&W)[kAdjC],
                                                      double (&sum)[5]) {
  double m1 = n[0], m2 = n[1];
#pragma unroll
  for (int m = kAdjC - 1; m >= 0; --m) {
    sum[1] = fma_(m1, U[m], sum[1]);
    sum[2] = fma_(m2, U[m], sum[2]);
    sum[3] = fma_(m1, W[m], sum[3]);
    sum[4] = fma_(m2, W[m], sum[4]);
    const double v = fma_(-t[2], m1, fma_(-t[3], m2, L[m]));
    sum[0] = fma_(v, U[m], sum[0]);
    L[m] = v;
    m2 = m1;
    m1 = v;
    if ((m & 3) == 0) __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int m = 0; m < kAdjC; ++m) {
    const double l1 = m + 1 < kAdjC ? L[m + 1] : n[0];
    const double l2 = m + 2 < kAdjC ? L[m + 2] : (m + 2 == kAdjC ? n[0] : n[1]);
    L[m] = fma_(t[1], l2, fma_(t[0], l1, L[m]));
    if ((m & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
  n[0] = m1;
  n[1] = m2;
}

// Sum over the wavefront, in every lane.
__device__ __forceinline__ double wave_total(double v) {
  v += shr<1>(v);
  v += shr<2>(v);
  v += shr<4>(v);
  v += shr<8>(v);   // per row, in its last lane
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  double s = 0.0;
#pragma unroll
  for (int r = 15; r < 64; r += 16) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, r);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), r);
    s += __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
  }
  return s;
}

// LDS per wave: one tile each of x, dL/dy (then dL/dx) and the checkpoints.
template <typename TI>
__host__ __device__ constexpr size_t adj_strip_lds() { return 3 * (size_t)StripStage<TI>::BYTES; }

template <typename TI>
__global__ __launch_bounds__(kWavesPerBlock * 64, 1) void strip_adjoint_kernel(const TI *__restrict__ gys,
                                                                               TI *__restrict__ gxs,
                                                                               const TI *__restrict__ xs,
                                                                               double *__restrict__ ws,
                                                                               AdjStripArgs a) {
  typedef StripStage<TI> St;
  typedef typename St::VT VT;
  constexpr int V = St::V, C = St::C, K = kAdjStripK, SUBS = C / kAdjC, PP = kAdjC / V;   // PP: pieces per 16 samples
  static_assert(sizeof(TI) == 4 && SUBS == 2, "FP32 I/O: 32 samples and K = 8 sections' states per line");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  AdjStrip d;
  const int64_t item = (int64_t)blockIdx.x * kWavesPerBlock + w;
  if (!adj_strip_item(a, item, d)) return;   // uniform per wave
  const StripChan &c = d.c;
  const int lane = lane_id();
  VT *tx = reinterpret_cast<VT *>(smem + (size_t)w * adj_strip_lds<TI>()), *tg = tx + 64 * St::PIECES;
  vd2 *ts = reinterpret_cast<vd2 *>(tg + 64 * St::PIECES);
  const int64_t wave = item - c.first_item, s0 = wave * kStripLanes, s = s0 + lane;
  const __amdgpu_buffer_rsrc_t rx = strip_rsrc(xs, c), rg = strip_rsrc(gys, c), ro = strip_rsrc(gxs, c);
  const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
      ws + d.ck_off, 0, (int)(uint32_t)(((c.n + c.shift) * (int64_t)sizeof(TI) + 127) / 128 * 128), 0x00020000);
  uint32_t at[St::OPS];   // as in strip_filter
#pragma unroll
  for (int j = 0; j < St::OPS; ++j) {
    const int row = j * St::ROWS + lane / St::PIECES;
    at[j] = (uint32_t)((s0 + row) * c.len - c.lead) * (uint32_t)sizeof(TI) +
            16u * (uint32_t)(St::slot(row, lane % St::PIECES) - row * St::PIECES);
  }
  const uint32_t mine = (uint32_t)(s * c.len - c.lead) * (uint32_t)sizeof(TI);   // the lane's strip
  const ctab<double> tab = as_ctab(c.tab);
  double cf[K][4];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j) cf[k][j] = tab[(int64_t)k * c.stride + OFF_B1 + j];
  // mu one and two samples past the strip's end
  double mu[K][2], acc[K][5];
  {
    const bool in = s + 1 < c.strips;
    const double *r = ws + d.rev_off + (in ? s : 0) * 2 * K;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      mu[k][0] = in ? r[2 * (K - 1 - k) + 1] : 0.0;
      mu[k][1] = in ? r[2 * (K - 1 - k)] : 0.0;
#pragma unroll
      for (int j = 0; j < 5; ++j) acc[k][j] = 0.0;
    }
  }
  const int chunks = (int)(c.len / C), head = s0 == 0 && c.shift > 0 ? c.lead / C : -1;   // uniform
  sv4u ix[St::OPS], ig[St::OPS], is[St::OPS];
  typedef float v2f __attribute__((ext_vector_type(2)));
  v2f hist;   // x[t-2], x[t-1] before the chunk
  auto fetch = [&](int ch) {
#pragma unroll
    for (int j = 0; j < St::OPS; ++j) {
      const uint32_t o = at[j] + 128u * (uint32_t)ch;
      ix[j] = __builtin_bit_cast(sv4u, __builtin_amdgcn_raw_buffer_load_b128(rx, o, 0, 0));
      ig[j] = __builtin_bit_cast(sv4u, __builtin_amdgcn_raw_buffer_load_b128(rg, o, 0, 0));
      is[j] = __builtin_bit_cast(sv4u, __builtin_amdgcn_raw_buffer_load_b128(rc, o, 0, 0));
    }
    hist = __builtin_bit_cast(
        v2f, __builtin_amdgcn_raw_buffer_load_b64(rx, mine + 128u * (uint32_t)ch - 2u * (uint32_t)sizeof(TI), 0, 0));
  };
  VT firsts = {};
  auto chunk = [&](int ch) {
#pragma unroll
    for (int j = 0; j < St::OPS; ++j) {
      tx[j * 64 + lane] = __builtin_bit_cast(VT, ix[j]);
      tg[j * 64 + lane] = __builtin_bit_cast(VT, ig[j]);
      reinterpret_cast<VT *>(ts)[j * 64 + lane] = __builtin_bit_cast(VT, is[j]);
    }
    const double h2 = (double)hist[0], h1 = (double)hist[1];
    __builtin_amdgcn_wave_barrier();
    if (ch == head && lane == 0) {
      // the samples before the channel's start are zeros, and so is dL/dy
      // there: the sums multiply mu by them, and a neighbour's NaN by 0 is NaN
      VT v = tx[St::slot(0, 0)], g = tg[St::slot(0, 0)];
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i < c.shift) v[i] = g[i] = TI(0);
      tx[St::slot(0, 0)] = v;
      tg[St::slot(0, 0)] = g;
    }
    __builtin_amdgcn_wave_barrier();
    fetch(ch > 0 ? ch - 1 : 0);
    auto read16 = [&](double (&X)[kAdjC], const VT *tile, int sub) {
#pragma unroll
      for (int p = 0; p < PP; ++p) {
        const VT v = tile[St::slot(lane, sub * PP + p)];
#pragma unroll
        for (int i = 0; i < V; ++i) X[p * V + i] = (double)v[i];
      }
    };
#pragma unroll 1
    for (int sub = SUBS - 1; sub >= 0; --sub) {
      vd2 st[K];   // every section's (y[-2], y[-1]) at the 16 samples' start
#pragma unroll
      for (int k = 0; k < K; ++k) st[k] = ts[St::slot(lane, k)];
      double X[kAdjC], q2 = h2, q1 = h1;
      if (sub > 0) {
        // the chunk's second half starts where the first one ends
        read16(X, tx, 0);
        double p2 = q2, p1 = q1;
        q2 = X[kAdjC - 2];
        q1 = X[kAdjC - 1];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const vd2 y0 = st[k];
          strip_section<kAdjC>(X, cf[k], p2, p1, y0);
          st[k] = vd2{X[kAdjC - 2], X[kAdjC - 1]};
          p2 = y0[0];
          p1 = y0[1];
        }
      }
      // the upper four sections' signals: u_4 from the lower four, then held
      double T[5][kAdjC];
      read16(T[0], tx, sub);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        strip_section<kAdjC>(T[0], cf[k], k ? st[k - 1][0] : q2, k ? st[k - 1][1] : q1, st[k]);
#pragma unroll
      for (int k = 4; k < 8; ++k) {
#pragma unroll
        for (int m = 0; m < kAdjC; ++m) T[k - 3][m] = T[k - 4][m];
        strip_section<kAdjC>(T[k - 3], cf[k], st[k - 1][0], st[k - 1][1], st[k]);
      }
      double L[kAdjC];
      read16(L, tg, sub);
#pragma unroll
      for (int k = 7; k >= 4; --k) strip_adjoint_section(L, cf[k], mu[k], T[k - 4], T[k - 3], acc[k]);
      // the lower four: u_0 .. u_3 again, u_4 is still there
#pragma unroll
      for (int m = 0; m < kAdjC; ++m) T[4][m] = T[0][m];
      read16(T[0], tx, sub);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int m = 0; m < kAdjC; ++m) T[k + 1][m] = T[k][m];
        strip_section<kAdjC>(T[k + 1], cf[k], k ? st[k - 1][0] : q2, k ? st[k - 1][1] : q1, st[k]);
      }
#pragma unroll
      for (int k = 3; k >= 0; --k) strip_adjoint_section(L, cf[k], mu[k], T[k], T[k + 1], acc[k]);
      // dL/dx in dL/dy's place
#pragma unroll
      for (int p = 0; p < PP; ++p) {
        VT v;
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = (TI)(L[p * V + i] * c.gain);
        tg[St::slot(lane, sub * PP + p)] = v;
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (ch == head) firsts = tg[St::slot(0, 0)];
#pragma unroll
    for (int j = 0; j < St::OPS; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(sv4u, tg[j * 64 + lane]), ro,
                                             ch == head && j == 0 && lane == 0 ? 0xffffff00u : at[j] + 128u * (uint32_t)ch,
                                             0, 0);
    __builtin_amdgcn_wave_barrier();
  };
  fetch(chunks - 1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < St::OPS; ++j)
    __builtin_amdgcn_raw_buffer_store_b128(sv4u{0, 0, 0, 0}, ro, 0xfffffc00u + 16 * j, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  int ch = chunks - 1;
  do chunk(ch); while (--ch >= 0);
  if (head >= 0 && lane < V && lane >= c.shift && lane - c.shift < c.n) {
    TI v = firsts[0];
#pragma unroll
    for (int i = 1; i < V; ++i)
      if (lane == i) v = firsts[i];
    gxs[c.off + lane - c.shift] = v;
  }
  // the strips' sums, scaled as in adjoint_rows: u_k and w_k are in the
  // scaled domain, mu_k is divided by the product of b0 over the sections
  // after k
  const ctab<double> cb = as_ctab(d.bwd);
  double *part = ws + d.part_off;
  double p = 1.0;
#pragma unroll
  for (int k = K - 1; k >= 0; --k) {
    const double su = (k > 0 ? cb[kBwdRow * (k - 1) + BW_SCALE] : 1.0) * p, sw = cb[kBwdRow * k + BW_SCALE] * p;
    p *= cb[kBwdRow * k + BW_B0];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const double v = wave_total(acc[k][j]) * (j < 3 ? su : sw);
      if (lane == 0) part[((int64_t)k * d.waves + wave) * 5 + j] = v;
    }
  }
}

}  // namespace sosf
