// The adjoint by strips (kernels_strip_adjoint.hpp): its tables, its geometry
// and its launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "batch.hpp"
#include "dispatch.hpp"
#include "kernels_strip_adjoint.hpp"
#include "plan.hpp"

using namespace sosf;

namespace sosf {

// FP32 I/O, K = 8: a line of signal (128 bytes, 32 samples) and a line of
// states (2K doubles) are then the same size, and the recompute mode's
// workspace has room for the lines.  (FP64 I/O: 16 samples a line, and the
// kernel's values no longer fit 512 registers.)
bool adj_strip_supported(const sos_plan_s &p) {
  return p.bwd && p.bwd->b0_factored && p.io_dtype == SOS_F32 && p.K == kAdjStripK && strip_supported(p) &&
         !(p.flags & (SOS_FLAG_ADJ_SAVE | SOS_FLAG_ADJ_RECOMPUTE)) && adjoint_recompute(p);
}

// The tables in reversed time: state q, q = K - 1 - k, is section k's (mu[t+1],
// mu[t]) at a strip's first sample t.  The layouts are upload_strip's.  Section
// q runs mu = in - a1 mu[+1] - a2 mu[+2] and hands mu + b1 mu[+1] + b2 mu[+2]
// on.
void adj_strip_tables(const sos_plan_s &p, double *hop, double *phi) {
  constexpr int K = kAdjStripK, D = 2 * K;
  // one sample of the cascade: z = (mu[+2], mu[+1]) per section, m the new mu
  auto step = [&](const double *z, double in, double *m) {
    for (int q = 0; q < K; ++q) {
      const double *o = &p.rows[5 * (size_t)(K - 1 - q)];
      m[q] = in - o[3] * z[2 * q + 1] - o[4] * z[2 * q];
      in = m[q] + o[1] * z[2 * q + 1] + o[2] * z[2 * q];
    }
  };
  double z[D] = {}, m[K];
  for (int j = 0; j < p.strip_rows; ++j) {
    double *blk = hop + (size_t)(j / 16) * (16 * D);
    const int e = j % 16;
    step(z, j == 0 ? 1.0 : 0.0, m);
    for (int q = 0; q < K; ++q) {
      double *at = blk + (((e % 4 / 2) * 64 + e / 4 * 16 + 2 * q) * 2 + e % 2);
      at[0] = z[2 * q + 1];   // response j - 1 (mu[t+1])
      at[2] = m[q];           // response j (mu[t])
      z[2 * q] = z[2 * q + 1];
      z[2 * q + 1] = m[q];
    }
  }
  double a[D][D] = {}, b[D][D];
  for (int col = 0; col < D; ++col) {
    double unit[D] = {};
    unit[col] = 1.0;
    step(unit, 0.0, m);
    for (int q = 0; q < K; ++q) {
      a[2 * q][col] = unit[2 * q + 1];
      a[2 * q + 1][col] = m[q];
    }
  }
  for (size_t w = 0; w < p.phi_pow.size(); ++w) {
    for (int i = 0; i < D; ++i)
      for (int j = 0; j < D; ++j) phi[w * D * D + (size_t)(j / 4) * 64 + j % 4 * 16 + i] = a[i][j];
    // block lower triangular, as square_powers
    for (int i = 0; i < D; ++i) {
      for (int j = 0; j < D; ++j) b[i][j] = 0.0;
      for (int k = 0; k < (i | 1) + 1; ++k)
        for (int j = 0; j < D; ++j) b[i][j] += a[i][k] * a[k][j];
    }
    std::copy(&b[0][0], &b[0][0] + D * D, &a[0][0]);
  }
}

namespace {

// A state area is 32 samples, and the lead that makes room for one in the last
// strip as many: shorter strips have no room for both.
constexpr int64_t kLeastLen = 64;
constexpr int64_t kAdjLeastTotal = 1500000;   // samples (adj_strip_pays)

// Strips of about `len` samples and their regions from `base` on, in doubles;
// false where the run-in needs more than 16 strips or the regions `room`.
bool adj_strip_geometry(const sos_plan_s &p, int64_t n, int32_t shift, int64_t len, int64_t base, int64_t room,
                        AdjStrip &d) {
  const int64_t runin = std::max(p.runin, p.bwd->runin);
  len = (std::max({len, kLeastLen, (runin + 15) / 16}) + 31) / 32 * 32;   // the sums reach over 16 strips
  if (runin > (int64_t)1 << p.phi_pow.size()) return false;   // the powers that the sums over strips take
  if (runin <= p.adj_span && len >= p.adj_span) {
    if (len % 512 == 0) len += 32;   // off the multiples of 2 KB, as in strip_geometry
    strip_cut(p, n, shift, len, p.adj_span, 1, d.c);
  } else {
    len = std::min<int64_t>(len, p.strip_rows);
    const int64_t terms = (runin + len - 1) / len;
    if (len < kLeastLen || terms > 16 || len >> p.phi_pow.size()) return false;
    strip_cut(p, n, shift, len, (int)len, std::max<int64_t>(terms, 2), d.c);
  }
  d.bwd = static_cast<const double *>(p.d_bwd_rows);
  d.waves = (d.c.strips + kStripLanes - 1) / kStripLanes;
  d.ck_off = base;
  d.rev_off = base + (n + shift + 31) / 32 * (2 * kAdjStripK);
  d.part_off = d.rev_off + d.c.strips * 2 * kAdjStripK;
  return strip_sound(p, d.c) && d.part_off + 5 * kAdjStripK * d.waves <= base + room &&
         (n + 96 * len) * 4 < ((int64_t)1 << 32);
}

// Whether `waves` wavefronts of strips of up to `len` samples beat the tiles
// over `total` samples.  The strips take about 45 us and 0.53 us per sample of
// the longest strip in every round of one wavefront per SIMD, whatever the
// lanes left idle; what the tiles take grows with the run-in.  sos_filt_backward
// (MI355X, us, tiles / strips): r <= 0.95, 2^20 samples 60 / 69, 1.5e6 74 / 69,
// 2^22 110 / 81, 2^24 270 / 187, 2^26 894 / 591; r <= 0.99, 2^21 147 / 102, 2^24
// 364 / 187; r <= 0.998, 1.5e6 281 / 198, 2^23 440 / 207.  Batches, both passes:
// 100 x 16000 r <= 0.95 234 / 83, r <= 0.99 636 / 178; 3000 x 1000 r <= 0.95 242
// / 220 (idle lanes: the ratio of the rounds' samples to the signals' is 4);
// 64 x 2^18 356 / 245.
bool adj_strip_pays(const sos_plan_s &p, int64_t runin, int64_t total, int64_t waves, int64_t len) {
  const int64_t rounds = (waves + p.simds - 1) / p.simds;
  return total >= kAdjLeastTotal && (double)(rounds * p.simds * kStripLanes * len) <= (double)total * (5.0 + runin / 256.0);
}

template <typename F>
sos_status launch_steps(bool forward, bool adjoint, int64_t items, const AdjStripArgs &a, const float *x, float *y,
                        const float *gy, float *gx, double *ws, hipStream_t s) {
  const dim3 blocks((unsigned)((items + kWavesPerBlock - 1) / kWavesPerBlock)), threads(kWavesPerBlock * 64);
  if (forward) {
    // the start states travel in the output, or in dL/dx before it is written
    hipLaunchKernelGGL(adj_strip_state_kernel<F>, blocks, threads, 0, s, x, y ? y : gx, a);
    if (y)
      hipLaunchKernelGGL((adj_strip_save_kernel<F, true>), blocks, threads, strip_lds_bytes<F>(), s, x, y, ws, a);
    else
      hipLaunchKernelGGL((adj_strip_save_kernel<F, false>), blocks, threads, strip_lds_bytes<F>(), s, x, gx, ws, a);
  }
  if (adjoint) {
    hipLaunchKernelGGL(adj_strip_rev_kernel<F>, blocks, threads, 0, s, gy, ws, a);
    hipLaunchKernelGGL(strip_adjoint_kernel<F>, blocks, threads, kWavesPerBlock * adj_strip_lds<F>(), s, gy, gx, x, ws,
                       a);
  }
  return hipGetLastError() == hipSuccess ? SOS_OK : SOS_E_DEVICE;
}

}  // namespace

bool adj_strip_single(const sos_plan_s &p, int64_t n, size_t room, AdjStrip &d) {
  if (!p.adj_span) return false;
  const int64_t lanes = (int64_t)p.simds * kStripLanes;
  return adj_strip_geometry(p, n, 0, (n + lanes - 1) / lanes, 0, (int64_t)(room / sizeof(double)), d) &&
         adj_strip_pays(p, p.bwd->runin, n, d.waves, d.c.len);
}

sos_status launch_adj_strip(bool forward, bool adjoint, const sos_plan_s &p, const AdjStrip &d, const void *x, void *y,
                            const void *gy, void *gx, double *ws, hipStream_t s) {
  (void)p;
  AdjStripArgs a{};
  a.items = d.waves;
  a.one = d;
  return launch_steps<float>(forward, adjoint, a.items, a, static_cast<const float *>(x), static_cast<float *>(y),
                             static_cast<const float *>(gy), static_cast<float *>(gx), ws, s);
}

// The shortest strips, a multiple of 32 samples from the channels' even share
// on, for which a wavefront per SIMD serves every channel; at most a wavefront
// for the longest.  Bisection: the channels' wavefronts, sum ceil(n / 64 len),
// fall with len and are at least C and at most total / (64 len) + C, so a set of
// more channels than SIMDs needs none, and one of few channels a step or two.  (A
// serving loop replans on every request: 3000 channels, the longest 2^23 samples,
// 15.5 ms with every length tried in turn, 0.7 ms so.)
int64_t adj_strip_len(const int64_t *n, int C, int64_t total, int64_t longest, int64_t simds) {
  const int64_t first = std::max(kLeastLen, (total / (simds * kStripLanes) + 31) / 32 * 32);
  auto up = [&](int64_t len) { return len <= first ? 0 : (len - first + 31) / 32; };   // steps of 32 from the first
  int64_t lo = 0, hi = up((longest + kStripLanes - 1) / kStripLanes);
  if (C < simds) hi = std::min(hi, up(total / (kStripLanes * (simds - C)) + 1));
  else lo = C > simds ? hi : 0;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2, per = kStripLanes * (first + 32 * mid);
    int64_t waves = 0;
    for (int c = 0; c < C && waves <= simds; ++c) waves += (n[c] + per - 1) / per;
    if (waves <= simds) hi = mid;
    else lo = mid + 1;
  }
  return first + 32 * lo;
}

// Every channel of a batch by strips, or none (the tiles and the strips would
// run one after the other).
void adj_strip_schedule(sos_batch_s &b, const sos_plan_t *plans) {
  if (!b.adj_rc) return;
  int64_t total = 0, runin = 0;
  int longest = 0;   // place in the launch order
  for (int i = 0; i < b.C; ++i) {
    const int32_t c = b.order[i];
    if (!plans[c]->adj_span || b.n[c] < kLeastLen) return;
    total += b.n[c];
    if (b.n[c] > b.n[b.order[longest]]) longest = i;
    runin = std::max(runin, plans[c]->bwd->runin);
  }
  if (total < kAdjLeastTotal) return;
  const int64_t simds = plans[0]->simds;
  const int64_t len = adj_strip_len(b.n.data(), b.C, total, b.n[b.order[longest]], simds);
  auto cut = [&](int i, AdjStrip &d) {
    const int32_t c = b.order[i];
    const AdjChan &t = b.adj_chans[i];
    const int64_t w = (b.n[c] + kStripLanes * len - 1) / (kStripLanes * len), per = kStripLanes * w;
    return adj_strip_geometry(*plans[c], b.n[c], (int32_t)(b.off[c] % 4), (b.n[c] + per - 1) / per, t.saved_off,
                              t.partial_off - t.saved_off, d);
  };
  // the longest channel's strips alone tell most sets that do not gain
  AdjStrip one;
  if (!cut(longest, one) || !adj_strip_pays(*plans[0], runin, total, one.waves, one.c.len)) return;
  std::vector<AdjStrip> strips(b.C);
  std::vector<int32_t> items;
  for (int i = 0; i < b.C; ++i) {
    AdjStrip &d = strips[i];
    if (!cut(i, d)) return;
    d.c.off = b.off[b.order[i]];
    d.c.first_item = (int64_t)items.size();
    items.insert(items.end(), (size_t)d.waves, i);
  }
  int64_t most = 0;
  for (const AdjStrip &d : strips) most = std::max(most, d.c.len);
  if ((int64_t)items.size() > b.adj_strip_room ||
      !adj_strip_pays(*plans[0], runin, total, (int64_t)items.size(), most))
    return;
  for (int i = 0; i < b.C; ++i) {   // the reduction's view
    b.adj_chans[i].partial_off = strips[i].part_off;
    b.adj_chans[i].ntiles = strips[i].waves;
  }
  b.adj_strip_items = (int64_t)items.size();
  b.adj_strips = std::move(strips);
  b.adj_item_chan = std::move(items);
}

sos_status launch_adj_strip_batched(bool forward, bool adjoint, const sos_batch_s &b, const void *x, void *y,
                                    const void *gy, void *gx, double *ws, hipStream_t s) {
  AdjStripArgs a{};
  a.chans = b.d_adj_strips;
  a.item_chan = b.d_adj_item;
  a.items = b.adj_strip_items;
  a.hdr = b.d_hdr;
  a.gen = b.gen;
  return launch_steps<float>(forward, adjoint, a.items, a, static_cast<const float *>(x), static_cast<float *>(y),
                             static_cast<const float *>(gy), static_cast<float *>(gx), ws, s);
}

}  // namespace sosf
