// Host sweep of the strip geometry (csrc/sosfilt_strip.hip): every cut that the
// library would launch keeps what the strip kernels assume.  No GPU: plans are
// host-only, with a placeholder for the device tables.  Prints each violation
// and the number of cuts looked at; exits 1 if there was one.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <vector>

#include "../paper_2607_14054_amd/csrc/batch.hpp"
#include "../paper_2607_14054_amd/csrc/plan.hpp"
#include "../paper_2607_14054_amd/csrc/strip_types.hpp"

using namespace sosf;

namespace {

int64_t looked = 0, bad = 0, shortest = INT64_MAX;

// r = 0: sections without poles
sos_plan_t make(int K, double r, int io, int N) {
  std::vector<double> s;
  for (int k = 0; k < K; ++k) {
    const double th = 0.3 + 2.5 * k / K, ph = 2.9 - 2.3 * k / K;
    const double row[6] = {1.0, -2.0 * std::cos(ph), 1.0, 1.0, -2.0 * r * std::cos(th), r * r};
    s.insert(s.end(), row, row + 6);
  }
  sos_opts o{io, SOS_F64, SOS_AUTO, N, 16, 0, SOS_FLAG_HOST_ONLY};
  sos_plan_t p = nullptr;
  if (create_plan(s.data(), K, &o, false, &p, 0.0) != SOS_OK) std::abort();
  static double placeholder[2];
  p->d_strip = placeholder;
  p->strip_span = p->strip_rows = (int)std::min<int64_t>((p->runin + 31) / 32 * 32, kStripMaxSpan);
  return p;
}

void fail(const char *what, const sos_plan_s &p, const StripChan &c) {
  if (++bad <= 20)
    std::printf("%s: io %d K %d runin %lld n %lld shift %d: len %lld lead %d strips %lld span %d terms %d\n", what,
                p.io_dtype, p.K, (long long)p.runin, (long long)c.n, c.shift, (long long)c.len, c.lead,
                (long long)c.strips, c.span, c.terms);
}

void check(const sos_plan_s &p, const StripChan &c, int64_t runin) {
  ++looked;
  const int64_t es = p.io_dtype == SOS_F64 ? 8 : 4, V = 16 / es, area = 16 * c.mt * 8 / es;
  const int64_t end = c.n + c.shift + c.lead, last = end - (c.strips - 1) * c.len;
  shortest = std::min(shortest, c.len);
  if (c.len % 32 || c.lead % 32 || c.span % 32 || c.span > c.len) fail("granularity", p, c);
  if (c.lead < 0 || c.lead >= c.len) fail("the lead fills strip 0", p, c);
  if (last <= 0 || last > c.len) fail("strip count", p, c);
  if (c.strips > 1 && last < area) fail("no room for the last strip's start state", p, c);
  if (c.strips > 1 && c.len - c.lead - c.shift < 0) fail("strip 1 starts before the signal", p, c);
  if (c.len < (c.terms > 16 ? 2 : 1) * area) fail("no room for a strip's states", p, c);
  if (c.terms > 16 && V + 2 * area > c.len - c.lead) fail("no room for strip 0's sums", p, c);
  if ((c.terms == 1 ? (int64_t)c.span : c.terms * c.len) < runin) fail("run-in not covered", p, c);
  if (c.terms > 1 && c.span != c.len) fail("sums over parts of strips", p, c);
  if ((c.terms > 16 || (c.terms > 1 && (c.mt == 2 || es == 8))) && (c.len & (c.len - 1))) fail("power of two", p, c);
  if ((c.strips + 80) * c.len * es >= (int64_t)1 << 32) fail("32-bit offsets", p, c);
}

// The strip length of a batch's adjoint against every length tried in turn, and
// a set for which that would take 1e9 divisions.
void lengths_of_batches() {
  uint64_t state = 1;
  auto draw = [&](int64_t lo, int64_t hi) {   // log-uniform
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return (int64_t)std::exp(std::log((double)lo) + (double)(state >> 11) / 9007199254740992.0 * std::log((double)hi / lo));
  };
  for (int t = 0; t < 4000; ++t) {
    const int64_t simds = t % 5 ? 1024 : draw(1, 64);
    const int C = t % 7 ? (int)draw(1, 300) : (int)(simds + draw(1, 4) - 2 > 0 ? simds + draw(1, 4) - 2 : 1);
    std::vector<int64_t> n(C);
    int64_t total = 0, longest = 0;
    for (int64_t &v : n) {
      v = draw(64, t % 3 ? 1 << 20 : 1 << 14);
      total += v;
      longest = std::max(longest, v);
    }
    const int64_t got = adj_strip_len(n.data(), C, total, longest, simds);
    int64_t len = std::max<int64_t>(64, (total / (simds * 64) + 31) / 32 * 32);
    for (; len * 64 < longest; len += 32) {
      int64_t waves = 0;
      for (int64_t v : n) waves += (v + 64 * len - 1) / (64 * len);
      if (waves <= simds) break;
    }
    if (got != len && ++bad <= 20)
      std::printf("strip length of %d channels: %lld, in turn %lld\n", C, (long long)got, (long long)len);
  }
  std::vector<int64_t> n(5000, 1000);
  n[7] = (int64_t)1 << 29;
  const auto start = std::chrono::steady_clock::now();
  int64_t sum = 0;
  for (int simds : {1024, 4999, 5000, 5001, 6000, 40000})
    sum += adj_strip_len(n.data(), 5000, n[7] + 4999000, n[7], simds);
  const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - start).count();
  if (s > 0.1 || sum <= 0) {
    ++bad;
    std::printf("strip lengths of 5000 channels took %g s\n", s);
  }
}

// The route of batches timed both ways on MI355X (us by tiles / by strips):
// strips where they gain, and only there.
void routes_of_batches() {
  struct Set {
    int C;
    int64_t lo, hi;
    int K, io, N;
    double r;
    bool strips;
  };
  const Set sets[] = {{16, 191977, 639924, 1, SOS_F32, 32, 0.9, false},      // 19 / 45
                      {265, 11321, 37739, 2, SOS_F32, 64, 0.98, false},      // 36 / 81
                      {300, 10000, 40000, 12, SOS_F32, 32, 0.9, false},      // 58 / 87
                      {99, 3095, 154758, 6, SOS_F64, 32, 0.9, false},        // 48 / 78
                      {54, 247306, 274785, 6, SOS_F32, 32, 0.95, false},     // 63 / 92
                      {64, 1 << 20, 1 << 20, 8, SOS_F32, 32, 0.999, true},   // 382 / 203
                      {13, 586752, 586752, 12, SOS_F32, 8, 0.999, true},     // 939 / 110
                      {40, 103368, 344561, 8, SOS_F64, 16, 0.999, true}};    // 604 / 106
  for (const Set &t : sets) {
    sos_plan_t p = make(t.K, t.r, t.io, t.N);
    std::vector<sos_plan_t> plans(t.C, p);
    std::vector<int64_t> n(t.C);
    for (int c = 0; c < t.C; ++c) n[c] = t.lo + (t.hi - t.lo) * c / t.C;
    sos_batch_opts o{0, SOS_FLAG_HOST_ONLY, 0, 0, 0};
    sos_batch_t b = nullptr;
    if (sos_batch_plan(plans.data(), t.C, n.data(), nullptr, &o, &b) != SOS_OK) std::abort();
    const std::vector<int32_t> tiles = b->item_chan;
    b->host_only = false;   // schedule as a device batch
    strip_schedule(*b, plans.data());
    if ((b->strip_items > 0) != t.strips && ++bad)
      std::printf("%d channels of %lld .. %lld, K %d: %s\n", t.C, (long long)t.lo, (long long)t.hi, t.K,
                  b->strip_items > 0 ? "strips" : "tiles");
    strip_unschedule(*b);
    if ((b->item_chan != tiles || b->rows_items != b->items) && ++bad) std::printf("the tiles' items are not back\n");
    b->host_only = true;
    sos_batch_destroy(b);
  }
}

// Single signals of one section (FP32): strips only with N = 64 and a run-in that
// the state table covers or that takes the tiles several of their lengths.
void routes_of_one_section() {
  struct Signal {
    int K, N;
    double r;
    int64_t n;
    bool strips;
  };
  for (const Signal &t : {Signal{1, 64, 0.99, 225000001, false}, Signal{1, 32, 0.85, 23000001, false},
                          Signal{1, 64, 0.9, 34000001, true}, Signal{1, 64, 0.996, 27000001, true},
                          Signal{1, 32, 0.997, 24700001, true}, Signal{2, 64, 0.99, 33500001, true},
                          Signal{2, 32, 0.9, 31000001, true}}) {
    sos_plan_t p = make(t.K, t.r, SOS_F32, t.N);
    StripChan c;
    if (strip_single(*p, t.n, 3 * 16 * t.N, false, c) != t.strips && ++bad)
      std::printf("K %d N %d run-in %lld n %lld: not %s\n", t.K, t.N, (long long)p->runin, (long long)t.n,
                  t.strips ? "strips" : "tiles");
  }
}

// FP64 plans' powers of the transition, Phi^(2^j), against squares in 113 bits of
// the same one-step transition (64 bits, from the coefficients).  Pairs of FP64
// numbers lose at most 32 * 2^-104 of the summands' size per square, which 13
// squares double to 2^-86, far below the last rounding: half a unit of the largest
// entry, and one for the pairs.  Plain FP64 squares are 2^-53 off at the first.
void powers_of_the_transition() {
  typedef __float128 q;
  for (int K : {1, 3, 8, 12, 15, 16})
    for (double r : {0.3, 0.9, 0.999}) {
      sos_plan_t p = make(K, r, SOS_F64, 32);
      p->d_strip = nullptr;
      (void)upload_strip(*p);   // (the tables' upload itself needs a GPU)
      const int D = 2 * K;
      std::vector<q> a(D * D), b(D * D);
      for (int col = 0; col < D; ++col) {
        long double in2 = 0, in1 = 0, now = 0;
        for (int k = 0; k < K; ++k) {
          const double *o = &p->rows[5 * k];
          const long double y2 = col == 2 * k, y1 = col == 2 * k + 1;
          const long double yn = o[0] * now + o[1] * in1 + o[2] * in2 - o[3] * y1 - o[4] * y2;
          a[2 * k * D + col] = y1;
          a[(2 * k + 1) * D + col] = yn;
          in2 = y2;
          in1 = y1;
          now = yn;
        }
      }
      for (size_t j = 1; j < p->phi_pow.size(); ++j) {
        for (int i = 0; i < D; ++i)
          for (int c = 0; c < D; ++c) {
            q sum = 0;
            for (int k = 0; k < D; ++k) sum += a[i * D + k] * a[k * D + c];
            b[i * D + c] = sum;
          }
        a.swap(b);
        double most = 0, off = 0;
        for (int i = 0; i < D * D; ++i) {
          most = std::max(most, std::fabs((double)a[i]));
          off = std::max(off, std::fabs((double)((q)p->phi_pow[j][i] - a[i])));
        }
        if (!(off <= most * 0x1p-52) && ++bad) std::printf("K %d r %g Phi^(2^%d): %g of %g off\n", K, r, (int)j, off, most);
      }
    }
}

}  // namespace

int main() {
  const double radii[] = {0.0, 0.02, 0.2, 0.3, 0.5, 0.9, 0.98, 0.999};
  for (int io : {SOS_F32, SOS_F64})
    for (int K : {1, 4, 5, 8, 9, 12, 16})
      for (double r : radii) {
        sos_plan_t p = make(K, r, io, 64);
        StripChan c;
        // channels of a batch: any length, any offset, any length of strip
        for (int64_t want : {1, 17, 32, 33, 48, 64, 65, 96, 100, 128, 160, 255, 256, 300, 512, 700, 1024, 1100, 2048})
          for (int64_t base : {(int64_t)16384, (int64_t)40000, (int64_t)1 << 20})
            for (int64_t rem = 0; rem < 2 * std::min<int64_t>(want, 160) + 130; ++rem)
              for (int shift = 0; shift < (io == SOS_F64 ? 2 : 4); ++shift)
                if (strip_geometry(*p, base + rem, shift, want, c)) check(*p, c, p->runin);
        // single signals by the rule, at every remainder around whole strips per lane
        for (int N : {16, 32, 64}) {
          p->N = N;
          const int64_t lanes = (int64_t)p->simds * 64;
          for (int64_t per : {4, 16, 22, 31, 32, 33, 46, 64, 65, 128, 200, 400, 600, 1100})
            for (int64_t d = -130; d <= 130; ++d)
              for (bool scan : {false, true}) {
                const int64_t n = per * lanes + d;
                if (strip_single(*p, n, (int64_t)N * 16 * 3, scan, c)) check(*p, c, p->runin);
              }
        }
        // the adjoint of single signals (FP32, K = 8)
        if (io == SOS_F32 && K == kAdjStripK) {
          p->N = 64;
          p->bwd = make(K, r, io, 16);
          for (double eps = 0x1p-40; eps > 0x1p-50; eps /= 2) p->bwd->runin += p->bwd->runin / 40;
          p->adj_span = (int)std::min<int64_t>((p->bwd->runin + 31) / 32 * 32, kStripMaxSpan);
          p->strip_rows = std::max(p->strip_span, p->adj_span);
          AdjStrip d;
          for (int64_t per : {22, 23, 32, 33, 64, 65, 96, 128, 200, 400, 600, 1100})
            for (int64_t off = -70; off <= 70; ++off)
              if (adj_strip_single(*p, per * p->simds * 64 + off, (size_t)1 << 40, d)) check(*p, d.c, p->bwd->runin);
        }
      }
  lengths_of_batches();
  routes_of_batches();
  routes_of_one_section();
  powers_of_the_transition();
  std::printf("%lld cuts, shortest strip %lld, %lld bad\n", (long long)looked, (long long)shortest, (long long)bad);
  return bad != 0 || looked < 100000;
}
