// Strip path (kernels_strip.hpp): its tables, its geometry and its launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "batch.hpp"
#include "dispatch.hpp"
#include "kernels_strip.hpp"
#include "plan.hpp"

using namespace sosf;

namespace sosf {

bool strip_supported(const sos_plan_s &p) {
  return p.solver_opt == SOS_AUTO && p.compute_dtype == SOS_F64 && p.L == kL && p.N >= 8 && p.N <= 64 &&
         p.K <= kStripMaxK && p.b0_factored && p.tile_groups == 0 &&
         !(p.flags & (SOS_FLAG_CARRY_SCAN | SOS_FLAG_CARRY_RUNIN));
}

namespace {

#if defined(__x86_64__)
typedef double v4d __attribute__((vector_size(32)));

// (ch, cl) = (hi, lo)^2, block lower triangular, in rows of ld doubles (a multiple
// of 4), each entry an unevaluated sum of two FP64 numbers: the rounding errors of
// the products (by FMA) and of the sums (Knuth's two-sum) are FP64 numbers too, and
// go into the low part.
__attribute__((target("avx2,fma"))) void square_pairs(const double *hi, const double *lo, double *ch, double *cl,
                                                      int D, int ld) {
#pragma clang fp contract(off)
  for (int i = 0; i < D; i += 2)
    for (int j = 0; j < i + 2; j += 4) {
      v4d sh[2] = {}, sl[2] = {};
      for (int k = j; k < i + 2; ++k) {
        v4d bh, bl;
        __builtin_memcpy(&bh, hi + k * ld + j, 32);
        __builtin_memcpy(&bl, lo + k * ld + j, 32);
        for (int r = 0; r < 2; ++r) {
          const double x = hi[(i + r) * ld + k], y = lo[(i + r) * ld + k];
          const v4d ah = {x, x, x, x}, al = {y, y, y, y};
          const v4d p = ah * bh, e = __builtin_elementwise_fma(ah, bh, -p);
          const v4d s = sh[r] + p, t = s - sh[r];
          sl[r] += (ah * bl + al * bh) + (e + ((sh[r] - (s - t)) + (p - t)));
          sh[r] = s;
        }
      }
      for (int r = 0; r < 2; ++r) {
        const v4d h = sh[r] + sl[r], l = sl[r] - (h - sh[r]);
        __builtin_memcpy(ch + (i + r) * ld + j, &h, 32);
        __builtin_memcpy(cl + (i + r) * ld + j, &l, 32);
      }
    }
}
#endif

// phi_pow again, each power the square of the one before in more than FP64
// precision, rounded to FP64 at the end.  The matrices are block lower triangular,
// as in the plan's own products.  Pairs of FP64 numbers where the CPU has FMA: the
// x87 products of one sum wait for each other (K = 16: 120 us of a plan's 345).
void square_powers(sos_plan_s &p) {
  const int D = 2 * p.K;
  std::vector<long double> a(p.phi.begin(), p.phi.end());
  // the one-step transition's last row of each section, from the coefficients
  // (its entries are short sums that FP64 rounds)
  for (int col = 0; col < D; ++col) {
    long double in2 = 0.0L, in1 = 0.0L, now = 0.0L;
    for (int k = 0; k < p.K; ++k) {
      const double *o = &p.rows[5 * k];
      const long double y2 = col == 2 * k ? 1.0L : 0.0L, y1 = col == 2 * k + 1 ? 1.0L : 0.0L;
      const long double yn = o[0] * now + o[1] * in1 + o[2] * in2 - o[3] * y1 - o[4] * y2;
      a[(size_t)(2 * k + 1) * D + col] = yn;
      in2 = y2;
      in1 = y1;
      now = yn;
    }
  }
#if defined(__x86_64__)
  if (__builtin_cpu_supports("avx2") && __builtin_cpu_supports("fma")) {
    const int ld = (D + 3) & ~3;
    std::vector<double> m(4 * (size_t)D * ld, 0.0);
    double *hi = m.data(), *lo = hi + D * ld, *ch = lo + D * ld, *cl = ch + D * ld;
    for (int i = 0; i < D; ++i)
      for (int j = 0; j < D; ++j) {
        hi[i * ld + j] = (double)a[(size_t)i * D + j];
        lo[i * ld + j] = (double)(a[(size_t)i * D + j] - hi[i * ld + j]);
      }
    for (size_t q = 1; q < p.phi_pow.size(); ++q) {
      square_pairs(hi, lo, ch, cl, D, ld);
      std::swap(hi, ch);
      std::swap(lo, cl);
      for (int i = 0; i < D; ++i) std::copy(hi + i * ld, hi + i * ld + D, p.phi_pow[q].begin() + (size_t)i * D);
    }
    return;
  }
#endif
  std::vector<long double> b((size_t)D * D, 0.0L);
  for (size_t q = 1; q < p.phi_pow.size(); ++q) {
    for (int i = 0; i < D; ++i)
      for (int j = 0; j < (i | 1) + 1; ++j) {
        long double sum = 0.0L;
        for (int k = j & ~1; k < (i | 1) + 1; ++k) sum += a[(size_t)i * D + k] * a[(size_t)k * D + j];
        b[(size_t)i * D + j] = sum;
      }
    a.swap(b);
    for (int i = 0; i < D * D; ++i) p.phi_pow[q][i] = (double)a[i];
  }
}

}  // namespace

// Device tables: the state table, the all-pole responses and the padded
// powers of the transition.
//   state table: entry (row i, j) is the response of state value i at a
//     strip's end to the raw input j samples before the end, h_k[j - d] with
//     k = i / 2 and d = 1 for even rows (y[-2]), 0 for odd ones (y[-1]);
//     element e (ascending time) of block b holds j = 16 b + 15 - e; in the
//     order the products read them, [block][row tile][pair][lane][2], lane
//     (i, q) of pair k holding row i, elements 4 q + 2 k and the next;
//   all-pole responses g_k: section k's output to a unit input of the first
//     section's recursive part.  (h_k = g_k + b1 g_k[. - 1] + b2 g_k[. - 2], but
//     that sum cancels digits where the first section's zeros lie near slow poles:
//     FP64, K = 11, poles to r = 0.999: results 1e-10 off where the recurrence
//     itself is 3e-12 off.  So h_k is the whole cascade's own response.)
sos_status upload_strip(sos_plan_s &p) {
  const int K = p.K, D = 2 * K, mt = (D + 15) / 16, R = 16 * mt;
  auto covering = [](int64_t runin) { return (int)std::min<int64_t>((runin + 31) / 32 * 32, kStripMaxSpan); };
  p.strip_span = covering(p.runin);
  p.adj_span = adj_strip_supported(p) ? covering(std::max(p.runin, p.bwd->runin)) : 0;
  const int span = p.strip_rows = std::max(p.strip_span, p.adj_span), gs = span + 16;
  const size_t hop = (size_t)span * R, gsz = (size_t)K * gs, psz = p.phi_pow.size() * (size_t)R * R;
  std::vector<double> t((hop + psz) * (p.adj_span ? 2 : 1) + gsz, 0.0);
  double *g = t.data() + hop, *ph = g + gsz;
  // both responses (g_k, h_k) side by side, every section per sample, so that the
  // sections' recurrences overlap
  typedef double v2d __attribute__((vector_size(16)));
  std::vector<v2d> state(4 * (size_t)K, v2d{0.0, 0.0});   // per section: input x1, x2, output y1, y2
  for (int j = 0; j < gs; ++j) {
    v2d v = j == 0 ? v2d{1.0, 1.0} : v2d{0.0, 0.0};
    const int e = 15 - j % 16;
    double *blk = &t[(size_t)(j / 16) * (16 * R) + ((e % 4 / 2) * 64 + e / 4 * 16) * 2 + e % 2];
    for (int k = 0; k < K; ++k) {
      const double *o = &p.rows[5 * k], on = k > 0 ? 1.0 : 0.0;   // g_0: the first section's recursive part alone
      v2d *z = &state[4 * (size_t)k];
      const v2d x0 = v;
      v = x0 + v2d{on * o[1], o[1]} * z[0] + v2d{on * o[2], o[2]} * z[1];
      z[1] = z[0];
      z[0] = x0;
      v -= o[3] * z[2] + o[4] * z[3];
      if (j < span) {
        double *at = blk + ((2 * k) / 16 * 128 + (2 * k) % 16) * 2;
        at[0] = z[2][1];   // d = 1: h_k[j - 1]
        at[2] = v[1];      // d = 0: h_k[j]
      }
      z[3] = z[2];
      z[2] = v;
      g[(size_t)k * gs + j] = v[0];
    }
  }
  // FP64 I/O: the powers squared in extended precision.  Repeated FP64
  // squaring loses digits that the states then carry through the signal
  // (K = 16, r = 0.99 .. 0.999: results 1.1e-12 off with FP64 powers, 1.4e-13
  // with these, the plain recurrence 6e-14).
  if (p.io_dtype == SOS_F64) square_powers(p);
  for (size_t q = 0; q < p.phi_pow.size(); ++q)
    for (int i = 0; i < D; ++i)
      for (int j = 0; j < D; ++j)   // the A operand's order: [row tile][step][lane]
        ph[q * R * R + (size_t)(i / 16 * 4 * mt + j / 4) * 64 + j % 4 * 16 + i % 16] = p.phi_pow[q][(size_t)i * D + j];
  if (p.adj_span) adj_strip_tables(p, ph + psz, ph + psz + hop);
  if (hipMalloc(&p.d_strip, t.size() * sizeof(double)) != hipSuccess) {
    p.d_strip = nullptr;
    return SOS_E_NOMEM;
  }
  if (hipMemcpy(p.d_strip, t.data(), t.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess)
    return SOS_E_DEVICE;
  p.strip_g = hop;
  p.strip_phi = hop + gsz;
  p.strip_hop_rev = p.strip_phi + psz;
  p.strip_phi_rev = p.strip_hop_rev + hop;
  return SOS_OK;
}

// Strips of len samples over [-shift, n), their start states summed over
// `terms` strips of `span` samples.
void strip_cut(const sos_plan_s &p, int64_t n, int32_t shift, int64_t len, int span, int64_t terms, StripChan &c) {
  const int64_t es = p.io_dtype == SOS_F64 ? 8 : 4;
  const int mt = (2 * p.K + 15) / 16;
  const int64_t area = 16 * mt * 8 / es;   // samples of one state area
  const int64_t rem = (n + shift) % len;
  const int64_t lead = rem > 0 && rem < area ? (area - rem + 31) / 32 * 32 : 0;
  c.tab = static_cast<const double *>(p.d_table);
  c.hop = p.d_strip;
  c.g = p.d_strip + p.strip_g;
  c.phi = p.d_strip + p.strip_phi;
  c.hop_rev = p.d_strip + p.strip_hop_rev;
  c.phi_rev = p.d_strip + p.strip_phi_rev;
  c.off = 0;
  c.n = n;
  c.len = len;
  c.strips = (n + shift + lead + len - 1) / len;
  c.first_item = 0;
  c.K = p.K;
  c.stride = p.stride;
  c.shift = shift;
  c.span = span;
  c.terms = (int32_t)terms;
  c.mt = mt;
  c.gstride = p.strip_rows + 16;
  c.lead = (int32_t)lead;
  c.gain = p.gain;
}

// Whether a cut keeps what the kernels assume, whatever branch chose its length:
// the lead leaves strip 0 a whole state area (with that, strip 1 starts in the
// channel and the channel's first chunk is strip 0's), the last strip holds its
// start state, and where more than 16 strips are summed, every strip a second area.
bool strip_sound(const sos_plan_s &p, const StripChan &c) {
  const int64_t es = p.io_dtype == SOS_F64 ? 8 : 4, V = 16 / es, area = 16 * c.mt * 8 / es;
  const int64_t last = c.n + c.shift + c.lead - (c.strips - 1) * c.len;
  if (c.strips < 1 || last < 1 || last > c.len) return false;
  if (c.strips == 1) return c.lead < c.len;
  return last >= area && c.len - c.lead >= (c.terms > 16 ? V + 2 * area : 32) && c.len >= (c.terms > 16 ? 2 : 1) * area;
}

// Strips of about `len` samples over [-shift, n).
bool strip_geometry(const sos_plan_s &p, int64_t n, int32_t shift, int64_t len, StripChan &c) {
  if (!p.d_strip) return false;
  const int64_t es = p.io_dtype == SOS_F64 ? 8 : 4;
  const int mt = (2 * p.K + 15) / 16;
  // a strip holds two state areas and, strip 0, the lead and the 16 bytes
  // before its first whole ones
  const int64_t area = 16 * mt * 8 / es, areas = 2 * area + 16 / es, least = areas + 32;
  // The state table covers the run-in, so a strip that long needs one term.
  // Shorter ones, at most 2 KB so that a long signal has two wavefronts per
  // SIMD: any multiple of 32 where the kernel makes their transition (FP32 I/O,
  // K <= 8, up to 16 strips' sums), so that every lane has one strip; otherwise
  // powers of two, whose transition is a table entry, down to 7/8 of that
  // rather than twice as many, but not 128 for more than a wavefront per SIMD
  // (1.2e7 FP32 samples, K = 5, r <= 0.999: 128 a strip 68 us, 2e7 in 256: 58;
  // 9e6, K = 8, r <= 0.9: 128 a strip 52, 160: 39).
  const bool covers = p.runin <= p.strip_span && len >= p.strip_span;
  if (covers) {
    // (off the multiples of 2 KB: strips a power of two apart meet in few HBM
    // channels; K = 3 on 2^26 FP32 samples, 1024 a strip: 167 us, 1184: 132).
    // Sections without poles, or with poles near 0, have run-ins shorter than a
    // state area: the lead of up to `area` samples, rounded up to 32, then still
    // has to leave the last strip an area.
    len = (std::max(len, area + 32) + 31) / 32 * 32;
    if (len * es % 2048 == 0) len += 32;
  } else {
    const int64_t most = 2048 / es;
    const int64_t any = (std::max({len, least, (p.runin + 15) / 16}) + 31) / 32 * 32;
    if (p.io_dtype == SOS_F32 && mt == 1 && any <= len + 31 && any < most && any <= p.strip_span &&
        any >> p.phi_pow.size() == 0) {
      len = any;
    } else {
      int64_t l = 32;
      while (2 * l <= len * 8 / 7 || l < least || (l == 128 && len > 128)) l *= 2;
      strip_cut(p, n, shift, l, (int)l, 1, c);
      if (l - c.lead < areas) l *= 2;
      len = std::min(l, most);
    }
    if (len > p.strip_span || len < least || (p.runin + len - 1) / len > kStripMaxTerms) return false;
  }
  strip_cut(p, n, shift, len, (int)(covers ? p.strip_span : len), covers ? 1 : (p.runin + len - 1) / len, c);
  // 32-bit byte offsets, with the strips past the end
  return strip_sound(p, c) && (n + 96 * len) * es < ((int64_t)1 << 32);
}

// Strips for a single signal of n samples, where they beat the tile kernels
// (which N = 16 and 32 shorten, so that odd sizes share out better).  Measured
// against PH (MI355X, us, tiles / strips):
//   poles up to r = 0.999, where the tiles carry by the scan: FP32, K = 8, 2^18
//     41 .. 55 (N = 16 .. 64) / 33, 2^20 43 .. 52 / 35, 9e6 86 .. 107 / 43; K =
//     4, 2^18 29 .. 35 / 29; K = 2, 3e6 28 / 31 (N = 64: 41 / 32), 5e6 34 / 34;
//     K = 12, 4e6 66 / 76 (N = 64), 9e6 126 / 81; K = 16, 3e6 95 / 84; FP64, K =
//     8, 2^18 40 .. 55 / 36; K = 5, r = 0.98, 1.5e6 29 / 31, 2.1e6 38 / 32; K =
//     12, 2^18 58 (N = 16) .. 94 (N = 64) / 62, 2^20 66 / 65;
//   run-ins, FP32, N = 64: K = 5, 1.05e6 25 / 25, 5e6 39 / 28, 2e7 86 / 57; K =
//     4, 1.05e6 24 / 25, 1.5e6 28 / 26; K = 2, 7e6 24 / 26, 9e6 49 / 33; K = 12,
//     2e7 124 / 147, 3.3e7 152 / 125; N = 32: K = 4, 5e6 24 / 26, 9e6 40 / 34;
//     K = 3, 1.6e7 44 / 47, 2e7 59 / 46; N = 16: K = 4, 1.2e7 33 / 40, 1.6e7 48
//     / 47; K = 8, 9e6 41 / 39, 1.2e7 50 / 46; N <= 32, K = 2: 5e7 92 / 101;
//   run-ins, FP64, N = 64: K = 8, 1.5e6 39 / 32, 2^24 + 5 148 / 88; K = 5, 1.05e6
//     28 / 29, 1.5e6 33 / 30, 4e7 204 / 230; K = 3, 1.2e7 64 / 72; K = 12, 2.5e7 182 / 191, 5e7
//     340 / 279; N = 32: K = 8, 9e6 52 / 56, 1.2e7 62 / 58, 4e7 206 / 232; K = 5,
//     1.2e7 53 / 58, 2^24 + 5 91 / 78; N = 16: K = 5, 2^24 + 5 73 / 78.
// With FP32 I/O the tiles keep signals that they share out evenly in powers of
// two, where they are at their best (N = 64, K = 5, 2^22: 22 us against 28; 2^26:
// 175 against 236; 2^28, launch after launch: 611 against 618).
bool strip_single(const sos_plan_s &p, int64_t n, int64_t tile, bool scan, StripChan &c) {
  if (!p.d_strip) return false;
  constexpr int64_t kNever = INT64_MAX;
  const bool f64 = p.io_dtype == SOS_F64, wide = p.N == 64;
  const int K = p.K;
  int64_t least, most = kNever;
  if (scan) {
    if (f64) least = K <= 3 ? (wide ? 3000000 : 5000000) : K <= 6 ? (wide ? 300000 : 2000000) : K <= 8 || wide ? 1 << 18 : 1000000;
    else least = K <= 3 ? (wide ? 3000000 : 5000000) : K <= 8 ? 1 << 18 : K <= 14 ? 7000000 : 3000000;
  } else if (f64) {
    if (wide) least = K <= 4 ? kNever : K <= 8 ? 1400000 : 40000000;
    else least = K <= 4 || K > 8 ? kNever : K > 6 ? 11000000 : p.N == 32 ? 14000000 : kNever;
  } else {
    if (wide) least = K <= 3 ? 8000000 : K <= 4 ? 1400000 : K <= 8 ? 1000000 : 30000000;
    else least = K <= 3 ? 18000000 : K > 8 ? 30000000 : p.N == 32 ? 8000000 : K <= 6 ? 16000000 : 10000000;
  }
  if (f64 && (!wide || K <= 6)) most = 30000000;
  if (!f64 && !wide && K <= 6) most = 40000000;
  if (n < least || n > most) return false;
  // A lone section is bound by memory either way, and the strips' state pass reads
  // x again: all of it where the run-in is longer than the state table.  That pays
  // against tiles that spend several of their lengths on run-ins, and otherwise
  // only where N = 64 shares odd sizes out unevenly (FP32, K = 1, N = 64, run-in
  // 1419, 3.4e7 samples: tiles 72 us, strips 111; 3019, 2.25e8: 417 and 625; N =
  // 32, run-in 161, 2.3e7: 38 and 46; run-in 9005, 2.5e7: 126 and 88.  The means of
  // 8 and 7 such sizes: strips 1.16 and 1.10 times as long).
  if (!f64 && !scan && K == 1 && p.runin < 4000 && (!wide || p.runin > p.strip_span)) return false;
  const int64_t lanes = (int64_t)p.simds * 64, groups = tile / ((int64_t)p.N * p.L);
  if (!f64 && !scan && (groups & (groups - 1)) == 0 && n % (tile * 4 * p.simds) == 0) return false;
  return strip_geometry(p, n, 0, (n + lanes - 1) / lanes, c);
}

namespace {

template <typename TI, int MT>
sos_status launch(const StripArgs &a, int64_t items, int terms, int K, const void *x, void *y, hipStream_t s) {
  const TI *xi = static_cast<const TI *>(x);
  TI *yi = static_cast<TI *>(y);
  const unsigned blocks = (unsigned)((items + kWavesPerBlock - 1) / kWavesPerBlock);
  if (terms == 1)
    hipLaunchKernelGGL((strip_state_kernel<TI, MT, false>), dim3(blocks), dim3(256), 0, s, xi, yi, a);
  else
    hipLaunchKernelGGL((strip_state_kernel<TI, MT, true>), dim3(blocks), dim3(256), 0, s, xi, yi, a);
  if (terms > 16)
    hipLaunchKernelGGL((strip_scan_kernel<TI, MT>), dim3((unsigned)items), dim3(256), 0, s, yi, a);
#define SOSF_STRIP_FILTER(KT)                                                                             \
  hipLaunchKernelGGL((strip_filter_kernel<TI, KT>), dim3(blocks), dim3(256), strip_lds_bytes<TI>(), s, xi, yi, a)
  switch (K) {
    case 1: SOSF_STRIP_FILTER(1); break;
    case 2: SOSF_STRIP_FILTER(2); break;
    case 3: SOSF_STRIP_FILTER(3); break;
    case 4: SOSF_STRIP_FILTER(4); break;
    case 5: SOSF_STRIP_FILTER(5); break;
    case 6: SOSF_STRIP_FILTER(6); break;
    case 7: SOSF_STRIP_FILTER(7); break;
    case 8: SOSF_STRIP_FILTER(8); break;
    default: SOSF_STRIP_FILTER(16); break;
  }
#undef SOSF_STRIP_FILTER
  return hipGetLastError() == hipSuccess ? SOS_OK : SOS_E_DEVICE;
}

}  // namespace

sos_status launch_strip(const sos_plan_s &p, const StripChan &c, const void *x, void *y, hipStream_t s) {
  StripArgs a{};
  a.items = (c.strips + kStripLanes - 1) / kStripLanes;
  a.one = c;
  if (p.io_dtype == SOS_F32)
    return c.mt == 1 ? launch<float, 1>(a, a.items, c.terms, p.K, x, y, s) : launch<float, 2>(a, a.items, c.terms, p.K, x, y, s);
  return c.mt == 1 ? launch<double, 1>(a, a.items, c.terms, p.K, x, y, s) : launch<double, 2>(a, a.items, c.terms, p.K, x, y, s);
}

namespace {

// What a batch's launch takes, in us, by tiles and by strips: fits to 900 random
// batches of 2 .. 1000 channels of 1000 .. 8e6 samples (1e6 .. 1.5e8 in all, K =
// 1 .. 16, N = 8 .. 64, poles to r = 0.9 .. 0.999), each timed both ways on
// MI355X; the ratio of the two is right to 20% (rms).  Tiles: the longest
// tile's chain with its run-in, K (warm + tile), and the tiles' share of a SIMD,
// in 1000 section-samples.  Strips: the filter's longest chain, (K + 5) len; the
// state pass, whose matrix products take as long whatever K, by its longest
// chain and its share of a SIMD; a third of the memory time is the second read;
// the scan's launches where run-ins reach over more than 16 strips; the longest
// chain of a channel that stays with the tiles.
struct BatchCost {
  double base, chain, share, chain8, share8;   // tiles (chain8, share8: more at N = 8)
  double sbase, filter, state, products, rest, scan, memory;
};
constexpr BatchCost kBatchCost[2] = {{10.1, 0.99, 0.89, 0.24, 0.27, 6.3, 6.5, 10.1, 11.7, 1.5, 16.4, 0.6},
                                     {9.4, 1.20, 1.11, 0.42, 0.13, 0.9, 6.3, 16.6, 17.3, 2.7, 11.9, 0.7}};

}  // namespace

// Strips in a batch, where the tiles would spend much of their work on
// run-ins: 64 channels x 2^20 with poles up to r = 0.999 (FP32, K = 8) take
// 382 us by tiles and 203 by strips, while a ragged batch with short run-ins
// (256 channels of 2^10 .. 2^22, K = 1 .. 16, r <= 0.95) is better off with
// the tiles (438 us against 520).  At least 1.5 times the channels' own
// section-samples, and 1.2 times the time that the strips would take: without
// the second line 202 of 557 of those 900 batches lost more than 5% (300 channels
// of 10000 .. 40000 samples, K = 12, r <= 0.9: 58 us by tiles, 87 by strips; one
// of 6e6 samples in 16 channels, K = 1: 19 and 45), with it none of 242 did.
// A wavefront of 64 strips costs about (K + 5) len (a chunk
// that filters nothing takes as long as five sections); the lengths share the
// long channels' work out to two wavefronts per SIMD.  Channels too short for
// 64 strips of a sensible length stay with the tiles.
void strip_schedule(sos_batch_s &b, const sos_plan_t *plans) {
  strip_unschedule(b);
  if (b.block || b.host_only || !b.b0one || b.mix != SOS_PH || b.tile_groups > 0) return;
  constexpr int64_t kLeast = 16384, kLeastTotal = 1 << 22;
  constexpr double kBase = 5.0, kRunIn = 1.5, kGain = 1.2;
  double work = 0.0, own = 0.0, tiles = 0.0, chain = 0.0, share = 0.0;
  int64_t total = 0;
  std::vector<char> takes(b.C, 0);
  std::vector<double> tile_chain(b.C, 0.0);   // 1000 section-samples
  for (int i = 0; i < b.C; ++i) {
    const int c = b.order[i];
    const int64_t items = (i + 1 < b.C ? b.chans[i + 1].first_item : b.items) - b.chans[i].first_item;
    if (items == 0) continue;
    tile_chain[c] = plans[c]->K * 1e-3 *
                    (double)(b.tile[c] + std::min<int64_t>(b.chans[i].warm, (b.n[c] - 1) / b.tile[c] * b.tile[c]));
    chain = std::max(chain, tile_chain[c]);
    share += (double)items * tile_chain[c];
    takes[c] = plans[c]->d_strip && b.n[c] >= kLeast;
    if (!takes[c]) continue;
    tiles += (double)items * (64 / b.L) * 1e3 * tile_chain[c];
    own += (double)b.n[c] * plans[c]->K;
    work += (double)b.n[c] * (plans[c]->K + kBase);
    total += b.n[c];
  }
  if (total < kLeastTotal || tiles < kRunIn * own) return;
  const double simds = plans[0]->simds, quota = work / (2.0 * simds * kStripLanes);   // a lane's share
  const int64_t V = b.io_dtype == SOS_F64 ? 2 : 4;
  std::vector<StripChan> chans;
  std::vector<double> cost;
  double filter = 0.0, state = 0.0, products = 0.0, rest = 0.0;
  bool scan = false;
  for (int c = 0; c < b.C; ++c) {
    if (!takes[c]) {
      rest = std::max(rest, tile_chain[c]);
      continue;
    }
    const int64_t n = b.n[c], want = std::max<int64_t>((int64_t)(quota / (plans[c]->K + kBase)), 64);
    const int64_t w = std::max<int64_t>((n + 64 * want / 2) / (64 * want), 1);   // wavefronts of the channel
    StripChan s{};
    if (!strip_geometry(*plans[c], n, (int32_t)(b.off[c] % V), (n + 64 * w - 1) / (64 * w), s)) {
      takes[c] = 0;
      rest = std::max(rest, tile_chain[c]);
      continue;
    }
    s.off = b.off[c];
    chans.push_back(s);
    cost.push_back((s.K + kBase) * (double)s.len);
    const double mfma = 1e-3 * (double)s.span * s.mt * (s.terms > 1 ? 5 : 4);   // 16-strip tiles of the state pass
    filter = std::max(filter, 1e-3 * cost.back());
    state = std::max(state, mfma);
    products += mfma * (double)((s.strips + kStripLanes - 1) / kStripLanes);
    scan = scan || s.terms > 16;
  }
  if (chans.empty()) return;
  const BatchCost &m = kBatchCost[b.io_dtype == SOS_F64];
  const double by_tiles = m.base + (m.chain + (b.N == 8 ? m.chain8 : 0.0)) * chain +
                          (m.share + (b.N == 8 ? m.share8 : 0.0)) * share / simds;
  const double mb = 1e-6 * (double)b.total * (b.io_dtype == SOS_F64 ? 8 : 4);
  const double by_strips = m.sbase + m.filter * filter + m.state * state + m.products * products / (2.0 * simds) +
                           m.rest * rest + (scan ? m.scan : 0.0) + m.memory * mb;
  if (by_tiles < kGain * by_strips) return;
  // costliest wavefronts first
  std::vector<int32_t> order(chans.size());
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int32_t i, int32_t j) { return cost[i] > cost[j]; });
  for (int32_t i : order) {
    StripChan s = chans[i];
    s.first_item = b.strip_items;
    const int64_t items = (s.strips + kStripLanes - 1) / kStripLanes;
    b.strip_item_chan.insert(b.strip_item_chan.end(), (size_t)items, (int32_t)b.strip_chans.size());
    b.strip_items += items;
    b.strip_scan = b.strip_scan || s.terms > 16;
    b.strip_chans.push_back(s);
  }
  // the tiles keep the other channels' items
  std::vector<int32_t> keep;
  for (int i = 0; i < b.C; ++i) {
    BatchChan &ch = b.chans[i];
    const int64_t first = ch.first_item, end = i + 1 < b.C ? b.chans[i + 1].first_item : b.items;
    ch.first_item = (int64_t)keep.size();
    if (!takes[b.order[i]]) keep.insert(keep.end(), (size_t)(end - first), i);
  }
  b.item_chan.swap(keep);
  b.rows_items = (int64_t)b.item_chan.size();
}

// Every channel back to the tiles.
void strip_unschedule(sos_batch_s &b) {
  if (b.strip_items == 0) return;
  b.strip_items = 0;
  b.strip_scan = false;
  b.strip_chans.clear();
  b.strip_item_chan.clear();
  b.item_chan.clear();
  const int64_t G = (int64_t)b.N * b.L, R = 64 / b.L;
  for (int i = 0; i < b.C; ++i) {
    BatchChan &ch = b.chans[i];
    ch.first_item = (int64_t)b.item_chan.size();
    const int64_t groups = ch.n ? (ch.n + ch.shift + G - 1) / G : 0, tg = ch.tile / G;
    b.item_chan.insert(b.item_chan.end(), (size_t)((groups + R * tg - 1) / (R * tg)), i);
  }
  b.rows_items = (int64_t)b.item_chan.size();
}

namespace {

template <typename TI, int N>
sos_status launch_batched(const sos_batch_s &b, const void *x, void *y, hipStream_t s) {
  const TI *xi = static_cast<const TI *>(x);
  TI *yi = static_cast<TI *>(y);
  StripArgs a{};
  a.chans = b.d_strips;
  a.item_chan = b.d_strip_item;
  a.items_live = b.d_hdr + 2;
  const unsigned blocks = (unsigned)((b.strip_cap + kWavesPerBlock - 1) / kWavesPerBlock);
  // (a batch whose channels all took strips may be replanned to some by tiles)
  const unsigned rows =
      (unsigned)std::max<int64_t>((b.strip_rows_cap + kWavesPerBlock - 1) / kWavesPerBlock, 1);
  hipLaunchKernelGGL((strip_state_batched_kernel<TI>), dim3(blocks), dim3(256), 0, s, xi, yi, a);
  if (b.strip_scan_cap) {
    hipLaunchKernelGGL((strip_scan_kernel<TI, 1>), dim3((unsigned)b.strip_cap), dim3(256), 0, s, yi, a);
    hipLaunchKernelGGL((strip_scan_kernel<TI, 2>), dim3((unsigned)b.strip_cap), dim3(256), 0, s, yi, a);
  }
  const size_t lds = std::max(strip_lds_bytes<TI>(), (size_t)lds_bytes<N, TI, double, kL>(b.kmax_cap));
  hipLaunchKernelGGL((strip_batched_kernel<N, TI>), dim3(rows + blocks), dim3(256), lds, s, xi, yi, b.d_chans,
                     b.d_item_chan, b.d_hdr, (int32_t)b.kmax_cap, a);
  return hipGetLastError() == hipSuccess ? SOS_OK : SOS_E_DEVICE;
}

template <typename TI>
sos_status launch_batched_n(const sos_batch_s &b, const void *x, void *y, hipStream_t s) {
  switch (b.N) {
    case 8: return launch_batched<TI, 8>(b, x, y, s);
    case 16: return launch_batched<TI, 16>(b, x, y, s);
    case 32: return launch_batched<TI, 32>(b, x, y, s);
    case 64: return launch_batched<TI, 64>(b, x, y, s);
    default: return SOS_E_UNSUPPORTED;
  }
}

}  // namespace

sos_status launch_strip_batched(const sos_batch_s &b, const void *x, void *y, hipStream_t s) {
  return b.io_dtype == SOS_F32 ? launch_batched_n<float>(b, x, y, s) : launch_batched_n<double>(b, x, y, s);
}

}  // namespace sosf
