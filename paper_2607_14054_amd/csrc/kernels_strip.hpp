// Strip kernels: long signals with one lane per strip of the time axis.
//
// A lane filters its own strip with the plain recurrences of Section II, all
// K sections on 32 samples at a time in registers: four FP64 FMA per section
// and sample, where a group shared by a row of lanes needs six (PH's
// homogeneous correction) and the row scans.  What a lane needs for that is
// the cascade's state at its strip's start, which is a sum over the samples
// before it (h_k: the response of section k's output to the raw input),
//   y_k[t-1-d] = sum_j h_k[j] x[t-1-d-j],  d = 0, 1.
// For all 2K state values of 16 strips at once that is a matrix product, and
// it runs on the FP64 matrix cores before the filter pass:
//   1. strip_state_kernel: the end state c_s of every strip from zero
//      section states.  Where the strip is at least as long as the run-in W
//      only its last W samples count, and c_s is the next strip's state.
//   2. strip_scan_kernel, where the strip is shorter than W: with Phi the
//      cascade's one-step transition (zero raw input) and R = ceil(W / T),
//      S_s = c_{s-1} + Phi^T (c_{s-2} + Phi^T (... c_{s-R})).
//   3. strip_filter_kernel: every strip from S_s, storing its outputs.
// The states travel in y itself: a strip's first output samples hold S_s,
// then c_s, until the filter pass, which reads S_s before it stores (each
// wavefront reads and writes only its own strips there).  So the path needs
// no workspace.
#pragma once

#include "kernels.hpp"
#include "strip_types.hpp"

namespace sosf {

typedef double sv4d __attribute__((ext_vector_type(4)));

struct StripArgs {
  const StripChan *chans;        // batched: channel descriptors; null for a single signal
  const int32_t *item_chan;      // batched: work item -> channel
  const int64_t *items_live;     // batched: live work items
  int64_t items;                 // single signal: work items
  StripChan one;                 // single signal
};

// A descriptor, through the constant address space, so that its fields arrive
// in scalar registers.
template <typename T>
__device__ __forceinline__ void load_desc(T &d, const T *src) {
  const ctab<uint64_t> p = as_ctab(reinterpret_cast<const uint64_t *>(src));
  uint64_t raw[sizeof(T) / 8];
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 8); ++i) raw[i] = p[i];
  __builtin_memcpy(&d, raw, sizeof(d));
}

// The channel and the strip range of a work item (64 strips); false past the
// last item (uniform per wave).
__device__ __forceinline__ bool strip_item(const StripArgs &a, int64_t item, StripChan &c) {
  if (a.chans) {
    if (item >= as_ctab(a.items_live)[0]) return false;
    load_desc(c, a.chans + as_ctab(a.item_chan)[item]);
  } else {
    if (item >= a.items) return false;
    c = a.one;
  }
  return true;
}

// A global-memory pointer: the tables' addresses come out of a descriptor, and
// without this their loads would be flat ones, whose waits drain every other
// load in flight.
template <typename T>
using gptr = const __attribute__((address_space(1))) T *;

// Doubles of one state area in y (S_s, then c_s at the strip's start).
__host__ __device__ constexpr int strip_state_elems(int mt) { return 16 * mt; }
// First sample of a strip's state areas, relative to the channel's start (a
// multiple of 16 bytes from y).
template <typename TI>
__device__ __forceinline__ int64_t strip_slot(const StripChan &c, int64_t s) {
  const int64_t t0 = s * c.len - c.lead - c.shift;
  return t0 < 0 ? Vec16<TI>::n - c.shift : t0;
}

typedef uint32_t sv4u __attribute__((ext_vector_type(4)));

// A raw buffer over the channel from the 16-byte boundary at or before its
// start (byte 0 is sample -shift).  Loads outside it return zeros, dword by
// dword, and stores there are dropped.
template <typename TI>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t strip_rsrc(const TI *p, const StripChan &c) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<TI *>(p + (c.off - c.shift)), 0,
                                           (int)(uint32_t)((c.n + c.shift) * (int64_t)sizeof(TI)), 0x00020000);
}

// 128 bytes of each strip (32 samples, FP64: 16) move between HBM and the
// lanes through a per-wave LDS tile of one row per strip.  Global accesses
// are 16-byte vectors, the 8 lanes of a strip covering its line; the 16-byte
// pieces of a row are permuted by the strip's index so that the 16 lanes that
// read or write the same piece of their rows fall on distinct banks.
template <typename TI>
struct StripStage {
  typedef typename Vec16<TI>::type VT;
  static constexpr int V = Vec16<TI>::n;
  static constexpr int C = 128 / (int)sizeof(TI);    // samples per chunk: a 128-byte line per strip
  static constexpr int PIECES = C / V;               // 16-byte pieces per row
  static constexpr int ROWS = 64 / PIECES;           // rows per wave-wide access
  static constexpr int OPS = PIECES;                 // accesses per tile
  static constexpr int BYTES = 64 * 128;
  static __device__ __forceinline__ int slot(int s, int p) { return s * PIECES + (p ^ ((s >> 1) & 7)); }
};

// Rotates a value d lanes up inside its 16-lane row (d = 1 .. 15).
template <int D>
__device__ __forceinline__ double row_ror(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + D, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x120 + D, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One doubling round over the wavefront's strips: v_s += P v_{s-D}, P the
// transition over D strips (A operand layout).  Strips before the first tile
// count as zero.  REV: v_s += P v_{s+D}, zero past the last tile.
template <int D, int NT, int MT, bool REV>
__device__ __forceinline__ void strip_round(sv4d (&v)[NT][MT], const double (&P)[MT][4 * MT], int i) {
  double sh[NT][MT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        constexpr int ROT = REV ? 16 - D : D;
        const int u = REV ? t + 1 : t - 1;   // the tile that shifts in
        const bool in = REV ? u < NT : u >= 0;
        const double cur = row_ror<ROT>(v[t][m][r]), next = in ? row_ror<ROT>(v[in ? u : t][m][r]) : 0.0;
        sh[t][m][r] = (REV ? i >= 16 - D : i < D) ? next : cur;
      }
#pragma unroll
  for (int k = 0; k < 4 * MT; ++k)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        v[t][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(P[m][k], sh[t][k / 4][k % 4], v[t][m], 0, 0, 0);
}

// Phi^(2^j), padded, in the A operand's layout (as the table holds it).
template <int MT>
__device__ __forceinline__ void strip_power(double (&P)[MT][4 * MT], const double *__restrict__ phi, int j) {
  const gptr<double> f = (gptr<double>)(phi + (int64_t)j * (256 * MT * MT) + lane_id());
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int k = 0; k < 4 * MT; ++k) P[m][k] = f[(m * 4 * MT + k) * 64];
}

// P[j] = Phi^(len 2^j), j < 4, of a 16-row state for any len: the product of
// the powers in len's bits, then squares.  D's layout of F^T G^T is the A
// operand's of G F, and the A operand's layout of M is the B operand's of M^T,
// so both P (M) and its transpose (Mt) are kept in the A operand's layout.
__device__ __forceinline__ void strip_transitions(double (&P)[4][1][4], const double *__restrict__ phi, int len) {
  const int lane = lane_id(), i = lane & 15, q = lane >> 4;
  double M[4], Mt[4];
  auto product = [&](const double (&A)[4], const double (&B)[4], double (&R)[4]) {
    sv4d r = sv4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k) r = __builtin_amdgcn_mfma_f64_16x16x4f64(A[k], B[k], r, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) R[k] = r[k];
  };
  bool have = false;
  for (int bits = len, j = 0; bits; bits >>= 1, ++j) {
    if (!(bits & 1)) continue;
    const gptr<double> f = (gptr<double>)(phi + (int64_t)j * 256);
    double F[4], Ft[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      F[k] = f[k * 64 + lane];                                     // F[i][4 k + q]
      Ft[k] = f[(i >> 2) * 64 + (i & 3) * 16 + 4 * k + q];         // F[4 k + q][i]
    }
    if (!have) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        M[k] = F[k];
        Mt[k] = Ft[k];
      }
      have = true;
    } else {
      double a[4], b[4];
      product(Ft, M, a);   // M F
      product(M, Ft, b);   // its transpose
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        M[k] = a[k];
        Mt[k] = b[k];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int k = 0; k < 4; ++k) P[j][0][k] = M[k];
    if (j == 3) break;
    double a[4], b[4];
    product(Mt, M, a);
    product(M, Mt, b);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      M[k] = a[k];
      Mt[k] = b[k];
    }
  }
}

// Start states of 64 strips per wavefront, in 16-strip tiles.  MFMA operands
// (16x16x4): A lane (i, q) = row i, inner index q; B lane (j, q) = strip j;
// D register r, lane (j, q) = row 4 r + q.  The inner dimension is time; the
// order of the samples in it is free, so that each lane loads four
// consecutive samples (element e of the four lanes q of a strip make one
// product step) and the table is laid out to match.
//
// SCAN (strips shorter than the run-in; len is 2^lg, or for MT = 1 and up to 16
// strips' sums any multiple of 32, see strip_transitions): the end states of the
// 16 strips before come along as one more tile, and log2 doubling rounds
// make every end state the sum over up to 16 strips; the product's output
// layout is the next product's input layout, so that the states stay in
// registers.  With more than 16 terms those sums go to strip_scan_kernel.
//
// The matrix cores take 64 cycles per product and SIMD: at 5 tiles and 32
// samples per step a step lasts 2560 cycles (MT = 1), which is what the next
// step's loads have to arrive.
//
// REV: the adjoint's states (kernels_strip_adjoint.hpp), in reversed time.
// The window is the strip's first samples, the sum up to strip s + 1 the state
// at the end of strip s; it goes to `rev`, 2K values per strip.
template <typename TI, int MT, bool SCAN, bool REV = false>
__device__ __forceinline__ void strip_state(const TI *__restrict__ xs, TI *__restrict__ ys, const StripChan &c,
                                            int s0, unsigned char *lds, double *__restrict__ rev = nullptr) {
  constexpr int T0 = SCAN && !REV ? 1 : 0;   // the first tile of the wavefront's own strips
  typedef StripStage<TI> St;
  typedef typename St::VT VT;
  constexpr int H = SCAN ? 1 : 0, NT = 4 + H, V = St::V, XP = 4 / V;
  constexpr int U = 8 / (int)sizeof(TI);   // 16-sample blocks per step: a 128-byte line per strip
  constexpr int OPS = 16 * NT / St::ROWS;  // accesses per step
  const int lane = lane_id(), i = lane & 15, q = lane >> 4;
  const __amdgpu_buffer_rsrc_t rx = strip_rsrc(xs, c);
  const int es = (int)sizeof(TI), len = (int)c.len;
  // byte offset of the lane's piece of op j (strips before the channel wrap
  // past the buffer's end: zeros)
  VT *stage = reinterpret_cast<VT *>(lds);
  uint32_t at[OPS];
#pragma unroll
  for (int j = 0; j < OPS; ++j) {
    const int row = j * St::ROWS + lane / St::PIECES;
    at[j] = (uint32_t)((s0 - 16 * T0 + row) * len - c.lead + (REV ? 0 : len - c.span)) * (uint32_t)es +
            16u * (uint32_t)(St::slot(row, lane % St::PIECES) - row * St::PIECES);
  }
  sv4d acc[NT][MT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[t][m] = sv4d{0.0, 0.0, 0.0, 0.0};
  const int blocks = c.span / kStripBlock;
  const gptr<vd2> hp = (gptr<vd2>)(REV ? c.hop_rev : c.hop) + (REV ? 0 : (int64_t)(blocks - 1) * (MT * 128)) + lane;
  struct Step {
    sv4u in[OPS];
    vd2 h[MT][U][2];
  };
  auto fetch = [&](Step &f, int n) {
#pragma unroll
    for (int j = 0; j < OPS; ++j)
      f.in[j] = __builtin_bit_cast(sv4u, __builtin_amdgcn_raw_buffer_load_b128(rx, at[j] + 128u * (uint32_t)n, 0, 0));
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < 2; ++k) f.h[m][u][k] = hp[(m * 2 + k) * 64 + (REV ? 1 : -1) * (int64_t)(U * n + u) * (MT * 128)];
  };
  // the step of strip 0 that starts with the channel's start: the samples
  // before it in the same 16 bytes are zeros
  // (REV: nothing needs strip 0's sums)
  const int head = !REV && s0 == 0 && c.shift > 0 ? (c.lead - (len - c.span)) / (16 * U) : -1;   // uniform
  // Through the tile, so that adjacent lanes load adjacent addresses (a load of
  // 16 bytes from each of 64 places takes 64 cycles of the texture unit, which
  // bound this kernel before: 135 us for 64 x 2^20 samples).
  auto use = [&](const Step &f, int n) {
#pragma unroll
    for (int j = 0; j < OPS; ++j) stage[j * 64 + lane] = __builtin_bit_cast(VT, f.in[j]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double xd[NT][4];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int k = 0; k < XP; ++k) {
          const VT v = stage[St::slot(16 * t + i, (4 * u * XP) + q * XP + k)];
#pragma unroll
          for (int e = 0; e < V; ++e) xd[t][k * V + e] = (double)v[e];
        }
      if (u == 0 && n == head) {
#pragma unroll
        for (int k = 0; k < 3; ++k) xd[T0][k] = lane == 0 && k < c.shift ? 0.0 : xd[T0][k];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[t][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.h[m][u][e / 2][e % 2], xd[t][e], acc[t][m], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_wave_barrier();
  };
  // Two steps in flight, fetched without branches (past the last step the
  // last one again), so that each wait covers its own step's loads only.
  const int steps = blocks / U;
  Step f[2];
  fetch(f[0], 0);
  __builtin_amdgcn_sched_barrier(0);
  int n = 0;
  for (; n + 2 <= steps; n += 2) {
    fetch(f[1], n + 1);
    __builtin_amdgcn_sched_barrier(0);
    use(f[0], n);
    fetch(f[0], n + 2 < steps ? n + 2 : steps - 1);
    __builtin_amdgcn_sched_barrier(0);
    use(f[1], n + 1);
  }
  if (n < steps) use(f[0], n);
  if constexpr (SCAN) {
    // Phi^(len 2^j) for the rounds the run-in needs (past its end, the first
    // one again), all at once where they fit the registers
    constexpr int PN = MT == 1 ? 4 : 1;
    const double *phi = REV ? c.phi_rev : c.phi;
    double P[PN][MT][4 * MT];
    const int lg = 31 - __builtin_clz((unsigned)len);   // len = 2^lg
    if (MT == 1 && (len & (len - 1))) {
      if constexpr (MT == 1) strip_transitions(P, phi, len);
    } else {
#pragma unroll
      for (int j = 0; j < PN; ++j) strip_power<MT>(P[j], phi, lg + (c.terms > (1 << j) ? j : 0));
    }
    if constexpr (!REV) {
      // the raw input's history: x[t0-2] and x[t0-1] enter through the first
      // section's non-recursive stage only (b2, and b1 then b2)
      const ctab<double> tab = as_ctab(c.tab);
      const double b1 = tab[OFF_B1], b2 = tab[OFF_B2];
      double hx[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int k = (16 * m + i) >> 1, d = 1 - (i & 1);
        const gptr<double> g = (gptr<double>)(c.g + (int64_t)(k < c.K ? k : 0) * c.gstride + len - 1 - d);
        const double h = q == 2 ? b2 * g[0] : fma_(b1, g[0], b2 * g[-1]);
        hx[m] = k < c.K && q >= 2 ? h : 0.0;
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int s = s0 + 16 * (t - T0) + i;
        double xe = 0.0;
        if (s > 0 && q >= 2) {
          const int o4 = s * len - c.lead - 4 + q;
          const uint32_t o = (uint32_t)o4 * (uint32_t)es;
          if constexpr (sizeof(TI) == 4) {
            xe = (double)__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, o, 0, 0));
          } else {
            typedef uint32_t v2u __attribute__((ext_vector_type(2)));
            xe = __builtin_bit_cast(double, __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rx, o, 0, 0)));
          }
          if (o4 < c.shift) xe = 0.0;
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[t][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(hx[m], xe, acc[t][m], 0, 0, 0);
      }
    }
    // sums over 2, 4, 8, 16 strips, as far as the run-in reaches
    strip_round<1, NT, MT, REV>(acc, P[0], i);
    if (c.terms > 2) {
      if (PN == 1) strip_power<MT>(P[0], phi, lg + 1);
      strip_round<2, NT, MT, REV>(acc, P[1 % PN], i);
    }
    if (c.terms > 4) {
      if (PN == 1) strip_power<MT>(P[0], phi, lg + 2);
      strip_round<4, NT, MT, REV>(acc, P[2 % PN], i);
    }
    if (c.terms > 8) {
      if (PN == 1) strip_power<MT>(P[0], phi, lg + 3);
      strip_round<8, NT, MT, REV>(acc, P[3 % PN], i);
    }
  }
  // the sum up to strip s is the state at the start of strip s + 1; sums that
  // need more than 16 strips go next to it, in strip s, for the scan kernel
  if constexpr (REV) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int s = s0 + 16 * t + i, d = s - 1;
      // this wavefront's 64 end states (SCAN), or its 64 strips' own sums
      if (d < 0 || s >= (int)c.strips || (SCAN && (d < s0 || d >= s0 + kStripLanes))) continue;
      double *o = rev + (int64_t)d * 2 * c.K;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * m + 4 * r + q < 2 * c.K) o[16 * m + 4 * r + q] = acc[t][m][r];
    }
    return;
  }
  const bool part = SCAN && c.terms > 16;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int s = s0 + 16 * (t - H) + i, d = part ? s : s + 1;
    // SCAN: this wavefront's 64 start states; otherwise its 64 strips' end states
    if (s < 0 || s + 1 >= (int)c.strips || (SCAN && (d < s0 || d >= s0 + kStripLanes))) continue;
    double *o = reinterpret_cast<double *>(ys + c.off + strip_slot<TI>(c, d)) + (part ? strip_state_elems(MT) : 0);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[16 * m + 4 * r + q] = acc[t][m][r];
  }
}

constexpr int kStripStateLds = 80 * 128;   // bytes per wave: a line of five tiles' strips

// Single signals: the instance of the cascade's size and the strips' length.
template <typename TI, int MT, bool SCAN>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void strip_state_kernel(const TI *__restrict__ xs,
                                                                             TI *__restrict__ ys, StripArgs a) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t item = (int64_t)blockIdx.x * kWavesPerBlock + w;
  StripChan c;
  if (!strip_item(a, item, c)) return;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kWavesPerBlock * kStripStateLds];
  strip_state<TI, MT, SCAN>(xs, ys, c, (int)((item - c.first_item) * kStripLanes), smem + w * kStripStateLds);
}

// Workgroup b of a batch's launch, so that eight in a row share an XCD (the
// hardware deals workgroups out to the eight XCDs in turn) and, with it, the
// channel's tables in its L2.
__device__ __forceinline__ int64_t strip_block() {
  const int b = (int)blockIdx.x, whole = (int)gridDim.x / 64 * 64;
  return b < whole ? b / 64 * 64 + b % 8 * 8 + b % 64 / 8 : b;
}

// Batches: a branch per wavefront on the channel's instance.
template <typename TI>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void strip_state_batched_kernel(const TI *__restrict__ xs,
                                                                                     TI *__restrict__ ys,
                                                                                     StripArgs a) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t item = strip_block() * kWavesPerBlock + w;
  StripChan c;
  if (!strip_item(a, item, c)) return;
  const int s0 = (int)((item - c.first_item) * kStripLanes);
  __shared__ __attribute__((aligned(16))) unsigned char smem[kWavesPerBlock * kStripStateLds];
  unsigned char *lds = smem + w * kStripStateLds;
  if (c.mt == 1) {
    if (c.terms > 1) strip_state<TI, 1, true>(xs, ys, c, s0, lds);
    else strip_state<TI, 1, false>(xs, ys, c, s0, lds);
  } else {
    if (c.terms > 1) strip_state<TI, 2, true>(xs, ys, c, s0, lds);
    else strip_state<TI, 2, false>(xs, ys, c, s0, lds);
  }
}

// Start states from sums over 16 strips, where the run-in reaches further:
// with Q = Phi^(16 len), S_s = e_{s-1} + Q (e_{s-17} + Q (e_{s-33} + ...)),
// 16 strips per wavefront.
template <typename TI, int MT>
__global__ __launch_bounds__(kWavesPerBlock * 64) void strip_scan_kernel(TI *__restrict__ ys, StripArgs a) {
  constexpr int PER = kStripLanes / 16, KS = 4 * MT;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t wave = (int64_t)blockIdx.x * kWavesPerBlock + w;
  StripChan c;
  // (a batch launches both MT)
  if (!strip_item(a, wave / PER, c) || c.mt != MT || c.terms <= 16) return;
  const int s0 = (int)((wave / PER - c.first_item) * kStripLanes + (wave % PER) * 16);
  if (s0 >= c.strips) return;
  const int lane = lane_id(), i = lane & 15, q = lane >> 4, s = s0 + i;
  auto sum_of = [&](sv4d (&v)[MT], int u) {
    const bool in = u >= 0 && u + 1 < c.strips;
    const double *o = reinterpret_cast<const double *>(ys + c.off + strip_slot<TI>(c, in ? u : 0)) + strip_state_elems(MT);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[m][r] = in ? o[16 * m + 4 * r + q] : 0.0;
  };
  const int hops = (c.terms + 15) / 16;
  sv4d acc[MT], nx[MT];
  sum_of(acc, s - 1 - 16 * (hops - 1));
  double P[MT][KS];
  strip_power<MT>(P, c.phi, 31 - __builtin_clz((unsigned)c.len) + 4);
  for (int r = hops - 2; r >= 0; --r) {
    sum_of(nx, s - 1 - 16 * r);
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        nx[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(P[m][k], acc[k / 4][k % 4], nx[m], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = nx[m];
  }
  if (s > 0 && s < c.strips) {
    double *o = reinterpret_cast<double *>(ys + c.off + strip_slot<TI>(c, s));
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[16 * m + 4 * r + q] = acc[m][r];
  }
}

// ------------------------------------------------------------ filter pass

// LDS of the filter pass per workgroup.
template <typename TI>
__host__ __device__ constexpr size_t strip_lds_bytes() { return (size_t)kWavesPerBlock * StripStage<TI>::BYTES; }

// One section on C samples of the lane's strip, in place: the non-recursive
// stage in descending order, then the recurrence.  t = (b1, b2, a1, a2), b0
// factored out; (p2, p1) the input's and y0 = (y[-2], y[-1]) the output's
// previous samples.
template <int C>
__device__ __forceinline__ void strip_section(double (&X)[C], const double (&t)[4], double p2, double p1, vd2 y0) {
#pragma unroll
  for (int m = C - 1; m >= 0; --m) {
    const double q1 = m >= 1 ? X[m - 1] : p1, q2 = m >= 2 ? X[m - 2] : (m == 1 ? p1 : p2);
    X[m] = fma_(t[1], q2, fma_(t[0], q1, X[m]));
    if ((m & 3) == 0) __builtin_amdgcn_sched_barrier(0);
  }
  particular_pass<C, double>(X, t[2], t[3], y0[1], y0[0]);
}

// One wavefront: the 64 strips from s0.  Every section's state stays in
// registers, so the sections are unrolled: KT <= 8 is the cascade's own K,
// with the coefficients in scalar registers too; KT = 16 serves any K up to
// 16 (a branch per section), with each section's coefficients loaded during
// the one before it.
// CKPT: also writes every section's state at the start of every chunk to
// `ckpt`, a buffer laid out like x (128 bytes per chunk, K <= 8); !STORE: no
// outputs (ys only holds the start states).
template <typename TI, int KT, bool CKPT = false, bool STORE = true>
__device__ __forceinline__ void strip_filter(const TI *__restrict__ xs, TI *__restrict__ ys, const StripChan &c,
                                             int64_t s0, unsigned char *lds, TI *__restrict__ ckpt = nullptr) {
  typedef StripStage<TI> St;
  typedef typename St::VT VT;
  constexpr int V = St::V, C = St::C;
  constexpr bool FIXED = KT <= 8;
  const int lane = lane_id(), K = FIXED ? KT : c.K;
  VT *stage = reinterpret_cast<VT *>(lds);
  const TI *x = xs + c.off;
  TI *y = ys + c.off;
  // the lane's own strip: start state and raw input history
  const int64_t s = s0 + lane, t0 = s * c.len - c.lead - c.shift;
  const bool live = s < c.strips;
  vd2 ys0[KT];   // every section's (y[-2], y[-1])
  {
    const vd2 *S = reinterpret_cast<const vd2 *>(y + strip_slot<TI>(c, live ? s : 0));
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      ys0[k] = vd2{0.0, 0.0};
      if (live && s > 0 && k < K) ys0[k] = S[k];
    }
  }
  double xm2 = (live && t0 >= 2) ? (double)x[t0 - 2] : 0.0;
  double xm1 = (live && t0 >= 1) ? (double)x[t0 - 1] : 0.0;
  // The access pattern: op j moves piece slot(row, lane % PIECES) of row
  // j * ROWS + lane / PIECES.  Loads and stores go through buffer descriptors
  // over the wave's part of the channel, which return zeros and drop stores
  // past its end: one code path for every chunk, so that a wait for a chunk's
  // loads counts exactly the accesses issued after them.
  const __amdgpu_buffer_rsrc_t rx = strip_rsrc(xs, c), ry = strip_rsrc(ys, c);
  // the checkpoints' buffer ends on a whole chunk and starts with the channel
  const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
      ckpt, 0, (int)(uint32_t)(((c.n + c.shift) * (int64_t)sizeof(TI) + 127) / 128 * 128), 0x00020000);
  uint32_t at[St::OPS];   // byte offset of the lane's piece of op j
#pragma unroll
  for (int j = 0; j < St::OPS; ++j) {
    const int row = j * St::ROWS + lane / St::PIECES;
    at[j] = (uint32_t)((s0 + row) * c.len - c.lead) * (uint32_t)sizeof(TI) +
            16u * (uint32_t)(St::slot(row, lane % St::PIECES) - row * St::PIECES);
  }
  const ctab<double> tab = as_ctab(c.tab);
  double cf[FIXED ? KT : 1][4];
#pragma unroll
  for (int k = 0; k < (FIXED ? KT : 1); ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j) cf[k][j] = tab[(int64_t)k * c.stride + OFF_B1 + j];
  const int chunks = (int)(c.len / C);
  auto fetch = [&](sv4u (&in)[St::OPS], int ch) {
#pragma unroll
    for (int j = 0; j < St::OPS; ++j)
      in[j] = __builtin_bit_cast(sv4u, __builtin_amdgcn_raw_buffer_load_b128(rx, at[j] + 128u * (uint32_t)ch, 0, 0));
  };
  // Three chunks are in flight: chunk ch in X, ch + 1 staged and read back as
  // the lane's own run (own) while ch is filtered, ch + 2 on its way from
  // HBM (in).  The LDS tile serves them and the outputs in turn; a wave's LDS
  // accesses stay in order.
  VT own[St::PIECES];
  auto stage_in = [&](const sv4u (&in)[St::OPS]) {
    // the tile's position `lane` of op j holds piece pc (slot is its own
    // inverse in the piece)
#pragma unroll
    for (int j = 0; j < St::OPS; ++j) stage[j * 64 + lane] = __builtin_bit_cast(VT, in[j]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int p = 0; p < St::PIECES; ++p) own[p] = stage[St::slot(lane, p)];
    __builtin_amdgcn_wave_barrier();
  };
  // the chunk of strip 0 that starts at the channel's aligned start
  const int head = s0 == 0 && c.shift > 0 ? c.lead / C : -1;   // uniform
  VT firsts = {};
  sv4u in[St::OPS];
  fetch(in, 0);
  stage_in(in);
  fetch(in, 1);
  auto chunk = [&](int ch) {
    double X[C];
#pragma unroll
    for (int p = 0; p < St::PIECES; ++p)
#pragma unroll
      for (int i = 0; i < V; ++i) X[p * V + i] = (double)own[p][i];
    stage_in(in);
    fetch(in, ch + 2);
    if (ch == head) {
      // the samples before the channel's start: zeros (lane 0)
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (lane == 0 && i < c.shift) X[i] = 0.0;
    }
    if constexpr (CKPT) {
      static_assert(!CKPT || KT <= 8, "one line per checkpoint");
#pragma unroll
      for (int p = 0; p < KT; ++p) reinterpret_cast<vd2 *>(stage)[St::slot(lane, p)] = ys0[p];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < St::OPS; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(sv4u, stage[j * 64 + lane]), rc,
                                               at[j] + 128u * (uint32_t)ch, 0, 0);
      __builtin_amdgcn_wave_barrier();
    }
    double p2 = xm2, p1 = xm1;
    xm2 = X[C - 2];
    xm1 = X[C - 1];
    double t[4] = {cf[0][0], cf[0][1], cf[0][2], cf[0][3]};
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      if (!FIXED && k >= K) break;   // uniform
      const vd2 y0 = ys0[k];
      if constexpr (FIXED) {
        strip_section<C>(X, cf[k], p2, p1, y0);
      } else {
        const ctab<double> tn = tab + (int64_t)(k + 1 < K ? k + 1 : 0) * c.stride + OFF_B1;
        const double n0 = tn[0], n1 = tn[1], n2 = tn[2], n3 = tn[3];
        __builtin_amdgcn_sched_barrier(0);
        strip_section<C>(X, t, p2, p1, y0);
        t[0] = n0;
        t[1] = n1;
        t[2] = n2;
        t[3] = n3;
      }
      ys0[k] = vd2{X[C - 2], X[C - 1]};
      p2 = y0[0];
      p1 = y0[1];
    }
    if constexpr (STORE) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int p = 0; p < St::PIECES; ++p) {
        VT v;
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = (TI)(X[p * V + i] * c.gain);
        stage[St::slot(lane, p)] = v;
      }
      __builtin_amdgcn_wave_barrier();
      if (ch == head) {
        // the first piece also covers samples before the channel's start: its
        // stores are dropped, and its samples of the channel kept for the end
        firsts = stage[St::slot(0, 0)];
      }
#pragma unroll
      for (int j = 0; j < St::OPS; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(sv4u, stage[j * 64 + lane]), ry,
                                               ch == head && j == 0 && lane == 0 ? 0xffffff00u : at[j] + 128u * (uint32_t)ch,
                                               0, 0);
      __builtin_amdgcn_wave_barrier();
    }
  };
  // dropped stores, so that the loop is entered with as many accesses behind
  // the loads of chunk 1 as it goes round with, and its waits count the same
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < St::OPS * ((CKPT ? 1 : 0) + (STORE ? 1 : 0)); ++j)
    __builtin_amdgcn_raw_buffer_store_b128(sv4u{0, 0, 0, 0}, ry, 0xfffffc00u + 16 * j, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  int ch = 0;
  do chunk(ch); while (++ch < chunks);
  if (STORE && head >= 0 && lane < V && lane >= c.shift && lane - c.shift < c.n) {
    TI v = firsts[0];
#pragma unroll
    for (int i = 1; i < V; ++i)
      if (lane == i) v = firsts[i];
    y[lane - c.shift] = v;
  }
}

// Single signals: the cascade's own instance.
template <typename TI, int KT>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void strip_filter_kernel(const TI *__restrict__ xs,
                                                                              TI *__restrict__ ys, StripArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t item = (int64_t)blockIdx.x * kWavesPerBlock + w;
  StripChan c;
  if (!strip_item(a, item, c)) return;   // uniform per wave
  strip_filter<TI, KT>(xs, ys, c, (item - c.first_item) * kStripLanes, smem + (size_t)w * StripStage<TI>::BYTES);
}

// Batches: the last workgroups, as many as the live strips need, take 64 strips
// per wavefront; all before them filter the channels that stay with the tiles
// (their serial chains start first and finish beside the strips), in turn where
// there are more tile items than wavefronts.  The split follows the present
// channels, as a replan moves them between the two; the launch holds a
// workgroup more than its strips can take (launch_batched).
template <int N, typename TI>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void strip_batched_kernel(
    const TI *__restrict__ xs, TI *__restrict__ ys, const BatchChan *__restrict__ chans,
    const int32_t *__restrict__ item_chan, const int64_t *__restrict__ hdr, int32_t kmax, StripArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int rows_blocks =
      (int)gridDim.x - (int)((as_ctab(a.items_live)[0] + kWavesPerBlock - 1) / kWavesPerBlock);
  if ((int)blockIdx.x < rows_blocks) {
    const int64_t step = (int64_t)rows_blocks * kWavesPerBlock;
    for (int64_t item = (int64_t)blockIdx.x * kWavesPerBlock + w; item < hdr[0]; item += step)
      batched_rows<N, TI, double, true, SOS_PH, kL>(xs, ys, chans, item_chan, item, w, kmax, smem);
    return;
  }
  const int64_t item = (int64_t)((int)blockIdx.x - rows_blocks) * kWavesPerBlock + w;
  StripChan c;
  if (!strip_item(a, item, c)) return;   // uniform per wave
  strip_filter<TI, 16>(xs, ys, c, (item - c.first_item) * kStripLanes, smem + (size_t)w * StripStage<TI>::BYTES);
}

}  // namespace sosf
