// Descriptors of the strip kernels (kernels_strip.hpp), shared by the plan
// and the launches.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace sosf {

constexpr int kStripBlock = 16;          // samples per block of the state table
constexpr int kStripMaxSpan = 1024;      // samples the state table covers at most
constexpr int kStripMaxK = 16;           // 2K state rows fit two 16-row tiles
constexpr int kStripMaxTerms = 512;      // strips a start state is summed over at most
constexpr int kStripLanes = 64;          // strips per wavefront of the filter kernel

// A channel (or a single signal) cut into strips of `len` samples over
// [-shift - lead, n); strip s starts at s * len - lead - shift.  The samples
// before 0 are zeros; the lead, a multiple of 32 that leaves at least 32 samples
// of strip 0, keeps the last strip long enough for its start state
// (strip_sound).
struct StripChan {
  const double *tab;       // the plan's section rows
  const double *hop;       // state table, in the order the products read it (upload_strip)
  const double *g;         // all-pole responses, [K][gstride]
  const double *phi;       // padded powers Phi^(2^j) in the A operand's order
  const double *hop_rev;   // the adjoint's state table and powers, in reversed time
  const double *phi_rev;
  int64_t off, n;          // first sample in x / y, length
  int64_t len, strips;     // strip length (a multiple of 32; a power of two where terms > 16, or > 1 and mt = 2), strips
  int64_t first_item;      // first work item (64 strips) of the channel
  int32_t K, stride;
  int32_t shift;           // off mod the samples per 16 bytes
  int32_t span;            // samples of a strip that its end state is summed over (a multiple of 16)
  int32_t terms;           // strips whose end states reach into the next strip's start
  int32_t mt;              // 16-row tiles of the state: ceil(2K / 16)
  int32_t gstride;         // doubles per row of g
  int32_t lead;            // zero samples before the aligned start
  int32_t pad;
  double gain;
};

static_assert(sizeof(StripChan) % 8 == 0, "copied by 64-bit words");

// The adjoint of a channel by strips: the forward's strips, and its regions
// of the workspace (in doubles).
constexpr int kAdjStripK = 8;
struct AdjStrip {
  StripChan c;
  const double *bwd;       // adjoint rows (BW_*)
  int64_t ck_off;          // checkpoints: 128 bytes per 128 bytes of signal
  int64_t rev_off;         // states at the strips' ends, 2K per strip
  int64_t part_off;        // coefficient sums, [K][waves][5]
  int64_t waves;           // wavefronts of 64 strips
};
static_assert(sizeof(AdjStrip) % 8 == 0, "copied by 64-bit words");

}  // namespace sosf
