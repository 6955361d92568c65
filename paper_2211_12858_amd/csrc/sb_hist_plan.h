// Constants and work plan of the histogram kernel (fixed point, workgroup
// shape, LDS budget, feature slicing).
#pragma once

#include <cstdint>

namespace sb {

// ---------------------------------------------------------------- fixed point
// Quantised magnitudes are <= 2^QBITS (qexp = QBITS-1 - floor(log2(max|v|))),
// so each value carries an error of at most 2^-(QBITS+1) of its channel's
// maximum magnitude.
constexpr int QBITS = 18;
// Each channel's LDS sum is a 32-bit running sum read back into int64 every
// window of WINDOW_ROWS rows (10 steps of the 768-thread workgroup), between
// two barriers.  A cell gets at most one value per row, so its change between
// two reads is at most WINDOW_ROWS * 2^QBITS, which must stay below 2^31.
// (Windows of 4 steps with one barrier each, whose changes may span two
// windows, folded more often: root of 2M x 100 148 against 138 us, 1M x 99 x
// 21 channels 322 against 307 us.)
constexpr int WINDOW_ROWS = 7680;
static_assert((int64_t)WINDOW_ROWS * (1ll << QBITS) < (1ll << 31), "fixed-point window overflow");
// The rotated kernel reads each row's quantised values, not its fp32 sketch:
// up to 6 channels as QFIELD_BITS-bit two's-complement fields of one 16-byte
// word (channels 0-2 in bits 0-62 of the low 64 bits, 3-5 in the high 64
// bits), written once per sketch, so that a row's values are one 16-byte load.
constexpr int QFIELD_BITS = 21;
constexpr int QROW_MAX_C = 6;
// More channels take several such words per row, one per channel group of
// four or six (see HistPlan); each group gets workgroups of its own (up to
// ROT_MAX_C channels).
constexpr int ROT_MAX_C = 24;
static_assert(QBITS + 2 <= QFIELD_BITS, "a quantised value of magnitude <= 2^QBITS and its sign must fit a field");

// ---------------------------------------------------------------- histogram plan
// MI355X: 8 XCDs of 32 CUs; workgroup b is dispatched to XCD b % 8.
constexpr int HIST_CUS = 256;
// A row group holds at least one step's rows (see groups_in_use): with all 256
// row groups, a tree on 10,000 rows x 10 features took 174 us, with at least
// 768 rows 110, 1152 rows 113, 1536 rows 116 and 2304 rows 117 us.  Of 35 trees on
// 1,000 to 200,000 rows x 10 to 200 features, 1536 rows made 29 no faster (up to 15%
// slower: 10,000 x 100, depth 8, 794 -> 915 us) and six faster, most of all wide levels
// of one slice (200,000 x 10, depth 3, 147 -> 131 us).
constexpr int GROUP_MIN_ROWS = 768;

// One histogram workgroup: 768 threads (12 waves, 3 per SIMD) and the cells
// of a slice of 16 features for up to 3 channel pairs (c <= 6), laid out
// [bin][pair][feature] for 256 bins (12288 64-bit cells, 96 KB of the
// 160 KB LDS), rot_cpt(pairs) cells per thread.
constexpr int ROT_THREADS = 768;
constexpr int ROT_F = 16;
constexpr int ROT_PMAX = 3;
constexpr int ROT_CELLS = 256 * ROT_PMAX * ROT_F;
// Cells per thread of a workgroup with that many pairs: 6, 11 and 16.  (With 16
// for every count, 47 registers spilled with one pair and 12 with two once a node's
// end also held the next node's rows: trees of 2M x 100 at k = 1 637 us, 609 so; two
// gathered nodes of 1M x 20 at 32 bins, k = 1, 40.8 and 38.4 us.)
constexpr int rot_cpt(int pairs) { return (256 * pairs * ROT_F + ROT_THREADS - 1) / ROT_THREADS; }
constexpr int ROT_ROWS = ROT_THREADS / ROT_F;  // rows of 16 cells that the workgroup touches at once
static_assert(ROT_ROWS % 2 == 0 && ROT_ROWS % 3 == 0, "a thread's cells must share one pair");
// Staging of a node's partials in the same LDS: rows of rot_stage_ld(n_bins)
// int32 pairs, at most 258.
constexpr int rot_stage_ld(int n_bins) { return (n_bins + 29) / 32 * 32 + 2; }
constexpr int ROT_STAGE_PAIRS = ROT_PMAX * (ROT_F * rot_stage_ld(256) + 1);
constexpr int ROT_LDS_BYTES = 8 * (ROT_STAGE_PAIRS > ROT_CELLS ? ROT_STAGE_PAIRS : ROT_CELLS);
static_assert(rot_cpt(ROT_PMAX) * ROT_THREADS == ROT_CELLS, "the threads' cells must lie in the LDS");
static_assert(WINDOW_ROWS % ROT_THREADS == 0, "a fixed-point window must be a whole number of steps");

struct HistPlan {
  int c;          // channels k+1
  int pairs;      // channel pairs: ceil(c/2)
  int nq;         // 4-feature quads per slice (0: the shape is not supported)
  int f;          // features per slice (16)
  int slices;     // feature slices
  int cells;      // 2 * pairs * f * n_bins channel cells of a partial
  int q;          // row groups per full slice
  int64_t slots;  // partial slots per slice: max(q, q_thin) + n_build
  // Rotated kernel: the first slices_full slices hold 16 features each; when
  // m is not a multiple of 16 the rest go to one thin slice of f_thin
  // features (a power of two below 16), whose workgroups keep 16 / f_thin
  // copies of each cell so that its adds stay conflict-free while a row
  // costs f_thin steps instead of 16: q row groups of every full
  // slice and q_thin of the thin slice, chosen to even out the work of the
  // 256 CUs.  Only for rows read straight from the data (the root): rows gathered through row
  // indices are cheaper to read when the slices of a row group share an XCD,
  // so there the last slice is a padded slice of 16 like the others.
  int slices_full, f_thin, q_thin;
  // Rotated kernel with c > 6 channels: cg = ceil(c / 6) channel groups of
  // gc channels (the channel pairs spread evenly, at most three each: 7 and 8
  // channels take two groups of two pairs, not one of three and one of one);
  // every (slice, channel group) of a row group is one workgroup, and all
  // groups of a slice write the same partial slots.  gc = c for one group.
  // (Histograms of a tree on 1,000,001 x 64 with k = 7: 346 us in groups of six,
  // 301 us so.)
  int cg, gc;
  // Workgroups: q * slices_full * cg of the full slices and q_thin * cg of the
  // thin one, an eighth to each XCD.  Row groups need not be a multiple of the
  // XCDs: 7 slices take 36 row groups (252 CUs), where 4 per XCD take 224.
  int grid;       // histogram workgroups
};
// Plan of one histogram launch; nq == 0 when c > ROT_MAX_C or n_bins > 256.
HistPlan hist_plan(int32_t m, int32_t n_bins, int32_t k, int32_t n_build, bool thin_ok = false);
// Workspace of one histogram launch (-1 when unsupported); quant_rows adds
// the n quantised sketch rows (16 * cg bytes each).
int64_t hist_ws_bytes(int64_t n, int32_t m, int32_t n_bins, int32_t k, int32_t n_build, bool quant_rows);

}  // namespace sb
