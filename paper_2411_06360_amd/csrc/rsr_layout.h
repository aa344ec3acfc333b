// Layout of the RSR index in device memory: what the builder (rsr_prep.hip) writes and the product kernels
// (rsr_lib.hip) read.
//
// Logical content, per part (B(1), B(2) of Proposition 2.1; the bit planes of a q-bit matrix) and per k-column
// block (Definition 3.1): the row permutation sigma of Definition 3.2 and the full segmentation L of Section 3.3.
//
//   * A row's value in a block is its k bits read with the first column most significant; a last block narrower
//     than k is treated as if its missing columns were zero (values shifted left by k - width).  Rows with value 0
//     add nothing (row 0 of Bin_[k] is zero) and are not stored.
//   * A PANEL is a piece of a block's segment sums u that is kept in LDS and folded at once: all values of the block,
//     both parts of a ternary matrix together, where they fit in kMaxPanelSlots slots, otherwise 2^kc consecutive
//     values of one part.  Slot of a value: part * pslots + (value mod 2^kc).
//   * The segments of a panel (sets of equal rows) are ranked by their number of rows, longest first, and dealt
//     to the 64 lanes of a wavefront in rank order: a GROUP is 64 consecutive segments, one per lane, walked for as
//     many positions as its longest segment has rows.  Ranking makes the 64 segments of a group almost equally long,
//     so that no lane needs a flag of its own: where a group ends is the same position for all lanes, a bit of a mask
//     in the unit's descriptor (which picks the code of a step), and the position behind it, the HEAD, holds the lanes' slots.
//     Among segments of equal length the order is such that the slots of neighbouring lanes lie in different LDS
//     banks.  Shorter segments in a group, and the lanes of a group that is not full, read the null row index `rows`
//     (a zero kept behind the activations in LDS); lanes without a segment store to a dummy slot.
//   * A long segment takes 8 neighbouring lanes, whose sums are added with lane exchanges at the head.  A segment
//     of more than kWideRows rows is cut; the further pieces go to extra slots behind the panel's, whose sums the fold
//     adds to the bits of the segment's value.  (No slot then sums more than 256 rows: an int8 sum fits 16 bits.)
//   * Values that no row has: either all slots are cleared before a panel uses them, or (`fill`, where few values are
//     absent) the absent values form groups of no rows at the end, whose heads store zeros.
//   * A UNIT is a run of whole groups of one width, at most kMaxPositions positions; a wavefront sums one unit at a
//     time.  In memory position p of a unit is 64 uint16, one per lane; a lane's 8 consecutive positions are adjacent
//     (a granule: 64 x 16 bytes, one 16-byte load per lane), the positions behind the last full granule are rows of
//     dwords (two positions per lane; the count is even).
//
// Streams on the device:
//   stream    bytes   unit streams, back to back, each on a 128-byte boundary
//   units     PUnit   32-byte descriptors, in panel order, and room for kUnitsBehind more (read ahead by wavefronts that have no unit)
//   blk_unit  uint32  nblocks+1 offsets into `units`
#ifndef RSR_LAYOUT_H_
#define RSR_LAYOUT_H_

#include <stdint.h>

#include "rsr_format.h"

namespace rsr {

constexpr int kMaxPanelBits = 12;                    // values per panel and part: at most 2^12
constexpr int kMaxPanelSlots = 1 << kMaxPanelBits;   // 16 KB of float sums
constexpr int kFoldRow = 256;                        // slots one step of the fold reads (64 lanes x 4); parts start on multiples
constexpr int kDummySlots = 32;                      // behind the slots of a panel: where lanes without a segment store
constexpr int kWideRows = 256;                       // rows of a piece of a segment at most (8 lanes, 32 rows each)
// Passes over several int8 vectors keep a slot's sum in 16 bits: kWideRows entries of -128 .. 127 are what these hold.
static_assert(kWideRows * 128 <= 32768 && kWideRows * 127 <= 32767, "the sum of a slot has to fit 16 bits");
constexpr int kMaxExtras = 2 * 32768 / kWideRows;    // extra slots of a panel at most (both parts of 32768 rows)

constexpr int kUnitsBehind = 16;                     // as many as a workgroup has wavefronts

struct alignas(16) PUnit {
  uint32_t stream_off;   // in multiples of kStreamAlign bytes
  uint32_t block;        // column block
  uint32_t panel;        // panel number in the tile = block * panels_per_block + number in the block
  uint32_t heads_lo;     // bit p: position p is a head
  uint16_t heads_hi;     // positions 32..47
  uint8_t npos;          // even, <= kMaxPositions; 0 = a panel without entries
  uint8_t wide;          // 1: every segment takes 8 lanes
  uint16_t units_in_panel;
  uint16_t extras;       // pieces in extra slots of this panel
  uint32_t first;        // rank of the unit's first segment (builder only)
  uint32_t reserved;
};
static_assert(sizeof(PUnit) == 32, "unit descriptor must be 32 bytes");

// The split of a tile into panels.
struct Shape {
  int kc;        // value bits inside a panel
  int both;      // 1: both parts of a ternary matrix share a panel (their slots are subtracted in the fold)
  int pslots;    // slots per part of a panel
  int nslots;    // slots of a panel
  int panels;    // panels per block
};

// The most values per panel for which four panels fit in the 160 KB of LDS beside the activations (one float per row).  Larger
// panels have fuller groups and fewer folds; with fewer than four of them in flight wavefronts wait for room
// (32768 rows, k = 13, four float vectors: 2^11 values 390 us, 2^10 365 us; 16384 rows, k = 12: 2^12 14.3 us, 2^11 15.4 us).
inline Shape panel_shape(int64_t rows, int k, int parts, bool signed_pair) {
  Shape s;
  const int64_t lds = 160 * 1024 - 4096;
  int most = kMaxPanelBits;
  while (most > 10 && (rows + 4) * 4 + 4 * 4 * (int64_t)((1 << most) + kDummySlots + kMaxExtras) > lds) --most;
  s.both = parts == 2 && signed_pair && k <= most - 1;
  s.kc = k < most ? k : most;
  s.pslots = (1 << s.kc) < kFoldRow ? kFoldRow : (1 << s.kc);
  s.nslots = s.both ? 2 * s.pslots : s.pslots;
  s.panels = s.both ? 1 : parts << (k - s.kc);
  return s;
}

}  // namespace rsr
#endif  // RSR_LAYOUT_H_
