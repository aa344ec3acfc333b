// Launch planning of the product kernels (rsr_lib.hip): grid, workgroup size, LDS layout, and how many vectors share a
// pass.  Host code without any HIP call, so that a program on a machine with no GPU can check it.
#ifndef RSR_PLAN_H_
#define RSR_PLAN_H_

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>

#include "../../include/rsr.h"
#include "rsr_layout.h"

namespace rsr {

constexpr int kItems = 16;  // words of a panel's record per vector: value bits 0 .. 11, the total, unused

// An activation mode as the planner sees it: vectors per pass, LDS bytes per row (1 << shift) and per slot of a panel.
struct Pass {
  int V, shift, slot_bytes;
};
constexpr Pass kF1{1, 2, 4}, kF2{2, 3, 8}, kF4{4, 4, 16};  // float
constexpr Pass kI1{1, 2, 4}, kP2{2, 2, 4}, kP4{4, 3, 8};   // int8: one vector in 32 bits, two and four in 16

// What a launch has to know of a row tile and of its matrix.
struct PlanTile {
  int64_t rows = 0, row0 = 0;
  Shape shape{};
  int extra_stride = 0, max_extras = 0;  // entries per panel in the list of extra slots; extra slots of a panel at most
  bool fill = false;  // absent values are stored as zeros: a panel's slots need no clearing
  uint32_t max_units_per_block = 0;
  int64_t nunits = 0;
  size_t stream_bytes = 0;  // of all units: kPositionBytes per position
};
struct PlanMatrix {
  int num_cu = 0;
  size_t lds_max = 0;
  int64_t rows = 0, cols = 0, nblocks = 0;
  int k = 0, last_width = 0;
  bool qbit = false;      // the parts are bit planes: part i weighs 2^(first_plane + i), negative_part its negative
  int first_plane = 0, negative_part = -1;
  int waves = 16;  // wavefronts per workgroup at most
  bool step2_plain = false;  // rsr_set_step2
};

// Kernel arguments.
struct KArgs {
  // what the start of a kernel and its units need, together (a scalar load takes neighbouring words)
  int nbuf;      // panels in flight per workgroup
  uint32_t ubytes;  // bytes of a panel's sums in LDS
  uint32_t off_u, off_rec, off_done, off_blocks, off_cnt, off_epoch, off_ctr;  // LDS byte offsets
  uint32_t buf_magic, rec_magic;  // x / nbuf and x / nrec as high halves of products
  int panels;       // of a block (rsr_layout.h)
  int extra_stride; // entries per panel in the list of extra slots
  // Slots have to be cleared ahead of the first panels.  Where every panel stores all its values (`fill`) only slots that are no
  // value's are: those of panels of fewer values than a step of the fold reads.  (The slot of value 0 is not stored, but counts under no bit.)
  int clear;
  int cols, k, nblocks, last_width;
  int accumulate;  // add to `out` instead of overwriting it (second and later row tiles, rsr_matvec_acc)
  int scaled;      // multiply the product by `scale` first (rsr_matvec_acc)
  uint32_t scale;  // bits of a float (float activations) or of an int (int8 activations)
  int kc, both, pslots;  // of a panel (rsr_layout.h)
  int fill;              // absent values are stored as zeros
  // a part's weight: 1 << (part * wshift + wfirst), negative for part `wneg` (-1: none)
  int wshift, wfirst, wneg;
  int nrec;      // blocks whose panel records are kept (panels > 1)
};

// What a workgroup needs to know before it can ask for anything: its share of the blocks, and where its activations are.  Six words, which
// go ahead of the other arguments with four pointers: the fourteen words that a wavefront finds in its scalar registers when it
// starts (rsr_lib.hip).
struct Start {
  uint32_t sets_more;   // sets of vectors | share_more << 16
  uint32_t sets_magic;  // x / sets as the high half of a product
  uint32_t share;       // column blocks of a workgroup; the first share_more workgroups have one more
  uint32_t rows_stride; // rows | vstride << 16 (elements between consecutive vectors: the matrix's row count)
  uint32_t row0_g1;     // first row of the row tile | g1 << 16 (workgroups per set of vectors)
  uint32_t shape;       // wavefronts that take units | wavefronts of the workgroup << 8 | vectors << 16
  constexpr uint32_t sets() const { return sets_more & 0xffffu; }
  constexpr uint32_t share_more() const { return sets_more >> 16; }
  constexpr int rows() const { return (int)(rows_stride & 0xffffu); }
  constexpr int vstride() const { return (int)(rows_stride >> 16); }
  constexpr uint32_t row0() const { return row0_g1 & 0xffffu; }
  constexpr uint32_t g1() const { return row0_g1 >> 16; }
  constexpr uint32_t waves() const { return shape & 0xffu; }
  constexpr int threads() const { return (int)(shape >> 8 & 0xffu) * 64; }
  constexpr int batch() const { return (int)(shape >> 16); }
};
static_assert(kTileRows < 65536 && kMaxRows < 65536, "rows and strides fit 16 bits");

// A workgroup's set of vectors and column blocks.  The siblings of a block range, one per set, sit 8 workgroup ids apart so that
// round-robin dispatch puts them on the same XCD (shared L2).  Without a division: in the kernel three of them (two in 64 bits) took 0.2 to
// 0.4 us of every launch (ternary 4096^2, one vector: 6.3 -> 6.1 us; 16384^2: 14.3 -> 13.9).  The magic product is exact: a
// workgroup's number over 8 is below the number of sets plus 2^10, both factors stay below 2^16.
struct Share {
  uint32_t set, first, last;  // blocks first .. last - 1
};
constexpr Share share_of(const Start& st, uint32_t wg) {
  const uint32_t sets = st.sets(), more = st.share_more(), eights = wg >> 3;
  const uint32_t grp = sets == 1 ? eights : (uint32_t)(((uint64_t)eights * st.sets_magic) >> 32);
  const uint32_t g = grp * 8 + (wg & 7);
  Share s{eights - grp * sets, 0, 0};
  if (g < st.g1()) {
    s.first = g * st.share + (g < more ? g : more);
    s.last = s.first + st.share + (g < more ? 1u : 0u);
  }
  return s;
}

struct LaunchPlan {
  KArgs p;
  int rows = 0, vstride = 0, row0 = 0, batch = 0;
  int sets = 0, g1 = 0;  // sets of vectors, workgroups for each
  uint32_t share = 0, share_more = 0;
  int64_t grid = 0;
  int waves = 0;  // wavefronts that take units; of the workgroup, too, unless it shares the launch with larger ones
  size_t lds = 0;
};

constexpr int kManyPanels = 16;  // panels per block from which the records of one block may do
constexpr int kMostBuffers = 8;  // panels in flight per workgroup at most

constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// x / d for small x as the high half of a product (d >= 2)
inline uint32_t magic(uint32_t d) { return d < 2 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

// How many workgroups of so many bytes share a compute unit's LDS, which is given out in pieces of 1280 bytes (binary 4713 x 1264, k = 11,
// eleven vectors, two per pass: three workgroups of 54 000 bytes, 690 in all, were planned where two fit, and took two rounds: 12.0 us, 8.2 now).
constexpr int groups_in_lds(size_t bytes, size_t lds_max) { return (int)(lds_max / align_up(bytes, 1280)); }

// Launch shape of one row tile for `batch` vectors on `num_cu` compute units in mode M.
// `max_wg_per_cu`: how many workgroups of this product may share a compute unit (a launch that carries
// several products gives every workgroup the largest LDS size any of them needs, so it plans with 1).
// Returns RSR_ERR_UNSUPPORTED if the mode does not fit in LDS, RSR_ERR_INVALID_ARGUMENT if the batch is too large for a grid.
inline int plan_tile(const Pass& M, const PlanMatrix& h, const PlanTile& T, bool accumulate, int batch, int num_cu, int max_wg_per_cu, LaunchPlan* plan) {
  KArgs& p = plan->p;
  std::memset(&p, 0, sizeof(p));
  const Shape& S = T.shape;
  p.cols = (int)h.cols; p.k = h.k;
  p.nblocks = (int)h.nblocks; p.last_width = h.last_width; p.accumulate = accumulate ? 1 : 0;
  p.kc = S.kc; p.both = S.both; p.pslots = S.pslots; p.panels = S.panels;
  p.fill = T.fill ? 1 : 0; p.extra_stride = T.extra_stride;
  p.clear = !T.fill || (1 << S.kc) < kFoldRow;
  p.wshift = h.qbit ? 1 : 0; p.wfirst = h.first_plane; p.wneg = h.negative_part;

  // LDS: activations, panels in flight, records of the blocks in flight, counters
  const size_t vbytes = align_up((size_t)(T.rows + 1) << M.shift, 16);
  p.ubytes = (uint32_t)((size_t)(S.nslots + kDummySlots + (T.max_extras + 7) / 8 * 8) * M.slot_bytes);
  const bool records = S.panels > 1 || h.qbit;
  const size_t rec_bytes = (size_t)S.panels * M.V * kItems * 4;
  // Records of as many blocks as can have a panel in flight.  Where those of one block leave room for more panels there is only one:
  // a wavefront that folds a panel of the next block then waits for the block before, which is rare with many panels a block
  // (65534 x 2048 ternary, k = 16, 128 panels: 139 -> 97 us; 32768 x 4096, k = 14, 32 panels: 35.3 -> 33.1).
  bool one_block = false;
  auto recs = [&](int nbuf) { return records ? 1 + (one_block ? 0 : (nbuf - 1 + S.panels - 1) / S.panels) : 0; };
  auto total = [&](int nbuf) { return vbytes + (size_t)nbuf * p.ubytes + (size_t)recs(nbuf) * (rec_bytes + 8) + (size_t)nbuf * 8 + 16; };
  // Grid and workgroup size.  Up to four workgroups per compute unit if they fit together (LDS, and 16
  // wavefronts per compute unit at this kernel's register count); never more workgroups than blocks; and
  // no more wavefronts than the largest share of a workgroup has units: idle wavefronts only lengthen
  // the start of the launch (1024 x 1024: 5.5 -> 4.0 us per product).
  const int64_t sets = ((int64_t)batch + M.V - 1) / M.V;
  int64_t g1 = 1;
  int waves = 0, nbuf = 0;
  for (int wg = max_wg_per_cu; wg >= 1; --wg) {
    // The siblings of a block range share an XCD, so a set has a multiple of 8 workgroups; rounded down, since one workgroup more than
    // the device holds is a second round for all (three vectors at 2048 x 8192, 88 * 3 workgroups on 256 compute
    // units: 12.6 us, 80 * 3: 8.0).
    g1 = std::max<int64_t>(8, (int64_t)num_cu * wg / sets / 8 * 8);
    if (g1 > h.nblocks) g1 = h.nblocks;
    const int64_t blocks_per_wg = (h.nblocks + g1 - 1) / g1;
    // Equal shares: no more workgroups than it takes to keep the largest share this small.  (1366 blocks
    // over 256 compute units would be 5 or 6 blocks each; 228 workgroups get 6 each, 28 compute units
    // stay idle, and the product is 0.5 us faster: the stream is shared by all compute units and the
    // workgroups with the larger share finish last either way, only later when more of them compete.)
    g1 = (h.nblocks + blocks_per_wg - 1) / blocks_per_wg;
    const int64_t units_per_wg = blocks_per_wg * (int64_t)std::max<uint32_t>(1, T.max_units_per_block);
    waves = (int)std::min<int64_t>(h.waves, units_per_wg);
    // Up to eight panels in flight where the LDS holds them (a wavefront whose unit belongs to a later panel waits).
    const int64_t panels_per_wg = blocks_per_wg * S.panels;
    const int most = (int)std::min<int64_t>(kMostBuffers, panels_per_wg), least = (int)std::min<int64_t>(2, panels_per_wg);
    auto most_that_fit = [&]() {
      int n = most;
      while (n > least && (total(n) > h.lds_max || (wg > 1 && groups_in_lds(total(n), h.lds_max) < wg))) --n;
      return n;
    };
    one_block = false;
    nbuf = most_that_fit();
    if (total(nbuf) > h.lds_max) return RSR_ERR_UNSUPPORTED;
    if (S.panels >= kManyPanels && nbuf < most) {
      one_block = true;
      const int n = most_that_fit();
      if (n > nbuf) nbuf = n;
      else one_block = false;
    }
    // (of five wavefronts only two workgroups share a compute unit, all other sizes fill its sixteen: timed with kernels that spin,
    // 256 * wg workgroups of n wavefronts at this register count, n = 1 .. 16; ternary 2902 x 6720, k = 9: 9.4 -> 6.7 us)
    if (wg == 1 || (wg * waves <= 16 && !(wg == 3 && waves == 5) && groups_in_lds(total(nbuf), h.lds_max) >= wg)) break;
  }
  const int64_t grid = (g1 + 7) / 8 * 8 * sets;
  if (grid > 0x7fffffff || batch > 65535 || g1 > 65535) return RSR_ERR_INVALID_ARGUMENT;  // (16 bits each in a Start)

  plan->rows = (int)T.rows; plan->vstride = (int)h.rows; plan->row0 = (int)T.row0; plan->batch = batch;
  plan->sets = (int)sets; plan->g1 = (int)g1;
  plan->share = (uint32_t)(h.nblocks / g1); plan->share_more = (uint32_t)(h.nblocks % g1);
  plan->grid = grid;
  plan->waves = waves;
  plan->lds = total(nbuf);
  p.nbuf = nbuf; p.buf_magic = magic((uint32_t)nbuf);
  p.nrec = recs(nbuf); p.rec_magic = magic((uint32_t)p.nrec);
  p.off_u = (uint32_t)vbytes;
  p.off_rec = (uint32_t)(vbytes + (size_t)nbuf * p.ubytes);
  p.off_done = (uint32_t)(p.off_rec + (size_t)p.nrec * rec_bytes);
  p.off_blocks = p.off_done + (uint32_t)p.nrec * 4;
  p.off_cnt = p.off_blocks + (uint32_t)p.nrec * 4;
  p.off_epoch = p.off_cnt + (uint32_t)nbuf * 4;
  p.off_ctr = p.off_epoch + (uint32_t)nbuf * 4;
  return RSR_OK;
}

// The words of a planned launch whose workgroups have so many wavefronts.
inline Start start_of(const LaunchPlan& p, int waves) {
  return {(uint32_t)p.sets | p.share_more << 16, magic((uint32_t)p.sets), p.share, (uint32_t)p.rows | (uint32_t)p.vstride << 16,
          (uint32_t)p.row0 | (uint32_t)p.g1 << 16, (uint32_t)p.waves | (uint32_t)waves << 8 | (uint32_t)p.batch << 16};
}

// ---- how many vectors share a pass ----
enum class Mode { one, two, four };
inline const Pass& pass_of(bool i8, Mode m) {
  return m == Mode::four ? (i8 ? kP4 : kF4) : m == Mode::two ? (i8 ? kP2 : kF2) : (i8 ? kI1 : kF1);
}
// Which pass.  A pass over V vectors takes as many times less units and folds, each of which costs more, and stages more rows.  A launch
// is estimated from its plan: how many rounds of workgroups an XCD goes through (the siblings of a block range share one: with fewer
// than eight block ranges some XCDs stay idle), and how long a round takes: the start and the rows staged, and then the longest of what
// keeps the compute unit busy, of a wavefront's units and a fold one after the other, and of the panels that wait for room, where
// there are more than fit (the root of the sum of the squares: none hides the others entirely).  In microseconds.  Float: fitted to the times
// of all three passes of 3222 products with 1024 to 32768 rows, k from 8 to 13 and 2 to 16 vectors, and 290 with 16 to 32768 rows, k from 3 to
// 16 and 2 to 300 vectors.  On 6535 of the former kind and 421 of the latter that nothing was fitted to, the choice is 0.24 and 0.21 % slower than the best of
// the three on average, one in 60 more than 5 % (with the constants before, fitted to kernels whose staging requested four pieces per thread and vector
// whatever the row count: 1.0 and 0.3 %, one in thirteen).  int8: fitted earlier, to 2227 products of both kinds; on 9943 and 661 others 0.7 %, one in 18 more than 5 %.
// `odd` for int8 was fitted by itself to 7245 products with rows that are no multiple of four, as a part of what it was when such rows were staged byte by byte (0.862,
// 1.290, 1.386): a quarter to a half does best on either half of them, and on the other half takes the choice from 0.71 to 0.59 % off the best
// (ternary 9645 x 9664, k = 10, seven vectors: 21.4 us with two per pass, 17.7 with four).  The rule before (rounds of units of the whole device, and a count
// of the units that have room; fitted to 170 products of the first kind): 1.2 and 1.5 %,
// and up to twice the time (ternary 16867 x 47, k = 8, 64 float vectors: 20.0 us with one per pass, 10.4 with two; binary 4868 x 19245,
// k = 11, eleven: 41 and 27).
struct PassCosts {
  double once, round;         // of a launch, of a round of workgroups
  double stage, odd;          // per 64 KB staged, and on top where the rows are no multiple of four (a load and a wait more behind the last piece)
  double share;               // staging per further workgroup on the compute unit
  double unit, second;        // latency of a unit of 48 positions; on top for a wavefront with more than one
  double sum, positions;      // the compute unit busy with 16 units, and with their positions
  double fold, panel, busy;   // latency of a fold of 2048 slots; busy with 16 panels, and with 2048 slots of each
  double wait;                // panels that wait for room
  double crowd;               // exponent of the workgroups that share a compute unit
};
constexpr PassCosts kCosts[2][3] = {  // [int8][one, two, four vectors]
    {{0.766, 2.774, 0.694, 0.158, 0.352, 0.727, 1.507, 1.253, 0.000, 0.097, 0.364, 1.036, 2.005, 0.860},
     {1.577, 2.220, 0.613, 0.225, 1.018, 0.455, 1.729, 0.991, 0.650, 0.597, 0.781, 2.085, 1.909, 0.776},
     {1.062, 3.340, 1.171, 0.477, 0.663, 0.239, 2.039, 0.569, 2.469, 1.300, 1.357, 6.309, 1.828, 0.842}},
    {{1.896, 1.799, 1.295, 0.215, 0.750, 1.035, 1.730, 1.048, 0.039, 0.508, 0.928, 0.785, 1.431, 0.916},
     {1.899, 2.131, 1.123, 0.323, 1.580, 1.094, 1.760, 1.124, 0.122, 0.775, 1.693, 1.448, 1.467, 0.928},
     {2.361, 2.728, 1.370, 0.346, 0.486, 1.444, 0.000, 0.888, 1.562, 0.405, 1.692, 6.280, 1.476, 0.924}}};
// Estimated microseconds of a launch on `cus` compute units, 1e30 if there is none.
inline double pass_time(bool i8, Mode m, const PlanMatrix& h, const PlanTile& T, int batch, int cus, int max_wg_per_cu) {
  const Pass& M = pass_of(i8, m);
  const PassCosts& c = kCosts[i8][(int)m];
  LaunchPlan plan;
  if (plan_tile(M, h, T, false, batch, cus, max_wg_per_cu, &plan) != RSR_OK) return 1e30;
  const KArgs& p = plan.p;
  const double on_xcd = std::max(1.0, cus / 8.0), groups = (double)((plan.g1 + 7) / 8) * plan.sets;
  const double fit = std::max(1.0, std::min(plan.waves == 5 ? 2.0 : (double)(16 / plan.waves), (double)groups_in_lds(plan.lds, h.lds_max)));
  const double rounds = std::max(1.0, std::ceil(groups / (on_xcd * fit))), together = std::min(fit, std::ceil(groups / on_xcd));
  const double blocks = (double)((h.nblocks + plan.g1 - 1) / plan.g1);  // of the largest share
  const double units = blocks * (double)T.nunits / (double)h.nblocks, per_wave = units / plan.waves;
  const double panels = blocks * T.shape.panels, slots = T.shape.nslots / 2048.0;
  const double positions = (double)T.stream_bytes / (48.0 * kPositionBytes * (double)std::max<int64_t>(1, T.nunits));
  const double staged = (double)(T.rows << M.shift) / 65536;
  const double unit = c.unit * positions, fold = c.fold * slots;
  const double busy = std::pow(together, c.crowd) * (units * (c.sum + c.positions * positions) + panels * (c.panel + c.busy * slots)) / 16;
  const double chain = std::max(1.0, per_wave) * unit + (per_wave > 1 ? c.second : 0.0) + fold;
  const double room = c.wait * std::max(0.0, panels / p.nbuf - 1) * (unit + fold);
  return c.once + rounds * (c.round + (c.stage + (T.rows % 4 ? c.odd : 0.0)) * staged * (1 + c.share * (together - 1)) +
                            std::sqrt(busy * busy + chain * chain + room * room));
}
inline Mode shortest(const double (&time)[3]) { return time[2] < time[1] && time[2] < time[0] ? Mode::four : time[1] < time[0] ? Mode::two : Mode::one; }
inline Mode pick_mode(bool i8, const PlanMatrix& h, const PlanTile& T, int batch, int cus, int max_wg_per_cu) {
  if (h.step2_plain || batch < 2) return Mode::one;
  double time[3];
  for (const Mode m : {Mode::one, Mode::two, Mode::four}) time[(int)m] = pass_time(i8, m, h, T, batch, cus, max_wg_per_cu);
  return shortest(time);
}

// The launch of one row tile's product.
inline int plan_product(bool i8, const PlanMatrix& h, const PlanTile& T, bool accumulate, int batch, Mode* mode, LaunchPlan* plan) {
  constexpr int most = 4;  // workgroups per compute unit
  *mode = pick_mode(i8, h, T, batch, h.num_cu, most);
  return plan_tile(pass_of(i8, *mode), h, T, accumulate, batch, h.num_cu, most, plan);
}

// The compute units of several products that share a launch, in proportion to the bytes of their tables: multiples of 8
// (one per XCD), at least 8, together no more than the device has (a workgroup that has to wait for a free compute unit
// would start when the others are nearly done).
inline void split_device(const int64_t* bytes, int njobs, int num_cu, int* share) {
  double bytes_total = 0;
  for (int j = 0; j < njobs; ++j) bytes_total += (double)bytes[j] + 1.0;
  int given = 0;
  for (int j = 0; j < njobs; ++j) {
    share[j] = std::max(8, (int)((double)num_cu * ((double)bytes[j] + 1.0) / bytes_total) / 8 * 8);
    given += share[j];
  }
  while (given > num_cu) {
    int big = 0;
    for (int j = 1; j < njobs; ++j) if (share[j] > share[big]) big = j;
    if (share[big] <= 8) break;
    share[big] -= 8; given -= 8;
  }
  while (given + 8 <= num_cu) {  // what is left over goes to the products with the most bytes per compute unit
    int best = 0;
    for (int j = 1; j < njobs; ++j)
      if ((double)bytes[j] / share[j] > (double)bytes[best] / share[best]) best = j;
    share[best] += 8; given += 8;
  }
}

// One launch for several products.
struct SharedJob {
  const PlanMatrix* h;
  const PlanTile* T;
  int64_t bytes;  // of its tables
};
constexpr int kMaxJobs = 8;
// The pass in which the product that takes longest on its share takes least, or narrower until all of them fit (a narrower pass has
// more sets of vectors, so fewer workgroups a set and more blocks a workgroup: that one product fits does not say that all do).  On
// failure *failed is the product that has no launch.
inline int plan_shared(bool i8, const SharedJob* jobs, int njobs, int num_cu, int batch, Mode* mode, LaunchPlan* plans, int* failed) {
  int64_t bytes[kMaxJobs];
  int share[kMaxJobs];
  for (int j = 0; j < njobs; ++j) bytes[j] = jobs[j].bytes;
  split_device(bytes, njobs, num_cu, share);
  double time[3] = {0, 0, 0};
  bool one = batch < 2;
  for (int j = 0; j < njobs; ++j) {
    share[j] = std::min(share[j], jobs[j].h->num_cu);
    one = one || jobs[j].h->step2_plain;
  }
  for (const Mode m : {Mode::one, Mode::two, Mode::four})
    for (int j = 0; j < njobs && !one; ++j) time[(int)m] = std::max(time[(int)m], pass_time(i8, m, *jobs[j].h, *jobs[j].T, batch, share[j], 1));
  const Mode most = one ? Mode::one : shortest(time);
  int rc = RSR_OK;
  for (const Mode m : {Mode::four, Mode::two, Mode::one}) {
    if (m > most) continue;
    rc = RSR_OK;
    for (int j = 0; j < njobs && rc == RSR_OK; ++j) {
      *failed = j;
      rc = plan_tile(pass_of(i8, m), *jobs[j].h, *jobs[j].T, false, batch, share[j], 1, &plans[j]);
    }
    if (rc == RSR_OK) { *mode = m; break; }
  }
  return rc;
}

// How many of the q bit planes of a matrix share a launch: as many as leave room for their records beside the activations.
inline int planes_per_handle(int64_t rows, int k, int q) {
  const int64_t height = std::min<int64_t>(rows, kTileRows);
  for (int n = q; n > 1; --n) {
    const Shape s = panel_shape(height, k, n, false);
    const int64_t lds = align_up((size_t)(height + 1) * 4, 16) + 2 * (int64_t)(s.nslots + kDummySlots + kMaxExtras) * 4 +
                        2 * ((int64_t)s.panels * kItems * 4 + 8) + 64;
    if (lds <= 160 * 1024) return n;
  }
  return 1;
}

}  // namespace rsr
#endif  // RSR_PLAN_H_
