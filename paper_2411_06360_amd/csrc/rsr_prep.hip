// Algorithm 1 (Section 3.4) on the device: the index of a matrix in device memory is built there, in the layout of
// rsr_layout.h.
//
//   1. values_kernel     the k-bit value of every row in every column block and part (Definition 3.2,
//                        first column most significant; a narrow last block is shifted left).
//   2. sort_kernel       per (block, part), by one wavefront: histogram of the values, its exclusive prefix
//                        (the full segmentation L of Section 3.3) and the counting sort that gives sigma
//                        ("bucket sort" in the proof of Theorem 3.6).
//   3. plan_kernel       per panel: the segments ranked by their number of rows, the groups they form, how many
//                        units and stream bytes those take.
//      begin_kernel      where every panel's units and streams begin, and what there is in all (which the host reads to
//                        allocate the tables).
//   4. units_kernel      per panel: the unit descriptors, the block offsets, the slots of cut segments.
//   5. emit_kernel       per half of a unit: the rows dealt out to the lanes, the rows of a lane's segment spread over the
//                        LDS banks, granule order.
//
// Steps 1 to 3 and 4 to 5 run over all column blocks at once where a grid can hold their panels and the device has the
// working memory, otherwise over as many blocks at a time as that allows (steps 1 to 3 then run twice per block: once to
// find how large the tables are, once more ahead of steps 4 and 5).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/rsr.h"
#include "rsr_internal.h"
#include "rsr_layout.h"

namespace {

using rsr::PUnit;

#define PREP_TRY(expr)                                                        \
  do {                                                                        \
    hipError_t e_ = (expr);                                                   \
    if (e_ != hipSuccess) {                                                   \
      (void)hipGetLastError();                                                \
      *err = std::string(#expr) + ": " + hipGetErrorString(e_);               \
      return RSR_ERR_HIP;                                                     \
    }                                                                         \
  } while (0)

// flags[workgroup], bit 0: some entry is -1, bit 1: some entry lies outside {-1,0,1}.  Bound by the reading of A: 16 bytes per load
// where A is aligned.  A word per workgroup, added up by the host: with one word for all, most wavefronts of a ternary matrix
// reached their atomic before the first of them was seen (ternary 4096^2: 58 us, 6.4 now).
constexpr int kKindGroups = 1024;
__global__ void kind_kernel(const int8_t* __restrict__ A, int64_t count, unsigned* __restrict__ flags) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  unsigned f = 0;
  auto look = [&](int x) {
    if (x < -1 || x > 1) f |= 2u;
    if (x == -1) f |= 1u;
  };
  const int64_t n16 = (reinterpret_cast<uintptr_t>(A) & 15) == 0 ? count / 16 : 0;
  for (int64_t i = id; i < n16; i += step) {
    const uint4 x = reinterpret_cast<const uint4*>(A)[i];
    const uint32_t d[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int b = 0; b < 4; ++b) look((int)(d[j] << (24 - 8 * b)) >> 24);
  }
  for (int64_t i = n16 * 16 + id; i < count; i += step) look(A[i]);
  __shared__ unsigned seen;
  if (threadIdx.x == 0) seen = 0;
  __syncthreads();
  const unsigned all = (__any((int)(f & 1u)) ? 1u : 0u) | (__any((int)(f & 2u)) ? 2u : 0u);
  if ((threadIdx.x & 63) == 0 && all) atomicOr(&seen, all);
  __syncthreads();
  if (threadIdx.x == 0) flags[blockIdx.x] = seen;
}

// val[(block * parts + part) * rows + r].  A workgroup takes 64 rows of kValueBlocks column blocks through LDS, so that
// A is read in whole lines and the values are written in runs of 64 rows.
constexpr int kValueBlocks = 8;
constexpr int kValueStride = kValueBlocks * rsr::kMaxK + 4;  // bytes between rows in LDS: an odd number of dwords
__global__ void __launch_bounds__(256)
values_kernel(const int8_t* __restrict__ A, int rows, int cols, int64_t ld, int k, int parts, int plane0, int nblocks, uint16_t* __restrict__ val) {
  __shared__ __align__(16) int8_t tile[64 * kValueStride];
  const int r0 = blockIdx.x * 64, tid = threadIdx.x;
  for (int b0 = blockIdx.y * kValueBlocks; b0 < nblocks; b0 += gridDim.y * kValueBlocks) {
    const int c0 = b0 * k, nc = min(kValueBlocks * k, cols - c0), nr = min(64, rows - r0);
    const int8_t* a = A + (int64_t)r0 * ld + c0;
    const bool words = ((reinterpret_cast<uintptr_t>(a) | (uintptr_t)ld) & 3) == 0;
    const int nw = words ? nc / 4 : 0;
    for (int i = tid; i < nr * nw; i += 256) {
      const int r = i / nw, c = i - r * nw;
      reinterpret_cast<uint32_t*>(tile + r * kValueStride)[c] = reinterpret_cast<const uint32_t*>(a + (int64_t)r * ld)[c];
    }
    const int rest = nc - nw * 4;
    for (int i = tid; i < nr * rest; i += 256) {
      const int r = i / rest, c = nw * 4 + i - r * rest;
      tile[r * kValueStride + c] = a[(int64_t)r * ld + c];
    }
    __syncthreads();
    for (int i = tid; i < 64 * kValueBlocks; i += 256) {
      const int r = i & 63, bi = i >> 6, b = b0 + bi;
      if (r < nr && b < nblocks) {
        const int width = min(k, cols - b * k), shift = k - width;
        const int8_t* t = tile + r * kValueStride + bi * k;
        uint16_t* out = val + (int64_t)b * parts * rows + r0 + r;
        if (plane0 >= 0) {  // bit planes of q-bit entries
          for (int p = 0; p < parts; ++p) {
            uint32_t x = 0;
            for (int c = 0; c < width; ++c) x = (x << 1) | (((uint32_t)(uint8_t)t[c] >> (plane0 + p)) & 1u);
            out[(int64_t)p * rows] = (uint16_t)(x << shift);
          }
        } else {
          uint32_t plus = 0, minus = 0;
          for (int c = 0; c < width; ++c) {
            const int x = t[c];
            plus = (plus << 1) | (uint32_t)(x == 1);
            minus = (minus << 1) | (uint32_t)(x == -1);
          }
          out[0] = (uint16_t)(plus << shift);
          if (parts == 2) out[rows] = (uint16_t)(minus << shift);
        }
      }
    }
    __syncthreads();
  }
}

// One wavefront per (block, part).  LDS: 2^k counters of 16 bits per wavefront (a tile has at most 32768 rows).  Both
// passes are LDS atomics of one wavefront, 64 rows per instruction, in row order; the counters are private to
// the wavefront, so the result does not depend on timing.
__global__ void sort_kernel(const uint16_t* __restrict__ val, int rows, int k, int nbp, int waves_per_wg,
                            uint32_t* __restrict__ off, uint16_t* __restrict__ sigma) {
  extern __shared__ uint32_t lds_hist[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int bp = blockIdx.x * waves_per_wg + wave;
  if (bp >= nbp) return;  // (no barriers below: the wavefronts are independent)
  const int nvals = 1 << k;
  const int ndw = max(1, nvals >> 1);
  uint32_t* const h = lds_hist + (size_t)wave * ndw;  // (counted up with atomics: what other lanes have counted is read behind a barrier to the compiler)
  const uint16_t* v = val + (int64_t)bp * rows;
  for (int i = lane; i < ndw; i += 64) h[i] = 0;
  constexpr int kAhead = 8;  // chunks of 64 rows whose values are fetched together
  for (int r0 = 0; r0 < rows; r0 += 64 * kAhead) {
    uint32_t x[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) x[j] = v[min(r0 + 64 * j + lane, rows - 1)];
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
      if (r0 + 64 * j + lane < rows) atomicAdd(&h[x[j] >> 1], 1u << (16 * (x[j] & 1)));
  }
  asm volatile("" ::: "memory");
  // exclusive prefix: the full segmentation (kept in LDS as the next free position of every value)
  uint32_t carry = 0;
  uint32_t* o = off + (int64_t)bp * (nvals + 1);
  for (int i0 = 0; i0 < ndw; i0 += 64) {
    const int i = i0 + lane;
    const uint32_t w = i < ndw ? h[i] : 0u;
    const uint32_t c0 = w & 0xffffu, c1 = w >> 16;
    uint32_t s = c0 + c1;
    uint32_t incl = s;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const uint32_t t = __shfl_up(incl, d);
      if (lane >= d) incl += t;
    }
    const uint32_t start0 = carry + incl - s, start1 = start0 + c0;
    if (i < ndw) {
      h[i] = start0 | (start1 << 16);
      o[2 * i] = start0;
      if (2 * i + 1 < nvals) o[2 * i + 1] = start1;
    }
    carry += __shfl(incl, 63);
  }
  asm volatile("" ::: "memory");
  if (lane == 0) o[nvals] = (uint32_t)rows;
  uint16_t* sg = sigma + (int64_t)bp * rows;
  for (int r0 = 0; r0 < rows; r0 += 64 * kAhead) {
    uint32_t x[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) x[j] = v[min(r0 + 64 * j + lane, rows - 1)];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int r = r0 + 64 * j + lane;
      if (r < rows) {
        const uint32_t sh = 16 * (x[j] & 1);
        const uint32_t at = (atomicAdd(&h[x[j] >> 1], 1u << sh) >> sh) & 0xffffu;
        sg[at] = (uint16_t)r;
      }
    }
  }
}

// What the kernels below need to know of a tile.
struct Geometry {
  int rows, k, parts;
  uint32_t block0, panel0;  // first column block and panel of this run: the lists below count from them
  rsr::Shape s;
  int list_stride, group_stride, extra_stride;  // entries per panel in the lists
  int fill;  // absent values form groups of no rows
};

struct PanelInfo {
  uint32_t n8, n1;         // list entries that take 8 lanes, one lane
  uint32_t units, stream;  // stream in multiples of kStreamAlign
  uint32_t extras, rows, segments;
};
struct PanelBase {
  uint32_t unit, stream;
};

constexpr int kKeys8 = 32, kKeys1 = 48;  // rank classes: 8 lanes with 32 .. 1 rows each, one lane with 47 .. 0
constexpr int kKeys = kKeys8 + kKeys1;
static_assert(8 * kKeys8 == rsr::kWideRows, "eight lanes hold a piece of kWideRows rows");
static_assert(kKeys1 - 1 <= rsr::kWideRows && kKeys1 <= rsr::kMaxPositions && kKeys8 + 1 <= rsr::kMaxPositions, "a group and its head fit in a unit");
constexpr uint16_t kNoSegment = 0xffff;  // the number of rows of a slot that takes no part

// The pieces a segment of n rows is cut into.
__device__ __forceinline__ uint32_t pieces_of(uint32_t n) { return n <= (uint32_t)rsr::kWideRows ? 1u : (n + rsr::kWideRows - 1) / rsr::kWideRows; }
// Its rank class, the widest and longest first.  `cap`: rows up to which a segment takes one lane.
__device__ __forceinline__ int key_of(uint32_t n, int cap) {
  if (n <= (uint32_t)cap) return kKeys8 + (kKeys1 - 1 - (int)n);
  const uint32_t np = pieces_of(n), piece = (n + np - 1) / np;
  return kKeys8 - (int)((piece + 7) / 8);
}
__device__ __forceinline__ int rows_of_key(int key) {  // positions a group of this class takes, without its head
  return key < kKeys8 ? kKeys8 - key : kKeys8 + kKeys1 - 1 - key;
}

// Rows per group of a panel, in LDS, for a wavefront that walks them together: 64 at a time in a register.
struct GroupRows {
  const uint8_t* rows;
  int lane;
  uint32_t base = 0xffffffffu;
  int held = 0;
  __device__ __forceinline__ uint32_t operator()(uint32_t i) {  // i: the same for all lanes
    i = (uint32_t)__builtin_amdgcn_readfirstlane((int)i);
    if ((i & ~63u) != base) { base = i & ~63u; held = rows[base + lane]; }
    return (uint32_t)__builtin_amdgcn_readlane(held, (int)(i & 63));
  }
};
// The units of a panel: whole groups of one width, in order, at most kMaxPositions positions and about equally many
// each.  By a whole wavefront.  f(wide, first list entry, first group, groups, positions) for every unit.
template <typename F>
__device__ __forceinline__ void walk_units(const PanelInfo& I, GroupRows group_rows, F f) {
  uint32_t group = 0, entry = 0;
#pragma unroll 1
  for (int wide = 1; wide >= 0; --wide) {
    const uint32_t per = wide ? 8u : 64u, count = wide ? I.n8 : I.n1;
    const uint32_t ng = (count + per - 1) / per;
    uint32_t all = 0;
    for (uint32_t i = (uint32_t)group_rows.lane; i < ng; i += 64) all += group_rows.rows[group + i] + 1u;
#pragma unroll
    for (int d = 32; d > 0; d /= 2) all += __shfl_xor(all, d);
    all = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
    const uint32_t nu = (all + rsr::kMaxPositions - 5) / (rsr::kMaxPositions - 4);
    const uint32_t target = nu ? (all + nu - 1) / nu : 0;
    uint32_t first = 0, cur = 0;
    for (uint32_t i = 0; i < ng; ++i) {
      const uint32_t m = group_rows(group + i) + 1;
      if (cur && (cur >= target || cur + m > (uint32_t)rsr::kMaxPositions)) {
        f(wide, entry + first * per, group + first, i - first, cur);
        first = i; cur = 0;
      }
      cur += m;
    }
    if (cur) f(wide, entry + first * per, group + first, ng - first, cur);
    group += ng;
    entry += count;
  }
}

// Part and value of a slot of a panel (counted from g.panel0); false: no segment belongs to it.
__device__ __forceinline__ bool slot_value(const Geometry& g, uint32_t panel, uint32_t slot, uint32_t* bp, uint32_t* value) {
  const uint32_t block = panel / g.s.panels, pi = panel % g.s.panels;
  const int wbits = g.k - g.s.kc;
  const uint32_t part = g.s.both ? slot / g.s.pslots : pi >> wbits;
  const uint32_t low = slot % g.s.pslots, window = g.s.both ? 0u : pi & ((1u << wbits) - 1);
  *bp = block * g.parts + part;
  *value = (window << g.s.kc) | low;
  return low < (1u << g.s.kc) && *value != 0;
}

// One workgroup per panel.  A chain of short steps on LDS counters: bound by their latency; several workgroups share a
// compute unit.  (With the limits' costs, the classes' sums and the walk over the groups each by single lanes: 59 us at ternary
// 4096^2, k = 10; 47 without; 39 now that offsets are fetched four at a time and a thread adds up a class, most of it the ranking by one wavefront and
// the places in the list.)
__global__ void __launch_bounds__(256)
plan_kernel(Geometry g, const uint32_t* __restrict__ off, uint16_t* __restrict__ list_all, uint8_t* __restrict__ group_all,
            uint32_t* __restrict__ extra_all, PanelInfo* __restrict__ info) {
  __shared__ uint16_t len[rsr::kMaxPanelSlots], rank[rsr::kMaxPanelSlots], list[rsr::kMaxPanelSlots + rsr::kMaxExtras];
  __shared__ __align__(4) uint16_t cnt[kKeys][64];
  __shared__ uint32_t hist[rsr::kWideRows + 1], above[rsr::kWideRows + 2], start[kKeys + 1], ex_slot[rsr::kMaxExtras];
  __shared__ uint16_t ex_rank[rsr::kMaxExtras];
  __shared__ uint8_t ex_key[rsr::kMaxExtras], groups[1024];
  __shared__ uint32_t cost[8], tot_rows, tot_segments, n_extra, best_cap;
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t panel = blockIdx.x;
  const int caps[7] = {47, 32, 24, 16, 12, 8, 6};
  for (int i = tid; i < kKeys * 64; i += 256) (&cnt[0][0])[i] = 0;
  for (int i = tid; i <= rsr::kWideRows; i += 256) hist[i] = 0;
  if (tid == 0) { tot_rows = 0; tot_segments = 0; n_extra = 0; }
  if (tid < 7) cost[tid] = 0;
  __syncthreads();
  {
    uint32_t my_rows = 0, my_segments = 0;
    constexpr int kTogether = 4;  // slots of a thread whose offsets are fetched together
    for (int s0 = tid; s0 < g.s.nslots; s0 += 256 * kTogether) {
      uint32_t o0[kTogether], o1[kTogether];
      bool real[kTogether];
#pragma unroll
      for (int j = 0; j < kTogether; ++j) {
        const uint32_t s = (uint32_t)min(s0 + 256 * j, g.s.nslots - 1);
        uint32_t bp, value;
        real[j] = slot_value(g, panel, s, &bp, &value);
        const uint32_t* o = off + (int64_t)bp * ((1 << g.k) + 1) + (real[j] ? value : 0u);
        o0[j] = o[0]; o1[j] = o[1];
      }
#pragma unroll
      for (int j = 0; j < kTogether; ++j) {
        const int s = s0 + 256 * j;
        if (s >= g.s.nslots) break;
        const uint32_t n = real[j] ? o1[j] - o0[j] : 0u;
        len[s] = n || (real[j] && g.fill) ? (uint16_t)n : kNoSegment;
        if (n) {
          my_rows += n; ++my_segments;
          if (n <= (uint32_t)rsr::kWideRows) atomicAdd(&hist[n], 1u);
        }
      }
    }
    atomicAdd(&tot_rows, my_rows);
    atomicAdd(&tot_segments, my_segments);
  }
  __syncthreads();
  // Up to how many rows a segment takes one lane: the limit that gives the fewest positions.  Thread t stands for the segments of
  // n = t + 1 rows: with `more` longer ones (above[n]: those of n rows and more) they begin ceil(..) further groups of n rows.
  {
    const int n = tid + 1;
    uint32_t sum = 0;
    if (tid < 64) {  // suffix sums of the histogram, four lengths per lane
      uint32_t part[4];
#pragma unroll
      for (int i = 3; i >= 0; --i) { sum += hist[4 * lane + i + 1]; part[i] = sum; }
      uint32_t after = sum;
#pragma unroll
      for (int d = 1; d < 64; d *= 2) {
        const uint32_t t = __shfl_down(after, d);
        if (lane + d < 64) after += t;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) above[4 * lane + i + 1] = part[i] + after - sum;
      if (lane == 0) above[rsr::kWideRows + 1] = 0;
    }
    __syncthreads();
    const uint32_t with = above[n], more = above[n + 1];
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      uint32_t mine = 0;
      if (n > caps[c]) {
        mine = ((with + 7) / 8 - (more + 7) / 8) * (uint32_t)((n + 7) / 8 + 1);
      } else {
        const uint32_t wide = above[caps[c] + 1];
        mine = ((with - wide + 63) / 64 - (more - wide + 63) / 64) * (uint32_t)(n + 1);
      }
#pragma unroll
      for (int d = 32; d > 0; d /= 2) mine += __shfl_xor(mine, d);
      if (lane == 0) atomicAdd(&cost[c], mine);
    }
  }
  __syncthreads();
  if (tid == 0) {
    int b = 0;
    for (int i = 1; i < 7; ++i) if (cost[i] < cost[b]) b = i;
    best_cap = (uint32_t)caps[b];
  }
  __syncthreads();
  const int cap = (int)best_cap;
  // Ranks: by class, and inside a class round robin over the 64 residues of the slot, so that the slots of
  // neighbouring lanes lie in different LDS banks.  One wavefront counts, lane = residue.
  if (tid < 64) {
    uint32_t extras = 0;
    for (int s0 = 0; s0 < g.s.nslots; s0 += 64) {
      const uint32_t n = len[s0 + lane];
      const bool in = n != kNoSegment;
      if (in) {
        const int key = key_of(n, cap);
        const uint16_t r = cnt[key][lane];
        rank[s0 + lane] = r; cnt[key][lane] = r + 1;
      }
      unsigned long long cut = __ballot(in && n > (uint32_t)rsr::kWideRows);
      while (cut) {
        const int l = __ffsll((long long)cut) - 1;
        cut &= cut - 1;
        const uint32_t n_l = (uint32_t)__shfl((int)n, l), np = pieces_of(n_l);
        const int key_l = key_of(n_l, cap);
        for (uint32_t i = 1; i < np; ++i) {
          const uint32_t e = extras++;
          if (lane == (int)(e & 63) && e < (uint32_t)g.extra_stride) {  // (pieces beyond the first: at most rows / kWideRows in all)
            ex_slot[e] = (uint32_t)(s0 + l) | (i << 16);
            ex_key[e] = (uint8_t)key_l;
            const uint16_t r = cnt[key_l][lane];
            ex_rank[e] = r; cnt[key_l][lane] = r + 1;
          }
        }
      }
    }
    if (lane == 0) n_extra = min(extras, (uint32_t)g.extra_stride);
  }
  __syncthreads();
  if (tid < kKeys) {  // a thread per class, two residues at a time, every thread from another bank on
    const uint32_t* const pairs = reinterpret_cast<const uint32_t*>(cnt[tid]);
    uint32_t s = 0;
#pragma unroll 8
    for (int i = 0; i < 32; ++i) {
      const uint32_t two = pairs[(i + tid) & 31];
      s += (two & 0xffffu) + (two >> 16);
    }
    start[tid + 1] = s;
  }
  __syncthreads();
  if (tid < 64) {  // prefix sums over the classes, two per lane
    static_assert(kKeys <= 128 && kKeys % 2 == 0, "two classes per lane");
    const bool in = 2 * lane < kKeys;
    const uint32_t a = in ? start[2 * lane + 1] : 0u, b = in ? start[2 * lane + 2] : 0u;
    uint32_t incl = a + b;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const uint32_t t = __shfl_up(incl, d);
      if (lane >= d) incl += t;
    }
    if (in) { start[2 * lane + 1] = incl - b; start[2 * lane + 2] = incl; }
    if (lane == 0) start[0] = 0;
  }
  __syncthreads();
  auto place = [&](int key, uint32_t r, int residue) {
    uint32_t at = start[key];
#pragma unroll 8
    for (int i = 0; i < 64; ++i) {
      const int c = (i + lane) & 63;
      at += min((uint32_t)cnt[key][c], r + (c < residue ? 1u : 0u));
    }
    return at;
  };
  for (int s = tid; s < g.s.nslots; s += 256)
    if (len[s] != kNoSegment) list[place(key_of(len[s], cap), rank[s], s & 63)] = (uint16_t)s;
  if (tid < (int)n_extra) list[place(ex_key[tid], ex_rank[tid], tid & 63)] = (uint16_t)(g.s.nslots + rsr::kDummySlots + tid);
  __syncthreads();
  const uint32_t n8 = start[kKeys8], n1 = start[kKeys] - n8, g8 = (n8 + 7) / 8, ng = g8 + (n1 + 63) / 64;
  uint8_t* group_out = group_all + (int64_t)panel * g.group_stride;
  for (uint32_t i = tid; i < ng; i += 256) {
    const uint32_t at = i < g8 ? i * 8 : n8 + (i - g8) * 64;
    const uint32_t s = list[at];
    const int key = s < (uint32_t)g.s.nslots ? key_of(len[s], cap) : (int)ex_key[s - g.s.nslots - rsr::kDummySlots];
    groups[i] = (uint8_t)rows_of_key(key);
    group_out[i] = groups[i];
  }
  uint16_t* list_out = list_all + (int64_t)panel * g.list_stride;
  for (uint32_t i = tid; i < start[kKeys]; i += 256) list_out[i] = list[i];
  if (tid < (int)n_extra) extra_all[(int64_t)panel * g.extra_stride + tid] = ex_slot[tid];
  __syncthreads();
  if (tid < 64) {
    PanelInfo I;
    I.n8 = n8; I.n1 = n1;
    I.units = 0; I.stream = 0;
    I.extras = n_extra; I.rows = tot_rows; I.segments = tot_segments;
    walk_units(I, GroupRows{groups, lane},
               [&](int, uint32_t, uint32_t, uint32_t, uint32_t npos) { ++I.units; I.stream += (npos + 1) & ~1u; });
    if (I.units == 0) I.units = 1;  // a panel without entries still has to count for its block
    if (lane == 0) info[panel] = I;
  }
}

// What the panels of a tile come to: read by the host when the last of them is planned.
struct Totals {
  unsigned long long units, stream, rows, segments, groups;  // stream in multiples of kStreamAlign
  uint32_t block_units, extras;                              // of a block, of a panel, at most
};

// One workgroup: prefix sums over the panels of a run (`totals` holds those of the runs before; `first`: there are none).  A panel is a thread.
// Bound by a chain: a read of memory, lane exchanges, the wavefronts' sums, a second read for the units of whole blocks.  (The sizes of all panels used
// to be copied to the host, added up there and copied back, the slots of cut segments as well: five copies of 13 to 30 us.  Ternary 4096^2 with
// product and release 324 us, 303 so.)
constexpr int kBeginThreads = 1024;
__global__ void __launch_bounds__(kBeginThreads)
begin_kernel(int panels_per_block, uint32_t panels, bool first, const PanelInfo* __restrict__ info, PanelBase* base, Totals* __restrict__ totals) {
  typedef unsigned long long u64;
  // (a turn's sums fit 32 bits: a panel's units fit 16)
  static_assert((u64)kBeginThreads * 0xffffu * rsr::kMaxPositions < (1ull << 32));
  constexpr int kWaves = kBeginThreads / 64;
  __shared__ uint32_t wave_units[kWaves], wave_stream[kWaves], block_units, extras;
  __shared__ u64 rows, segments, groups;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) { rows = segments = groups = 0; block_units = extras = 0; }
  u64 units = first ? 0 : totals->units, stream = first ? 0 : totals->stream;  // of the panels ahead of this turn
  u64 my_rows = 0, my_segments = 0, my_groups = 0;
  uint32_t my_extras = 0;
  for (uint32_t p0 = 0; p0 < panels; p0 += nt) {
    const uint32_t p = p0 + tid;
    PanelInfo I{};
    if (p < panels) I = info[p];
    uint32_t u = I.units, st = I.stream;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const uint32_t x = __shfl_up(u, d), y = __shfl_up(st, d);
      if (lane >= d) { u += x; st += y; }
    }
    if (lane == 63) { wave_units[wave] = u; wave_stream[wave] = st; }
    __syncthreads();
    uint32_t all_units = 0, all_stream = 0;
    for (int w = 0; w < nt / 64; ++w) {
      if (w == wave) { u += all_units; st += all_stream; }
      all_units += wave_units[w]; all_stream += wave_stream[w];
    }
    if (p < panels) base[p] = PanelBase{(uint32_t)units + u - I.units, (uint32_t)stream + st - I.stream};
    units += all_units; stream += all_stream;
    my_rows += I.rows; my_segments += I.segments; my_groups += (I.n8 + 7) / 8 + (I.n1 + 63) / 64;
    my_extras = max(my_extras, I.extras);
    __syncthreads();  // (the wavefronts' sums are read; and behind it the panels' beginnings are there for the whole workgroup)
  }
  uint32_t my_units = 0;
  for (uint32_t b = tid; b < panels / panels_per_block; b += nt) {
    const uint32_t next = (b + 1) * panels_per_block;
    my_units = max(my_units, (next < panels ? base[next].unit : (uint32_t)units) - base[b * panels_per_block].unit);
  }
#pragma unroll
  for (int d = 32; d > 0; d /= 2) {
    my_rows += __shfl_xor(my_rows, d); my_segments += __shfl_xor(my_segments, d); my_groups += __shfl_xor(my_groups, d);
    my_units = max(my_units, (uint32_t)__shfl_xor(my_units, d)); my_extras = max(my_extras, (uint32_t)__shfl_xor(my_extras, d));
  }
  if (lane == 0) {
    atomicAdd(&rows, my_rows); atomicAdd(&segments, my_segments); atomicAdd(&groups, my_groups);
    atomicMax(&block_units, my_units); atomicMax(&extras, my_extras);
  }
  __syncthreads();
  if (tid == 0) {
    Totals t{};
    if (!first) t = *totals;
    t.units = units; t.stream = stream;
    t.rows += rows; t.segments += segments; t.groups += groups;
    t.block_units = max(t.block_units, block_units); t.extras = max(t.extras, extras);
    *totals = t;
  }
}

// One wavefront per panel.  `extra_slots`: null if no segment of the tile is cut.
__global__ void __launch_bounds__(64)
units_kernel(Geometry g, int nblocks, uint32_t nunits, const uint8_t* __restrict__ group_all, const PanelInfo* __restrict__ info,
             const PanelBase* __restrict__ base, const uint32_t* __restrict__ extra_all, PUnit* __restrict__ units, uint32_t* __restrict__ blk_unit,
             uint16_t* __restrict__ extra_slots) {
  __shared__ uint8_t groups[1024];
  const uint32_t panel = blockIdx.x;
  const PanelInfo I = info[panel];
  if (panel % g.s.panels == 0 && threadIdx.x == 0) {
    const uint32_t block = g.block0 + panel / g.s.panels;
    blk_unit[block] = base[panel].unit;
    if (block + 1 == (uint32_t)nblocks) blk_unit[nblocks] = nunits;
  }
  if (extra_slots)
    for (uint32_t i = threadIdx.x; i < (uint32_t)g.extra_stride; i += 64)
      extra_slots[(size_t)(g.panel0 + panel) * g.extra_stride + i] = i < I.extras ? (uint16_t)(extra_all[(int64_t)panel * g.extra_stride + i] & 0xffffu) : (uint16_t)0;
  const uint32_t ng = (I.n8 + 7) / 8 + (I.n1 + 63) / 64;
  for (uint32_t i = threadIdx.x; i < ng; i += 64) groups[i] = group_all[(int64_t)panel * g.group_stride + i];
  __syncthreads();
  const int lane = threadIdx.x;
  PUnit u;
  u.block = g.block0 + panel / g.s.panels; u.panel = g.panel0 + panel;
  u.units_in_panel = (uint16_t)I.units; u.extras = (uint16_t)I.extras; u.reserved = 0;
  uint32_t at = base[panel].unit, stream = base[panel].stream;
  if (ng == 0) {
    u.stream_off = stream; u.heads_lo = 0; u.heads_hi = 0; u.npos = 0; u.wide = 0; u.first = 0;
    if (lane == 0) units[at] = u;
    return;
  }
  GroupRows rows{groups, lane};
  walk_units(I, rows,
             [&](int wide, uint32_t first, uint32_t group, uint32_t n, uint32_t npos) {
               uint64_t heads = 0;
               uint32_t p = 0;
               for (uint32_t i = 0; i < n; ++i) { p += rows(group + i); heads |= 1ull << p; ++p; }
               u.stream_off = stream;
               u.heads_lo = (uint32_t)heads; u.heads_hi = (uint16_t)(heads >> 32);
               u.npos = (uint8_t)((npos + 1) & ~1u); u.wide = (uint8_t)wide;
               u.first = first;
               if (lane == 0) units[at] = u;
               ++at;
               stream += (npos + 1) & ~1u;
             });
}

// One wavefront per half of a unit (lanes 0 to 31 or 32 to 63 of those that will sum it: the LDS serves the halves one after the other, so
// that their banks have nothing to do with each other).  Two lanes work on every column of rows: they collect every other group's rows and
// heads in LDS (ent), let the rows of every segment trade places in two halves of the unit, and write every other granule.  Bound by the latency
// of chains - list, offsets, rows from memory; entries, bank loads, exchange in LDS - so four groups go through the first together, and
// there are twice as many and half as long chains as with a wavefront per unit (ternary 4096^2, k = 10: 60 us so, 45 now).
constexpr int kEmitWaves = 4;
constexpr int kGroupsAtOnce = 4;
constexpr int kReach = 3;        // positions a row may move per trade
constexpr int kTradeRounds = 2;  // times every lane looks at every row of its segments
__global__ void __launch_bounds__(64 * kEmitWaves)
emit_kernel(Geometry g, uint32_t nunits, const PUnit* __restrict__ units, const PanelInfo* __restrict__ info, const uint16_t* __restrict__ list_all,
            const uint32_t* __restrict__ extra_all, const uint32_t* __restrict__ off, const uint16_t* __restrict__ sigma,
            unsigned char* __restrict__ stream) {
  __shared__ uint16_t ent_all[kEmitWaves][rsr::kMaxPositions + kReach][32];
  __shared__ uint32_t load_all[kEmitWaves][rsr::kMaxPositions + kReach][8];  // rows per LDS bank (a byte each) and position
  __shared__ uint8_t ends_all[kEmitWaves][rsr::kMaxPositions];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t ui = (blockIdx.x * kEmitWaves + wave) / 2;
  if (ui >= nunits) return;  // (no barriers below: the wavefronts are independent)
  const int half = wave & 1, c = lane & 31, turn = lane >> 5;  // the lane's column of the half, and which of its two lanes it is
  const uint32_t column_lane = (uint32_t)(half * 32 + c);      // the lane that will sum it
  const PUnit U = units[ui];
  const int npos = U.npos;
  if (npos == 0) return;
  // (Plain accesses, and a barrier to the compiler where other lanes' atomics have to be seen: volatile ones through these pointers are
  // flat instructions, each with a wait of its own - 2000 clocks for every position of a trade round.)
  uint16_t (*const ent)[32] = ent_all[wave];
  uint32_t* const load_words = &load_all[wave][0][0];
  uint8_t* const ends = ends_all[wave];
  auto settle = []() { asm volatile("" ::: "memory"); };
  auto add_load = [&](int p, int b) { atomicAdd(&load_words[p * 8 + (b >> 2)], 1u << (8 * (b & 3))); };
  const uint32_t panel = U.panel - g.panel0;
  const PanelInfo I = info[panel];
  const uint64_t heads = (uint64_t)U.heads_lo | ((uint64_t)U.heads_hi << 32);
  const int wbits = U.wide ? 3 : 0;
  const uint32_t end = U.wide ? I.n8 : I.n8 + I.n1;
  const uint32_t sub = column_lane & ((1u << wbits) - 1);
  const bool owner = sub == 0;
  const uint16_t* list = list_all + (int64_t)panel * g.list_stride;
  const uint16_t null_index = (uint16_t)g.rows;
  for (int i = lane; i < rsr::kMaxPositions * 8; i += 64) load_words[i] = 0;
  const uint32_t step = 64u >> wbits;
  uint32_t entry = U.first + (column_lane >> wbits) + (turn ? step : 0u);
  for (int p0 = 0; p0 < npos;) {
    // the next groups: where they begin and how many rows a lane has
    int at[kGroupsAtOnce], m[kGroupsAtOnce];
    uint32_t s[kGroupsAtOnce], n[kGroupsAtOnce], slot[kGroupsAtOnce];
    const uint16_t* rows[kGroupsAtOnce];
#pragma unroll
    for (int i = 0; i < kGroupsAtOnce; ++i) {
      at[i] = 0; m[i] = -1; s[i] = 0xffffffffu;
#pragma unroll
      for (int which = 0; which < 2; ++which) {  // the next two groups, one for either lane of a column
        const uint64_t rest = p0 < npos ? heads >> p0 : 0;
        if (rest == 0) {
          for (; p0 < npos; ++p0) ent[p0][c] = null_index;  // the position that makes the count even
          continue;
        }
        const int length = __ffsll((long long)rest) - 1;
        if (which == turn) { at[i] = p0; m[i] = length; }
        p0 += length + 1;
      }
      if (m[i] >= 0 && entry < end) s[i] = list[entry];
      entry += 2 * step;
    }
    uint32_t o0[kGroupsAtOnce], o1[kGroupsAtOnce], piece[kGroupsAtOnce], bp[kGroupsAtOnce];
#pragma unroll
    for (int i = 0; i < kGroupsAtOnce; ++i) {
      o0[i] = o1[i] = piece[i] = bp[i] = 0;
      slot[i] = (uint32_t)g.s.nslots + (column_lane & (rsr::kDummySlots - 1));
      if (s[i] == 0xffffffffu) continue;
      uint32_t of = s[i];
      if (of >= (uint32_t)g.s.nslots) {
        const uint32_t x = extra_all[(int64_t)panel * g.extra_stride + (of - g.s.nslots - rsr::kDummySlots)];
        of = x & 0xffffu; piece[i] = x >> 16;
      }
      uint32_t value;
      slot_value(g, panel, of, &bp[i], &value);
      const uint32_t* o = off + (int64_t)bp[i] * ((1 << g.k) + 1) + value;
      o0[i] = o[0]; o1[i] = o[1];
      if (owner) slot[i] = s[i];
    }
#pragma unroll
    for (int i = 0; i < kGroupsAtOnce; ++i) {
      const uint32_t all = o1[i] - o0[i], np = pieces_of(all);
      const uint32_t a = all * piece[i] / np, b = all * (piece[i] + 1) / np;
      rows[i] = sigma + (int64_t)bp[i] * g.rows + o0[i] + a;
      n[i] = b - a;
    }
    int most = 0;
#pragma unroll
    for (int i = 0; i < kGroupsAtOnce; ++i) most = max(most, m[i]);
    for (int j = 0; j < most; ++j) {
      const uint32_t r = ((uint32_t)j << wbits) + sub;
      uint16_t row[kGroupsAtOnce];
#pragma unroll
      for (int i = 0; i < kGroupsAtOnce; ++i) row[i] = j < m[i] && r < n[i] ? rows[i][r] : null_index;
#pragma unroll
      for (int i = 0; i < kGroupsAtOnce; ++i)
        if (j < m[i]) {
          ent[at[i] + j][c] = row[i];
          if (row[i] != null_index) add_load(at[i] + j, row[i] & 31);
        }
    }
#pragma unroll
    for (int i = 0; i < kGroupsAtOnce; ++i)
      if (m[i] >= 0) ent[at[i] + m[i]][c] = (uint16_t)slot[i];
  }
  // The order of the rows inside a segment is free (a segment is a sum).  The LDS has 32 banks of 4 bytes and
  // serves the two halves of a wavefront one after the other; a half costs as many clocks as its fullest bank has
  // distinct addresses.  Two rows of a lane's segment trade places where that lowers the squared loads of the banks
  // (row mod 32) at their two positions most: the gathers of the product then meet in fewer banks.
  // A quarter of the columns at a time at a position: the lanes of a group stand at the same one, and would all leave a crowded bank at
  // once.  The four quarters, and the two lanes of a column, go round the unit's positions apart from each other.  (Fullest bank of a half wavefront
  // for 4096 segments of 4 rows on average, by simulation: 3.45 deep without trades, 2.44 and 2.28 after one and two rounds, 2.24 after
  // three; trades over five positions instead of three 2.27.  One quarter after the other through every group, first improvement first: 2.24.)
  // The two lanes of a column stay half a unit apart, further than a trade reaches; in units too short for that one of them does it all.
  // Bound by the instructions of one wavefront and two waits for the LDS per position: the end of a position's group comes from a table, what is
  // kReach positions on has the same address plus a constant (up to kReach rows behind a unit may be read, and are not used), and a row
  // that would trade places with one of its own bank needs no test (the loads do not change: a difference of 2).
  if (lane < npos) {
    const uint64_t rest = heads >> lane;
    ends[lane] = (uint8_t)(rest ? lane + __ffsll((long long)rest) - 1 : 0);  // the group's head
  }
  settle();
  const bool two = npos / 2 > kReach;
  const int places = two ? npos / 2 : npos;  // (npos is even)
  const int start = two ? (c & 3) * npos / 8 + turn * places : (c & 3) * npos / 4;
  uint16_t* const column = &ent[0][c];
  uint8_t* const banks = reinterpret_cast<uint8_t*>(load_words);
  for (int round = 0; round < kTradeRounds && (two || turn == 0); ++round)
    for (int t = 0; t < places; ++t) {
      settle();
      const int p = t + start < npos ? t + start : t + start - npos;
      const int others = (int)ends[p] - p - 1;  // rows of the group behind this one
      uint16_t* const at = column + p * 32;
      uint8_t* const load = banks + p * 32;
      const uint32_t row = at[0];
      uint32_t other[kReach];
#pragma unroll
      for (int i = 0; i < kReach; ++i) other[i] = at[(i + 1) * 32];
      const uint32_t b = row & 31;
      const int here = load[b];
      int best = 0, with = 0;
      int there_b[kReach], here_o[kReach], there_o[kReach];
#pragma unroll
      for (int i = 0; i < kReach; ++i) {
        const uint32_t o = other[i] & 31;
        there_b[i] = load[b + (i + 1) * 32]; here_o[i] = load[o]; there_o[i] = load[o + (i + 1) * 32];
      }
#pragma unroll
      for (int i = 0; i < kReach; ++i) {
        const int delta = (here_o[i] - here + 1) + (there_b[i] - there_o[i] + 1);
        if (i < others && other[i] != null_index && delta < best) { best = delta; with = i; }
      }
      if (best < 0 && row != null_index) {
        uint32_t o = other[0];
#pragma unroll
        for (int i = 1; i < kReach; ++i) o = with == i ? other[i] : o;
        // (rows of a byte per bank: a bank's counter is a byte of a word)
        uint32_t* const lb = load_words + p * 8 + b / 4;
        uint32_t* const lo = load_words + p * 8 + (o & 31) / 4;
        const uint32_t one_b = 1u << (8 * (b & 3)), one_o = 1u << (8 * (o & 3));
        const int q = (with + 1) * 8;
        atomicAdd(lb, 0u - one_b); atomicAdd(lo, one_o);
        atomicAdd(lo + q, 0u - one_o); atomicAdd(lb + q, one_b);
        at[0] = (uint16_t)o; at[(with + 1) * 32] = (uint16_t)row;
      }
    }
  unsigned char* to = stream + (int64_t)U.stream_off * rsr::kStreamAlign;
  settle();  // (what the other lane of the column has left)
  const int full = npos / rsr::kGranulePositions;
  for (int gq = turn; gq < full; gq += 2) {
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (uint32_t)ent[gq * 8 + 2 * j][c] | ((uint32_t)ent[gq * 8 + 2 * j + 1][c] << 16);
    reinterpret_cast<uint4*>(to)[gq * 64 + column_lane] = make_uint4(w[0], w[1], w[2], w[3]);
  }
  for (int p = full * 8 + 2 * turn; p < npos; p += 4)
    reinterpret_cast<uint32_t*>(to)[p * 32 + column_lane] = (uint32_t)ent[p][c] | ((uint32_t)ent[p + 1][c] << 16);
}

struct DevBuf {  // frees on scope exit
  void* p = nullptr;
  ~DevBuf() { if (p) (void)hipFree(p); }
  void* release() { void* q = p; p = nullptr; return q; }
};

}  // namespace

namespace rsr_internal {

int device_matrix_kind(const int8_t* dA, int64_t count, int* kind, std::string* err) {
  DevBuf flags;
  const int grid = (int)std::min<int64_t>(kKindGroups, (count + 4095) / 4096);
  PREP_TRY(hipMalloc(&flags.p, (size_t)grid * sizeof(unsigned)));
  hipLaunchKernelGGL(kind_kernel, dim3((unsigned)grid), dim3(256), 0, nullptr, dA, count, static_cast<unsigned*>(flags.p));
  PREP_TRY(hipGetLastError());
  unsigned seen[kKindGroups], f = 0;
  PREP_TRY(hipMemcpy(seen, flags.p, (size_t)grid * sizeof(unsigned), hipMemcpyDeviceToHost));
  for (int i = 0; i < grid; ++i) f |= seen[i];
  *kind = (f & 2u) ? 0 : ((f & 1u) ? 2 : 1);
  return 0;
}

int device_build_tile(const int8_t* dA, int64_t rows, int64_t cols, int64_t ld, int k, int parts, int plane0, BuiltTile* out, std::string* err) {
  const int64_t nblocks = (cols + k - 1) / k;
  const int nvals = 1 << k;
  if (rows < 1 || rows > rsr::kTileRows) { *err = "tile height out of range"; return RSR_ERR_INVALID_ARGUMENT; }
  Geometry g;
  g.rows = (int)rows; g.k = k; g.parts = parts;
  g.block0 = 0; g.panel0 = 0;
  g.s = rsr::panel_shape(rows, k, parts, plane0 < 0);
  const int64_t npanels = nblocks * g.s.panels;
  if (nblocks > 0x3fffffff || npanels > 0x7fffffff || nblocks * parts > 0x7fffffff) { *err = "too many column blocks"; return RSR_ERR_UNSUPPORTED; }
  g.extra_stride = (int)std::max<int64_t>(2, (rows * (g.s.both ? 2 : 1) / rsr::kWideRows + 1) / 2 * 2);  // (even: read two at a time)
  g.list_stride = g.s.nslots + g.extra_stride;
  // Clearing a slot costs a share of an LDS store, an absent value two bytes of the stream and a share of a gather and a store:
  // with rows spread evenly over the values, one in eight is absent where there are about two rows per value.
  g.fill = rows >= (int64_t)2 << k ? 1 : 0;
  // groups of a panel at most: one lane per segment; 8 lanes (segments of more than 6 rows, and pieces)
  const int64_t seen = rows * (g.s.both ? 2 : 1);
  g.group_stride = (int)((g.s.nslots + 63) / 64 + (std::min<int64_t>(g.s.nslots, seen / 7) + g.extra_stride + 7) / 8 + 1);
  if (g.group_stride > 1024) { *err = "too many segments in a panel"; return RSR_ERR_UNSUPPORTED; }

  // One allocation for all working memory, for `at_once` blocks: as many as a grid of 256 threads per panel holds (2^32 threads
  // in a launch) and, where that is much, as fit in a quarter of the free memory (the tables have to fit beside it).
  size_t bytes = 0;
  auto take = [&](size_t n) { const size_t at = bytes; bytes += (n + 255) / 256 * 256; return at; };
  constexpr int64_t kPanelsAtOnce = (int64_t)1 << 23;
  int64_t at_once = std::min(nblocks, std::max<int64_t>(1, kPanelsAtOnce / g.s.panels));
  DevBuf work;
  size_t most = 0;  // bytes; 0: not asked yet
  constexpr size_t kMuch = (size_t)4 << 30;
  size_t at_val, at_sigma, at_off, at_list, at_group, at_extra, at_info, at_base, at_totals;
  for (;;) {
    const size_t nbp = (size_t)at_once * parts, np = (size_t)at_once * g.s.panels;
    bytes = 0;
    at_val = take(nbp * rows * 2); at_sigma = take(nbp * rows * 2); at_off = take(nbp * (nvals + 1) * 4);
    at_list = take(np * g.list_stride * 2); at_group = take(np * g.group_stride); at_extra = take(np * g.extra_stride * 4);
    at_info = take(np * sizeof(PanelInfo)); at_base = take((size_t)npanels * sizeof(PanelBase)); at_totals = take(sizeof(Totals));
    if (bytes > kMuch && most == 0) {
      size_t total = 0;
      PREP_TRY(hipMemGetInfo(&most, &total));
      most = std::max(kMuch, most / 4);
    }
    if (bytes <= kMuch || bytes <= most || at_once == 1) break;
    at_once = (at_once + 1) / 2;
  }
  PREP_TRY(hipMalloc(&work.p, bytes));
  unsigned char* const w = static_cast<unsigned char*>(work.p);
  uint16_t* const val = reinterpret_cast<uint16_t*>(w + at_val);
  uint16_t* const sigma = reinterpret_cast<uint16_t*>(w + at_sigma);
  uint32_t* const off = reinterpret_cast<uint32_t*>(w + at_off);
  uint16_t* const list = reinterpret_cast<uint16_t*>(w + at_list);
  uint8_t* const group = w + at_group;
  uint32_t* const extra = reinterpret_cast<uint32_t*>(w + at_extra);
  PanelInfo* const info = reinterpret_cast<PanelInfo*>(w + at_info);
  PanelBase* const base = reinterpret_cast<PanelBase*>(w + at_base);  // of all panels
  Totals* const totals = reinterpret_cast<Totals*>(w + at_totals);

  // Steps 1 to 3 for the blocks b0 .. b0 + nb - 1.
  auto plan = [&](int64_t b0, int64_t nb) -> int {
    const int64_t c0 = b0 * k, nc = std::min(cols - c0, nb * k), nbp = nb * parts;
    g.block0 = (uint32_t)b0; g.panel0 = (uint32_t)(b0 * g.s.panels);
    hipLaunchKernelGGL(values_kernel, dim3((unsigned)((rows + 63) / 64), (unsigned)std::min<int64_t>((nb + kValueBlocks - 1) / kValueBlocks, 32768)),
                       dim3(256), 0, nullptr, dA + c0, (int)rows, (int)nc, ld, k, parts, plane0, (int)nb, val);
    PREP_TRY(hipGetLastError());
    const size_t per_wave = (size_t)std::max(1, nvals >> 1) * 4;
    int waves = (int)std::min<size_t>(4, (size_t)(128 * 1024) / per_wave);
    if (waves < 1) waves = 1;
    const void* kern = reinterpret_cast<const void*>(sort_kernel);
    PREP_TRY(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    hipLaunchKernelGGL(sort_kernel, dim3((unsigned)((nbp + waves - 1) / waves)), dim3((unsigned)(64 * waves)), per_wave * waves, nullptr,
                       static_cast<const uint16_t*>(val), (int)rows, k, (int)nbp, waves, off, sigma);
    PREP_TRY(hipGetLastError());
    hipLaunchKernelGGL(plan_kernel, dim3((unsigned)(nb * g.s.panels)), dim3(256), 0, nullptr, g, static_cast<const uint32_t*>(off), list, group, extra, info);
    PREP_TRY(hipGetLastError());
    return 0;
  };
  Totals sums{};
  std::vector<uint32_t> first_unit;  // of every run
  for (int64_t b0 = 0; b0 < nblocks; b0 += at_once) {
    const int64_t nb = std::min(at_once, nblocks - b0);
    const int rc = plan(b0, nb);
    if (rc != 0) return rc;
    first_unit.push_back((uint32_t)sums.units);
    hipLaunchKernelGGL(begin_kernel, dim3(1), dim3((unsigned)std::min<int64_t>(kBeginThreads, (nb * g.s.panels + 63) / 64 * 64)), 0, nullptr, g.s.panels, (uint32_t)(nb * g.s.panels), b0 == 0,
                       static_cast<const PanelInfo*>(info), base + b0 * g.s.panels, totals);
    PREP_TRY(hipGetLastError());
    PREP_TRY(hipMemcpy(&sums, totals, sizeof(Totals), hipMemcpyDeviceToHost));
    if (sums.units > 0x7fffffffull || sums.stream > 0xffffffffull) { *err = "index too large"; return RSR_ERR_UNSUPPORTED; }
  }
  const uint64_t nunits = sums.units, nstream = sums.stream;
  const uint32_t extras = sums.extras;
  first_unit.push_back((uint32_t)nunits);
  out->stored_rows = (int64_t)sums.rows; out->segments = (int64_t)sums.segments; out->head_bytes = (int64_t)sums.groups * rsr::kPositionBytes;

  // One allocation for the tables: streams, descriptors, block offsets, slots of cut segments.
  DevBuf tables;
  bytes = 0;
  out->stream_bytes = (size_t)nstream * rsr::kStreamAlign;
  out->unit_bytes = (size_t)nunits * sizeof(PUnit);
  out->blk_bytes = (size_t)(nblocks + 1) * 4;
  out->extra_bytes = extras ? (size_t)npanels * g.extra_stride * 2 : 0;
  const size_t at_stream = take(out->stream_bytes + 1024), at_units = take(out->unit_bytes + rsr::kUnitsBehind * sizeof(PUnit)), at_blk = take(out->blk_bytes + 16);
  const size_t at_slots = take(out->extra_bytes);
  PREP_TRY(hipMalloc(&tables.p, bytes));
  unsigned char* const t = static_cast<unsigned char*>(tables.p);
  PUnit* const units = reinterpret_cast<PUnit*>(t + at_units);
  uint16_t* const slots = extras ? reinterpret_cast<uint16_t*>(t + at_slots) : nullptr;
  for (int64_t b0 = 0, run = 0; b0 < nblocks; b0 += at_once, ++run) {
    const int64_t nb = std::min(at_once, nblocks - b0), p0 = b0 * g.s.panels, np = nb * g.s.panels;
    if (at_once < nblocks) {
      const int rc = plan(b0, nb);
      if (rc != 0) return rc;
    }
    const uint32_t u0 = first_unit[(size_t)run], nu = first_unit[(size_t)run + 1] - u0;
    hipLaunchKernelGGL(units_kernel, dim3((unsigned)np), dim3(64), 0, nullptr, g, (int)nblocks, (uint32_t)nunits, static_cast<const uint8_t*>(group),
                       static_cast<const PanelInfo*>(info), static_cast<const PanelBase*>(base + p0), static_cast<const uint32_t*>(extra), units,
                       reinterpret_cast<uint32_t*>(t + at_blk), slots);
    PREP_TRY(hipGetLastError());
    // (a grid holds 2^32 threads, a unit takes 128)
    constexpr uint32_t kUnitsAtOnce = 1u << 24;
    for (uint32_t u = 0; u < nu; u += kUnitsAtOnce) {
      const uint32_t n = std::min(kUnitsAtOnce, nu - u);
      hipLaunchKernelGGL(emit_kernel, dim3((2 * n + kEmitWaves - 1) / kEmitWaves), dim3(64 * kEmitWaves), 0, nullptr, g, n,
                         static_cast<const PUnit*>(units) + u0 + u, static_cast<const PanelInfo*>(info), static_cast<const uint16_t*>(list),
                         static_cast<const uint32_t*>(extra), static_cast<const uint32_t*>(off), static_cast<const uint16_t*>(sigma), t + at_stream);
      PREP_TRY(hipGetLastError());
    }
  }
  PREP_TRY(hipStreamSynchronize(nullptr));
  out->shape = g.s;
  out->extra_stride = g.extra_stride; out->max_extras = (int)extras; out->fill = g.fill != 0;
  out->nunits = (int64_t)nunits;
  out->max_units_per_block = sums.block_units;
  out->d_stream = t + at_stream;
  out->d_units = units;
  out->d_blk_unit = t + at_blk;
  out->d_extras = slots;
  out->d_tables = tables.release();
  return 0;
}

}  // namespace rsr_internal
