// C ABI (include/rsr.h) and the gfx950 kernels of the RSR++ vector x binary/ternary-matrix product.
//
// Kernel structure (one launch per product; rsr_layout.h describes the index it reads):
//   * A workgroup stages the activations of one, two or four vectors in LDS (with a zero behind them for the null row
//     index) and owns a contiguous range of column blocks, i.e. a contiguous byte range of the index streams.
//     Column blocks are independent (the paper's parallelisation I, Appendix C.1).
//   * Its wavefronts take units (whole groups of 64 segments, one segment per lane) from an LDS counter.  For a unit a
//     wavefront
//       1. reads the unit's stream with 16-byte buffer loads (the next unit's loads go out while the current one is
//          summed) and walks its positions: every lane gathers the activations of its segment's rows from LDS into
//          running sums - the segmented sums of Eq. SS2 - and at a group's end, the same position for all lanes,
//          stores them to the slot of its segment's value in the panel's part of LDS (u of Algorithm 2);
//       2. counts itself off.  The wavefront that completes a panel reads its sums back in value order and takes the
//          RSR++ fold (Section 4.3, Algorithm 3), "sum the odd-indexed entries, then add neighbours": the upper value
//          bits inside a lane, the lower six across the 64 lanes.
//   * A block whose values are one panel (both parts of a ternary matrix are subtracted slot by slot, Proposition 2.1)
//     is then stored; otherwise the panels leave records, and the wavefront that completes the block's last panel adds
//     them up: bits inside a panel sum over panels, bits above it see only panel totals.
// All float additions happen in a fixed order (no floating-point atomics), so results are
// reproducible from run to run.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "../../include/rsr.h"
#include "rsr_format.h"
#include "rsr_internal.h"
#include "rsr_layout.h"
#include "rsr_pack.h"
#include "rsr_plan.h"

namespace {

thread_local std::string g_error;

int fail(int code, const std::string& msg) {
  g_error = msg;
  return code;
}

}  // namespace

namespace rsr_internal {
// shared with the other translation units of the library (rsr_dense.hip)
int set_error(int code, const std::string& msg) { return fail(code, msg); }
}  // namespace rsr_internal

namespace {

#define RSR_HIP_TRY(expr)                                                                   \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) {                                                                 \
      (void)hipGetLastError();                                                              \
      return fail(RSR_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_));         \
    }                                                                                       \
  } while (0)

constexpr uint64_t kMagic = 0x5253522b2b763031ull;  // "RSR++v01"

}  // namespace

// One row tile of the index on the device (a matrix of up to rsr::kTileRows rows has one).
struct DeviceTile : rsr::PlanTile {
  size_t unit_bytes = 0, blk_bytes = 0, extra_bytes = 0;
  void* d_tables = nullptr;  // the allocation that holds them all
  void* d_stream = nullptr;
  void* d_units = nullptr;
  void* d_blk_unit = nullptr;
  void* d_extras = nullptr;  // slots of the pieces of segments that were cut (null if there are none)
};

struct rsr_handle : rsr::PlanMatrix {
  uint64_t magic = 0;
  int device = 0, parts = 0;
  int64_t stored_rows = 0, segments = 0, nunits = 0;
  int64_t head_bytes = 0, stream_bytes = 0, schedule_bytes = 0;
  std::vector<DeviceTile> tiles;
  // host copy of the device tables, fetched on the first rsr_export_block
  std::vector<rsr_internal::TileTables> downloaded;
};

struct rsr_host_index {
  uint64_t magic = 0;
  rsr::Index X;
};

namespace {

constexpr uint64_t kHostMagic = 0x525352686f737431ull;  // "RSRhost1"

bool valid(const rsr_host_index* x) { return x && x->magic == kHostMagic; }

void fill_info(const rsr::Index& X, rsr_info_t* info) {
  std::memset(info, 0, sizeof(*info));
  const rsr::Packed& P = X.tiles[0];
  info->rows = X.rows; info->cols = X.cols; info->k = P.k; info->parts = P.parts;
  info->nblocks = P.nblocks; info->last_block_width = P.last_width;
  info->lo_bits = P.kw; info->hi_bits = P.k - P.kw;
  for (const rsr::Packed& T : X.tiles) {
    info->stored_rows += T.stored_rows; info->segments += T.segments; info->work_units += (int64_t)T.units.size();
    info->segment_bytes += T.flag_bytes;
    info->index_bytes += (int64_t)(T.stream.size() * sizeof(uint16_t)) - T.flag_bytes;
    info->schedule_bytes += (int64_t)(T.units.size() * sizeof(rsr::Unit) + T.blk_unit.size() * sizeof(uint32_t));
  }
  info->table_bytes = info->index_bytes + info->segment_bytes + info->schedule_bytes;
  info->device = -1; info->compute_units = 0;
  info->row_tiles = (int32_t)X.tiles.size();
}

bool valid(const rsr_handle* h) { return h && h->magic == kMagic; }

// ---------------------------------------------------------------------------------------------
// device code
// ---------------------------------------------------------------------------------------------
using rsr::KArgs;
using rsr::kItems;
using rsr::LaunchPlan;
using rsr::Mode;

// The leading arguments of a kernel, fourteen words (four pointers and rsr::Start), are in scalar registers when a wavefront starts
// (-amdgpu-kernarg-preload-count, build.py); the rest it reads from the memory they were passed in.
struct KMore {
  const uint16_t* extra_slots;
  void* out;
  KArgs p;
};
#ifdef __HIP_DEVICE_COMPILE__
#define RSR_CONSTANT const __attribute__((address_space(4)))
#define RSR_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ RSR_CONSTANT char* argument_memory() { return (RSR_CONSTANT char*)__builtin_amdgcn_kernarg_segment_ptr(); }
#else
#define RSR_CONSTANT const
#define RSR_GLOBAL
__device__ inline const char* argument_memory() { return nullptr; }  // (the host pass only has to parse the kernels)
#endif
typedef RSR_CONSTANT KMore* KMorePtr;
typedef RSR_CONSTANT uint32_t* TablePtr;  // a table that is read with scalar loads
__device__ __forceinline__ KMorePtr launder(KMorePtr p) {
  asm volatile("" : "+s"(p));
  return p;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Lane swaps of a value with itself, in assembly: the compiler takes the two results of the swap
// builtins for equal when they are combined as floats.  (The s_nop covers the wait states a lane
// swap needs after a vector write of its operands.)
struct Swapped { uint32_t x, y; };
__device__ __forceinline__ Swapped swap32(uint32_t v) {  // .x: lanes 0-31 twice, .y: lanes 32-63 twice
  Swapped r{v, v};
  asm volatile("s_nop 1\n v_permlane32_swap_b32 %0, %1" : "+v"(r.x), "+v"(r.y));
  return r;
}
__device__ __forceinline__ Swapped swap16(uint32_t v) {  // .x: rows 0,0,2,2 of v, .y: rows 1,1,3,3
  Swapped r{v, v};
  asm volatile("s_nop 1\n v_permlane16_swap_b32 %0, %1" : "+v"(r.x), "+v"(r.y));
  return r;
}

// counter += 1 on behalf of the wavefront; returns the old value (wavefront-uniform).  One lane
// does it, with the execution mask set by hand: the compiler's own version of "lane 0 only" costs
// a dozen instructions.  LDS operations of a wavefront execute in order, so stores issued before
// this are in place before the counter moves.
__device__ __forceinline__ uint32_t lds_count_up(uint32_t lds_byte_addr) {
  uint32_t old;
  asm volatile(
      "v_mov_b32 v116, %[ad]\n v_mov_b32 v117, 1\n s_mov_b64 s[88:89], exec\n s_mov_b64 exec, 1\n ds_add_rtn_u32 v116, v116, v117\n"
      " s_mov_b64 exec, s[88:89]\n s_waitcnt lgkmcnt(0)\n v_readfirstlane_b32 %[o], v116\n"
      : [o] "=&s"(old)
      : [ad] "s"(__builtin_amdgcn_readfirstlane((int)lds_byte_addr))
      : "v116", "v117", "s88", "s89", "memory");
  return old;
}

// LDS words of the workgroup's bookkeeping, in assembly: through generic pointers a volatile access becomes a flat
// instruction, and the wait for one is a wait for everything the wavefront has under way in memory.
__device__ __forceinline__ uint32_t lds_load(uint32_t lds_byte_addr) {
  uint32_t x;
  asm volatile("ds_read_b32 %0, %1\n s_waitcnt lgkmcnt(0)" : "=v"(x) : "v"(lds_byte_addr) : "memory");
  return x;
}
// counter += 1 on behalf of the wavefront, without its old value
__device__ __forceinline__ void lds_bump(uint32_t lds_byte_addr) {
  uint64_t saved;
  asm volatile("s_mov_b64 %[sv], exec\n s_mov_b64 exec, 1\n ds_add_u32 %[ad], %[one]\n s_mov_b64 exec, %[sv]\n"
               : [sv] "=&s"(saved) : [ad] "v"(lds_byte_addr), [one] "v"(1u) : "memory");
}
__device__ __forceinline__ void lds_clear(uint32_t lds_byte_addr) {
  asm volatile("ds_write_b32 %0, %1" ::"v"(lds_byte_addr), "v"(0u) : "memory");
}

// ---- the positions of a unit, eight (one granule) at a time, four in the pass over four float vectors ----
// Per position and lane the stream holds a uint16: a row index, or where the unit's mask says that a group ends (the same
// position for all lanes), the lane's slot.  A row costs one address extraction, one LDS read and one add per activation
// vector; a head stores the running sums to the panel's slot (byte address s91 + slot) and restarts them.  Which positions of a
// step are heads is one of 2^8 (2^4) patterns, the same for all lanes, and every pattern has straight code of its own
// in a table that the assembler expands: the step's addresses are extracted to fixed registers and the code of its pattern is called.
// With a bit test and a branch per position in their place a wavefront issued 90 branches per unit (24 now), and gathered at the
// heads too (one position in five, an LDS read of 3 clocks each): binary 16384^2, k = 12, eight vectors 49.8 -> 44.5 us, eight int8
// vectors 37.3 -> 35.2, transformer block with sixteen vectors 90.0 -> 85.7; one vector, bound by the stream: 13.6 -> 13.7.
// Tables, in KB, and those of wide units: F1 and I1 33 + 8, F2 and P2 41 + 11, P4 57 + 17, F4 (four positions) 2 + 9; an index uses the
// patterns of its groups' lengths (some sixty).  P4 by four positions too (10 KB): of a million instruction fetches of a launch 3.4 thousand
// miss instead of 7.0 (ternary 5215 x 1990, k = 11, sixteen vectors), which is not what that launch waits for (12.7 us, 12.5 so); over 520 matrices
// with 2 to 64 vectors 0.2 to 1.5 % more time, from 8 % more (2112 x 2112, eleven vectors: 7.8 us, 8.5 so) to 2 % less.
// All gathers of a step are issued before the first sum so that their latencies overlap; the wait before the add of a
// position allows as many LDS operations as follow it (they complete in order; scalar loads that are under way besides only make
// the wait stricter).  Every gather has been waited for when its step returns.
// Fixed registers: a position's address, then its gathered activations: v96 + (position of the step) * (16-byte row: 4, 8-byte
// row: 2, else 1); the running sums from v112 on; s90 pattern, s91 panel base, s86-s89 and s92-s95 addresses.
// What an activation mode M defines: vectors V per pass, LDS bytes per row (1 << shift) and per slot, and its sums.
#define RSR_EXTRACT(sh, v, w, half) "v_lshlrev_b32_sdwa v" #v ", " #sh ", %[w" #w "] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:" half "\n"
#define RSR_EXTRACT2(sh, v0, v1, w) RSR_EXTRACT(sh, v0, w, "WORD_0") RSR_EXTRACT(sh, v1, w, "WORD_1")
// The code of every pattern of `positions` positions, `stride` bytes each, at the label `name`: rsr_p the pattern, rsr_q the position,
// rsr_n LDS operations that may be under way, rsr_z 1 where the running sums have been stored and not restarted yet.  rsr_v is the
// register of position 0; `back` holds the return address.  The assembler places the patterns itself (.org), `stride` bytes apart
// whatever their instructions take, and refuses one that is longer.
#define RSR_TABLE(name, v0, positions, stride, READ, ADD, FIRST, STORE, ZERO, back)                            \
  ".Lrsr_" name "_%=:\n.set rsr_v, " #v0 "\n.set rsr_p, 0\n.rept 1 << " #positions "\n.set rsr_q, 0\n.set rsr_n, 0\n.set rsr_z, 0\n" \
  ".rept " #positions "\n.if ((rsr_p >> rsr_q) & 1) == 0\n" READ ".set rsr_n, rsr_n+1\n.endif\n.set rsr_q, rsr_q+1\n.endr\n" \
  ".set rsr_q, 0\n.rept " #positions "\n.if (rsr_p >> rsr_q) & 1\n.if rsr_z\n" ZERO ".endif\n" STORE            \
  ".set rsr_n, rsr_n+1\n.set rsr_z, 1\n"                                                                      \
  ".else\n.set rsr_n, rsr_n-1\n s_waitcnt lgkmcnt(rsr_n)\n.if rsr_z\n" FIRST ".else\n" ADD ".endif\n.set rsr_z, 0\n" \
  ".endif\n.set rsr_q, rsr_q+1\n.endr\n"                                                                       \
  ".if rsr_z\n" ZERO ".endif\n s_setpc_b64 " back "\n"                                                        \
  ".set rsr_p, rsr_p+1\n.org .Lrsr_" name "_%=+" #stride "*rsr_p\n.endr\n"
// Behind the table, for units whose segments take 8 lanes: the lanes' sums are first added at a head with lane exchanges (the s_nop
// cover the wait states an exchange needs after a vector write), which is more code: tables of four positions, for either half of a step.
// Branches, 4 bytes per pattern, lead to the step without heads or to the calls of the two halves.  (With a test and
// a branch per position in their place the units of long segments, which a panel begins with, took half as long again as the others and
// the launch waited for them: transformer block 29.5 us, 27.1 with the tables; sixteen vectors 85.8 and 80.9; ternary 4096^2 5.92 and
// 5.35.)
#define RSR_WIDE_LANES(LANES)                                                                                  \
  " s_nop 1\n" LANES("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf") " s_nop 1\n" LANES("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf") \
  " s_nop 1\n" LANES("row_half_mirror row_mask:0xf bank_mask:0xf")
#define RSR_WIDE(v_low, v_high, stride, READ, ADD, FIRST, LANES, STORE, ZERO)         \
  " s_branch .Lrsr_table_%=\n.rept 255\n s_branch .Lrsr_halves_%=\n.endr\n"                                    \
  ".Lrsr_halves_%=:\n s_getpc_b64 s[88:89]\n.Lrsr_at_%=:\n"                                                    \
  " s_and_b32 s92, s90, 15\n s_mul_i32 s92, s92, " #stride "\n s_add_u32 s92, s92, .Lrsr_low_%=-.Lrsr_at_%=\n" \
  " s_add_u32 s92, s88, s92\n s_addc_u32 s93, s89, 0\n s_swappc_b64 s[86:87], s[92:93]\n"                      \
  " s_lshr_b32 s92, s90, 4\n s_mul_i32 s92, s92, " #stride "\n s_add_u32 s92, s92, .Lrsr_high_%=-.Lrsr_at_%=\n" \
  " s_add_u32 s92, s88, s92\n s_addc_u32 s93, s89, 0\n s_setpc_b64 s[92:93]\n"                                 \
  RSR_TABLE("low", v_low, 4, stride, READ, ADD, FIRST, RSR_WIDE_LANES(LANES) STORE, ZERO, "s[86:87]") \
  RSR_TABLE("high", v_high, 4, stride, READ, ADD, FIRST, RSR_WIDE_LANES(LANES) STORE, ZERO, "s[94:95]")
// How a unit's steps find their code: pattern 0 at `code`, every further one `stride` bytes on.
struct Steps {
  uint64_t code;
  uint32_t stride, base;  // base: LDS byte address of the panel's slots
};
// Emits a mode's table into the kernel (once per kernel: the wavefronts jump over it) and returns its address.  The compiler takes a .rept for
// a few instructions and plans short branches: they reach 128 KB, the largest kernel (P4) has 109; beyond that the assembler refuses
// the branches over the table.
#define RSR_STEPS(TABLE, WIDE)                                                                                 \
  __device__ static __forceinline__ uint64_t table() {                                                         \
    uint32_t lo, hi;                                                                                           \
    asm volatile("s_getpc_b64 s[92:93]\n.Lrsr_here_%=:\n s_add_u32 %[lo], s92, .Lrsr_table_%=-.Lrsr_here_%=\n" \
                 " s_addc_u32 %[hi], s93, 0\n s_branch .Lrsr_over_%=\n.p2align 6\n" TABLE WIDE ".Lrsr_over_%=:\n" \
                 : [lo] "=&s"(lo), [hi] "=&s"(hi)::"s92", "s93", "scc");                                       \
    return (uint64_t)hi << 32 | lo;                                                                            \
  }
#define RSR_FIND "s_mul_i32 s92, s90, %[stride]\n s_add_u32 s92, %[lo], s92\n s_addc_u32 s93, %[hi], 0\n"
#define RSR_CALL " s_swappc_b64 s[94:95], s[92:93]\n"
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }  // (into a scalar register)
#define RSR_CTL(pattern) "{s90}"(uniform(pattern)), "{s91}"(uniform(s.base)), [stride] "s"(uniform(s.stride)), [lo] "s"(uniform((uint32_t)s.code)), [hi] "s"(uniform((uint32_t)(s.code >> 32)))
#define RSR_CLOBBER                                                                                            \
  "s86", "s87", "s88", "s89", "s92", "s93", "s94", "s95", "scc", "memory", "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", \
      "v108", "v109", "v110", "v111"
// A step of eight positions from four dwords; the last one of a unit, of up to six positions, from three dwords and the null row.
// With TICKET a counter in LDS (byte address `counter`) goes up by one besides; returns its old value.  It is one LDS operation ahead of the
// gathers, whose wait is longer.
// (Registers of its own, v116 and v117: the compiler would take ones that a load of the stream may still write, as it sees it, and wait.)
#define RSR_TICKET                                                                                             \
  "v_mov_b32 v116, %[counter]\n v_mov_b32 v117, 1\n s_mov_b64 s[88:89], exec\n s_mov_b64 exec, 1\n ds_add_rtn_u32 v116, v116, v117\n" \
  " s_mov_b64 exec, s[88:89]\n"
#define RSR_TAKEN " s_waitcnt lgkmcnt(0)\n v_readfirstlane_b32 %[ticket], v116\n"
#define RSR_STEP8(shift, sums, v0, v1, v2, v3, v4, v5, v6, v7, ...)                                            \
  template <bool TICKET>                                                                                       \
  __device__ static __forceinline__ uint32_t step8(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, Sums& acc, uint32_t heads, const Steps& s, \
                                                   uint32_t counter) {                                         \
    if constexpr (TICKET) {                                                                                    \
      uint32_t ticket;                                                                                         \
      asm volatile(RSR_TICKET RSR_FIND RSR_EXTRACT2(shift, v0, v1, 0) RSR_EXTRACT2(shift, v2, v3, 1) RSR_EXTRACT2(shift, v4, v5, 2) \
                   RSR_EXTRACT2(shift, v6, v7, 3) RSR_CALL RSR_TAKEN                                           \
                   : "+{" sums "}"(acc), [ticket] "=&s"(ticket)                                                \
                   : [w0] "v"(w0), [w1] "v"(w1), [w2] "v"(w2), [w3] "v"(w3), [counter] "s"(uniform(counter)), RSR_CTL(heads & 0xffu) \
                   : RSR_CLOBBER, "v116", "v117" __VA_OPT__(,) __VA_ARGS__);                                   \
      return ticket;                                                                                           \
    } else {                                                                                                   \
      asm volatile(RSR_FIND RSR_EXTRACT2(shift, v0, v1, 0) RSR_EXTRACT2(shift, v2, v3, 1) RSR_EXTRACT2(shift, v4, v5, 2) \
                   RSR_EXTRACT2(shift, v6, v7, 3) RSR_CALL                                                     \
                   : "+{" sums "}"(acc)                                                                        \
                   : [w0] "v"(w0), [w1] "v"(w1), [w2] "v"(w2), [w3] "v"(w3), RSR_CTL(heads & 0xffu)            \
                   : RSR_CLOBBER __VA_OPT__(,) __VA_ARGS__);                                                   \
      return 0;                                                                                                \
    }                                                                                                          \
  }                                                                                                            \
  __device__ static __forceinline__ void step6(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t null_row, Sums& acc, uint32_t heads, const Steps& s) { \
    asm volatile(RSR_FIND RSR_EXTRACT2(shift, v0, v1, 0) RSR_EXTRACT2(shift, v2, v3, 1) RSR_EXTRACT2(shift, v4, v5, 2)  \
                 "v_mov_b32 v" #v6 ", %[null]\n v_mov_b32 v" #v7 ", %[null]\n" RSR_CALL                \
                 : "+{" sums "}"(acc)                                                                          \
                 : [w0] "v"(w0), [w1] "v"(w1), [w2] "v"(w2), [null] "s"(uniform(null_row)), RSR_CTL(heads & 0x3fu) \
                 : RSR_CLOBBER __VA_OPT__(,) __VA_ARGS__);                                                     \
  }

// One 32-bit word per row and slot.
#define RSR_READ1 " ds_read_b32 v[rsr_v+rsr_q], v[rsr_v+rsr_q]\n"
#define RSR_STORE1 " v_add_u32 v[rsr_v+rsr_q], s91, v[rsr_v+rsr_q]\n ds_write_b32 v[rsr_v+rsr_q], v112\n"
#define RSR_ZERO1 " v_mov_b32 v112, 0\n"
#define RSR_ADD_F1 " v_add_f32 v112, v112, v[rsr_v+rsr_q]\n"
#define RSR_FIRST_F1 " v_add_f32 v112, 0, v[rsr_v+rsr_q]\n"
#define RSR_LANES_F1(x) " v_add_f32_dpp v112, v112, v112 " x "\n"
#define RSR_ADD_I1 " v_add_u32 v112, v112, v[rsr_v+rsr_q]\n"
#define RSR_FIRST_I1 " v_mov_b32 v112, v[rsr_v+rsr_q]\n"
#define RSR_LANES_I1(x) " v_add_u32_dpp v112, v112, v112 " x "\n"
#define RSR_ADD_P2 " v_pk_add_u16 v112, v112, v[rsr_v+rsr_q]\n"
#define RSR_LANES_P2(x) " v_mov_b32_dpp v114, v112 " x "\n v_pk_add_u16 v112, v112, v114\n"
// Two words: two floats, or four 16-bit sums.
#define RSR_READ2 " ds_read_b64 v[rsr_v+2*rsr_q:rsr_v+2*rsr_q+1], v[rsr_v+2*rsr_q]\n"
#define RSR_STORE2 " v_add_u32 v[rsr_v+2*rsr_q], s91, v[rsr_v+2*rsr_q]\n ds_write_b64 v[rsr_v+2*rsr_q], v[112:113]\n"
#define RSR_ZERO2 " v_mov_b32 v112, 0\n v_mov_b32 v113, 0\n"
#define RSR_ADD_F2 " v_add_f32 v112, v112, v[rsr_v+2*rsr_q]\n v_add_f32 v113, v113, v[rsr_v+2*rsr_q+1]\n"
#define RSR_FIRST_F2 " v_add_f32 v112, 0, v[rsr_v+2*rsr_q]\n v_add_f32 v113, 0, v[rsr_v+2*rsr_q+1]\n"
#define RSR_LANES_F2(x) " v_add_f32_dpp v112, v112, v112 " x "\n v_add_f32_dpp v113, v113, v113 " x "\n"
#define RSR_ADD_P4 " v_pk_add_u16 v112, v112, v[rsr_v+2*rsr_q]\n v_pk_add_u16 v113, v113, v[rsr_v+2*rsr_q+1]\n"
#define RSR_FIRST_P4 " v_mov_b32 v112, v[rsr_v+2*rsr_q]\n v_mov_b32 v113, v[rsr_v+2*rsr_q+1]\n"
#define RSR_LANES_P4(x) " v_mov_b32_dpp v114, v112 " x "\n v_mov_b32_dpp v115, v113 " x "\n v_pk_add_u16 v112, v112, v114\n v_pk_add_u16 v113, v113, v115\n"
// Four floats.  (One ds_write_b128: 14 LDS clocks; two ds_write2_b32 would take 25.)
#define RSR_READ4 " ds_read_b128 v[rsr_v+4*rsr_q:rsr_v+4*rsr_q+3], v[rsr_v+4*rsr_q]\n"
#define RSR_STORE4 " v_add_u32 v[rsr_v+4*rsr_q], s91, v[rsr_v+4*rsr_q]\n ds_write_b128 v[rsr_v+4*rsr_q], v[112:115]\n s_nop 0\n"
#define RSR_ZERO4 " v_mov_b32 v112, 0\n v_mov_b32 v113, 0\n v_mov_b32 v114, 0\n v_mov_b32 v115, 0\n"
#define RSR_ADD_F4                                                                                             \
  " v_add_f32 v112, v112, v[rsr_v+4*rsr_q]\n v_add_f32 v113, v113, v[rsr_v+4*rsr_q+1]\n v_add_f32 v114, v114, v[rsr_v+4*rsr_q+2]\n v_add_f32 v115, v115, v[rsr_v+4*rsr_q+3]\n"
#define RSR_FIRST_F4                                                                                           \
  " v_add_f32 v112, 0, v[rsr_v+4*rsr_q]\n v_add_f32 v113, 0, v[rsr_v+4*rsr_q+1]\n v_add_f32 v114, 0, v[rsr_v+4*rsr_q+2]\n v_add_f32 v115, 0, v[rsr_v+4*rsr_q+3]\n"
#define RSR_LANES_F4(x)                                                                                        \
  " v_add_f32_dpp v112, v112, v112 " x "\n v_add_f32_dpp v113, v113, v113 " x "\n v_add_f32_dpp v114, v114, v114 " x "\n v_add_f32_dpp v115, v115, v115 " x "\n"
// int8 activations of several vectors are widened to 16 bits when they are staged, two vectors to a dword, and
// summed two at a time (v_pk_add_u16).  Nothing is lost: no lane and no slot sums more than kWideRows = 256 rows (the builder cuts
// longer segments), so a sum lies in -128 * 256 .. 127 * 256, which 16 bits hold (rsr_layout.h asserts it); from the
// slots on, and between pieces, panels and parts, sums are 32 bits wide.
// (kStride: bytes of the longest pattern; kWide: where the branches of wide units are, kWideStride bytes each.)
struct F1 {  // one float vector
  using In = float;
  using Acc = float;
  using Sums = float;  // the running sums
  static constexpr rsr::Pass pass = rsr::kF1;
  static constexpr int V = pass.V, shift = pass.shift, slot_bytes = pass.slot_bytes;
  static constexpr uint32_t kStride = 132, kWide = 256 * kStride, kWideStride = 4;
  using Slot = float;  // the sums of a slot
  __device__ static __forceinline__ float get(float x, int) { return x; }
  RSR_STEPS(RSR_TABLE("table", 96, 8, 132, RSR_READ1, RSR_ADD_F1, RSR_FIRST_F1, RSR_STORE1, RSR_ZERO1, "s[94:95]"),
            RSR_WIDE(96, 100, 212, RSR_READ1, RSR_ADD_F1, RSR_FIRST_F1, RSR_LANES_F1, RSR_STORE1, RSR_ZERO1))
  RSR_STEP8(2, "v112", 96, 97, 98, 99, 100, 101, 102, 103)
};
struct I1 {  // one int8 vector
  using In = int8_t;
  using Acc = int32_t;
  using Sums = int32_t;
  static constexpr rsr::Pass pass = rsr::kI1;
  static constexpr int V = pass.V, shift = pass.shift, slot_bytes = pass.slot_bytes;
  static constexpr uint32_t kStride = 132, kWide = 256 * kStride, kWideStride = 4;
  using Slot = int32_t;
  __device__ static __forceinline__ int32_t get(int32_t x, int) { return x; }
  RSR_STEPS(RSR_TABLE("table", 96, 8, 132, RSR_READ1, RSR_ADD_I1, RSR_FIRST_I1, RSR_STORE1, RSR_ZERO1, "s[94:95]"),
            RSR_WIDE(96, 100, 212, RSR_READ1, RSR_ADD_I1, RSR_FIRST_I1, RSR_LANES_I1, RSR_STORE1, RSR_ZERO1))
  RSR_STEP8(2, "v112", 96, 97, 98, 99, 100, 101, 102, 103)
};
struct F2 {  // two float vectors
  using In = float;
  using Acc = float;
  typedef float Sums __attribute__((ext_vector_type(2)));
  static constexpr rsr::Pass pass = rsr::kF2;
  static constexpr int V = pass.V, shift = pass.shift, slot_bytes = pass.slot_bytes;
  static constexpr uint32_t kStride = 164, kWide = 256 * kStride, kWideStride = 4;
  typedef float Slot __attribute__((ext_vector_type(2)));
  __device__ static __forceinline__ float get(Slot x, int j) { return x[j]; }
  RSR_STEPS(RSR_TABLE("table", 96, 8, 164, RSR_READ2, RSR_ADD_F2, RSR_FIRST_F2, RSR_STORE2, RSR_ZERO2, "s[94:95]"),
            RSR_WIDE(96, 104, 324, RSR_READ2, RSR_ADD_F2, RSR_FIRST_F2, RSR_LANES_F2, RSR_STORE2, RSR_ZERO2))
  RSR_STEP8(3, "v[112:113]", 96, 98, 100, 102, 104, 106, 108, 110)
};
struct P2 {  // two int8 vectors
  using In = int8_t;
  using Acc = int32_t;
  using Sums = uint32_t;
  static constexpr rsr::Pass pass = rsr::kP2;
  static constexpr int V = pass.V, shift = pass.shift, slot_bytes = pass.slot_bytes;
  static constexpr uint32_t kStride = 164, kWide = 256 * kStride, kWideStride = 4;
  typedef int16_t Slot __attribute__((ext_vector_type(2)));
  __device__ static __forceinline__ int32_t get(Slot x, int j) { return x[j]; }
  RSR_STEPS(RSR_TABLE("table", 96, 8, 164, RSR_READ1, RSR_ADD_P2, RSR_FIRST_I1, RSR_STORE1, RSR_ZERO1, "s[94:95]"),
            RSR_WIDE(96, 100, 308, RSR_READ1, RSR_ADD_P2, RSR_FIRST_I1, RSR_LANES_P2, RSR_STORE1, RSR_ZERO1))
  RSR_STEP8(2, "v112", 96, 97, 98, 99, 100, 101, 102, 103, "v114")
};
struct P4 {  // four int8 vectors
  using In = int8_t;
  using Acc = int32_t;
  typedef uint32_t Sums __attribute__((ext_vector_type(2)));
  static constexpr rsr::Pass pass = rsr::kP4;
  static constexpr int V = pass.V, shift = pass.shift, slot_bytes = pass.slot_bytes;
  static constexpr uint32_t kStride = 228, kWide = 256 * kStride, kWideStride = 4;
  typedef int16_t Slot __attribute__((ext_vector_type(4)));
  __device__ static __forceinline__ int32_t get(Slot x, int j) { return x[j]; }
  RSR_STEPS(RSR_TABLE("table", 96, 8, 228, RSR_READ2, RSR_ADD_P4, RSR_FIRST_P4, RSR_STORE2, RSR_ZERO2, "s[94:95]"),
            RSR_WIDE(96, 104, 516, RSR_READ2, RSR_ADD_P4, RSR_FIRST_P4, RSR_LANES_P4, RSR_STORE2, RSR_ZERO2))
  RSR_STEP8(3, "v[112:113]", 96, 98, 100, 102, 104, 106, 108, 110, "v114", "v115")
};
struct F4 {  // four float vectors; four positions per step (16 registers of gathered activations)
  using In = float;
  using Acc = float;
  typedef float Sums __attribute__((ext_vector_type(4)));
  static constexpr rsr::Pass pass = rsr::kF4;
  static constexpr int V = pass.V, shift = pass.shift, slot_bytes = pass.slot_bytes;
  static constexpr uint32_t kStride = 132, kWide = 16 * kStride, kWideStride = 564;
  typedef float Slot __attribute__((ext_vector_type(4)));
  __device__ static __forceinline__ float get(Slot x, int j) { return x[j]; }
  RSR_STEPS(RSR_TABLE("table", 96, 4, 132, RSR_READ4, RSR_ADD_F4, RSR_FIRST_F4, RSR_STORE4, RSR_ZERO4, "s[94:95]"),
            RSR_TABLE("wide", 96, 4, 564, RSR_READ4, RSR_ADD_F4, RSR_FIRST_F4, RSR_WIDE_LANES(RSR_LANES_F4) RSR_STORE4, RSR_ZERO4, "s[94:95]"))
  __device__ static __forceinline__ void step4(uint32_t w0, uint32_t w1, Sums& acc, uint32_t heads, const Steps& s) {
    asm volatile(RSR_FIND RSR_EXTRACT2(4, 96, 100, 0) RSR_EXTRACT2(4, 104, 108, 1) RSR_CALL
                 : "+{v[112:115]}"(acc)
                 : [w0] "v"(w0), [w1] "v"(w1), RSR_CTL(heads & 0xfu)
                 : RSR_CLOBBER);
  }
  template <bool TICKET>
  __device__ static __forceinline__ uint32_t step8(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, Sums& acc, uint32_t heads, const Steps& s,
                                                   uint32_t counter) {
    uint32_t ticket = 0;
    if constexpr (TICKET) {
      asm volatile(RSR_TICKET RSR_FIND RSR_EXTRACT2(4, 96, 100, 0) RSR_EXTRACT2(4, 104, 108, 1) RSR_CALL RSR_TAKEN
                   : "+{v[112:115]}"(acc), [ticket] "=&s"(ticket)
                   : [w0] "v"(w0), [w1] "v"(w1), [counter] "s"(uniform(counter)), RSR_CTL(heads & 0xfu)
                   : RSR_CLOBBER, "v116", "v117");
    } else {
      step4(w0, w1, acc, heads, s);
    }
    step4(w2, w3, acc, heads >> 4, s);
    return ticket;
  }
  __device__ static __forceinline__ void step6(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t null_row, Sums& acc, uint32_t heads, const Steps& s) {
    step4(w0, w1, acc, heads, s);
    asm volatile(RSR_FIND RSR_EXTRACT2(4, 96, 100, 0) "v_mov_b32 v104, %[null]\n v_mov_b32 v108, %[null]\n" RSR_CALL
                 : "+{v[112:115]}"(acc)
                 : [w0] "v"(w2), [null] "s"(uniform(null_row)), RSR_CTL((heads >> 4) & 0x3u)
                 : RSR_CLOBBER);
  }
};
// The scalar fields of a unit descriptor.  The unit number is wavefront-uniform, so the descriptor is
// read with scalar loads: these do not queue with the vector loads of the compute unit, which
// return in the order they were issued across all its wavefronts - a descriptor that has to come
// from memory would hold back everything requested after it (the other wavefronts' share of the
// activation vector at the start, stream data later).
struct Desc {
  uint32_t stream_off, block, panel, heads_lo;
  uint32_t heads_hi, npos, wide;
  uint32_t units_in_panel, extras;
};
__device__ __forceinline__ Desc make_desc(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t w4, uint32_t w5) {
  Desc d;
  d.stream_off = w0;
  d.block = w1;
  d.panel = w2;
  d.heads_lo = w3;
  d.heads_hi = w4 & 0xffffu;
  d.npos = (w4 >> 16) & 0xffu;
  d.wide = w4 >> 24;
  d.units_in_panel = w5 & 0xffffu;
  d.extras = w5 >> 16;
  return d;
}
__device__ __forceinline__ Desc load_desc(TablePtr unit_words, uint32_t u) {
  const TablePtr w = unit_words + (size_t)__builtin_amdgcn_readfirstlane((int)u) * 8;
  return make_desc(w[0], w[1], w[2], w[3], w[4], w[5]);
}

// Sums of sixteen values over the 64 lanes, all at once.  In each of four exchanges a lane keeps half of its values and gives the other half
// to its partner, so that they cost 8 + 4 + 2 + 1 additions instead of 16 each: over lane bits 5 and 4 with lane swaps of two values (what was one
// value's upper half and the other's lower half change places; the sum of the two is the exchange), over bits 3 and 2 with additions that
// write a part of the banks.  Two plain additions over bits 1 and 0 follow.  On return every lane holds the sum of v[lane >> 2].
// Bound by the instructions of one wavefront, four clocks each: 32 and six waits, and no masks.  (With an exchange inside the quads first, which takes two
// selections a pair, 65, and masks: transformer block with sixteen vectors
// 65.7 us, 64.0 so; binary 16384^2, eight int8 vectors 30.5 and 30.0.)  In assembly: the compiler takes the two results of the swap
// builtins for equal when they are combined as floats.  (The s_nop cover the wait states a swap and a lane exchange need after
// a vector write of their operands.)
#define RSR_REST_OF_SIXTEEN(ADD)                                                                               \
  "s_nop 1\n " ADD " %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n " ADD " %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n " \
  ADD " %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc\n " ADD " %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n s_nop 1\n " \
  ADD " %0, %0, %0 row_shl:4 row_mask:0xf bank_mask:0x5\n " ADD " %0, %1, %1 row_shr:4 row_mask:0xf bank_mask:0xa\n s_nop 1\n " \
  ADD " %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n s_nop 1\n " ADD " %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
template <typename AT>
__device__ __forceinline__ AT sums_of_sixteen(const AT (&v)[16]) {
  AT a[16], w[8], x[4];
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = v[i];
  asm("s_nop 1\n v_permlane32_swap_b32 %0, %8\n v_permlane32_swap_b32 %1, %9\n v_permlane32_swap_b32 %2, %10\n v_permlane32_swap_b32 %3, %11\n"
      " v_permlane32_swap_b32 %4, %12\n v_permlane32_swap_b32 %5, %13\n v_permlane32_swap_b32 %6, %14\n v_permlane32_swap_b32 %7, %15"
      : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]),
        "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15]));
#pragma unroll
  for (int i = 0; i < 8; ++i) w[i] = a[i] + a[i + 8];
  asm("s_nop 1\n v_permlane16_swap_b32 %0, %4\n v_permlane16_swap_b32 %1, %5\n v_permlane16_swap_b32 %2, %6\n v_permlane16_swap_b32 %3, %7"
      : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), "+v"(w[7]));
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = w[i] + w[i + 4];
  if constexpr (sizeof(AT) == 4 && (AT)0.5 != (AT)0)
    asm(RSR_REST_OF_SIXTEEN("v_add_f32_dpp") : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
  else
    asm(RSR_REST_OF_SIXTEEN("v_add_u32_dpp") : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
  return x[0];
}
// x where the lane's bit 2, 3, 4 or 5 is set, 0 elsewhere, for all four bits.
template <typename AT>
__device__ __forceinline__ void by_lane_bits(AT x, AT& b2, AT& b3, AT& b4, AT& b5) {
  b2 = b3 = b4 = b5 = (AT)0;
  asm("s_nop 1\n v_mov_b32_dpp %0, %4 quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0xa\n v_mov_b32_dpp %1, %4 quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0xc\n"
      " v_mov_b32_dpp %2, %4 quad_perm:[0,1,2,3] row_mask:0xa bank_mask:0xf\n v_mov_b32_dpp %3, %4 quad_perm:[0,1,2,3] row_mask:0xc bank_mask:0xf"
      : "+v"(b2), "+v"(b3), "+v"(b4), "+v"(b5) : "v"(x));
}

constexpr int NG = rsr::kMaxGranules;
constexpr int kLongStaging = 48 * 1024;  // bytes of activations (rsr_body)
constexpr int kTotal = 12;      // where a record (kItems words) holds its panel's total
constexpr int kExtraAhead = 128;  // extra sums of a panel whose slots are fetched ahead of the fold

// ---- the slots of four neighbouring values, 4 lane .. 4 lane + 3 of a step's 256, as one lane reads them ----
// 16 bytes per read: slots of 4 bytes take one ds_read_b128 (5.0 LDS clocks; four ds_read_b32 take 12), slots of 8 bytes two, of 16 bytes
// four.  A ds_read_b128 is served 16 lanes at a time - lanes 0-3, 12-15, 20-27 and lanes 4-11, 16-19, 28-31 of each half, by
// measurement - and meets in 16 classes of 16 bytes: lanes 32 or 64 bytes apart would meet two or four deep.  So lanes take their
// pieces in an order of their own: piece c ^ turn first, with turn such that the lanes of a group of 16 differ in class.
// The sums below do not depend on that order (a + b = b + a).
typedef uint32_t u32x4a __attribute__((ext_vector_type(4)));
template <class M>
struct SlotRead {
  using AT = typename M::Acc;
  static constexpr int kPieces = M::slot_bytes / 4;                    // of 16 bytes
  u32x4a piece[kPieces];
  __device__ static __forceinline__ int turn(int lane) { return kPieces == 1 ? 0 : kPieces == 2 ? (lane >> 4) & 1 : (lane >> 3) & 3; }
  __device__ __forceinline__ void read(const unsigned char* quad, int turn) {  // quad: the lane's first slot
#pragma unroll
    for (int c = 0; c < kPieces; ++c) piece[c] = *reinterpret_cast<const u32x4a*>(quad + ((c ^ turn) * 16));
  }
  __device__ static __forceinline__ void clear(unsigned char* quad) {
    uint32_t zero = 0;
    asm volatile("" : "+v"(zero));  // (a zero of this place: four registers of zeros would be kept from the start of the kernel)
#pragma unroll
    for (int c = 0; c < kPieces; ++c) *reinterpret_cast<u32x4a*>(quad + c * 16) = u32x4a{zero, zero, zero, zero};
  }
  // vector j's sum in slot i of the lane's four, in the order of the pieces: slot i ^ (turn << shift)
  __device__ __forceinline__ AT get(int i, int j) const {
    constexpr int per = 16 / M::slot_bytes, words = M::slot_bytes / 4;  // slots per piece, words per slot
    // (element by element: __builtin_bit_cast of a vector's element was compiled as one of its first element)
    struct { uint32_t w[words]; } x;
#pragma unroll
    for (int k = 0; k < words; ++k) x.w[k] = piece[i / per][(i % per) * words + k];
    return M::get(__builtin_bit_cast(typename M::Slot, x), j);
  }
  // Differences in place, where a sum fills its word.
  __device__ __forceinline__ void subtract(const SlotRead& m) {
    static_assert(sizeof(typename M::Slot) == 4 * M::V);
#pragma unroll
    for (int c = 0; c < kPieces; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t a = piece[c][k], b = m.piece[c][k];
        piece[c][k] = __builtin_bit_cast(uint32_t, (AT)(__builtin_bit_cast(AT, a) - __builtin_bit_cast(AT, b)));
      }
  }
};
// What the fold needs of four neighbouring sums: those with value bit 0, those with bit 1, all.
template <typename AT>
struct Quad {
  AT odd, high, all;
};
// d[i]: the sum of value i ^ swap, where swap = turn for slots of 16 bytes and 2 turn for slots of 8.
template <class M>
__device__ __forceinline__ Quad<typename M::Acc> quad_of(const typename M::Acc (&d)[4], int turn) {
  using AT = typename M::Acc;
  const AT lower = d[0] + d[1], upper = d[2] + d[3];
  Quad<AT> q;
  q.all = lower + upper;
  q.odd = d[1] + d[3];
  q.high = upper;
  if constexpr (M::slot_bytes == 8) q.high = turn ? lower : upper;
  if constexpr (M::slot_bytes == 16) {
    const AT even = d[0] + d[2];
    q.odd = (turn & 1) ? even : q.odd;
    q.high = (turn & 2) ? lower : upper;
  }
  return q;
}

// u . Bin_[k] by its definition, for the values 256 step + 4 lane + c, c = 0 .. 3: for every column (value bit) the sum of the
// u[j] with that bit, one addition per column and four values (which differ in bits 0 and 1 only).  Bound by vector
// instructions of the wavefront that folds; `step` is the same for all lanes.
template <typename AT>
__device__ __forceinline__ void plain_sums(AT (&sums)[12], int step, int lane, const Quad<AT>& d) {
  sums[0] += d.odd;
  sums[1] += d.high;
#pragma unroll
  for (int bit = 2; bit < 8; ++bit) sums[bit] += ((lane >> (bit - 2)) & 1) ? d.all : (AT)0;
#pragma unroll
  for (int bit = 8; bit < 12; ++bit) sums[bit] += ((step >> (bit - 8)) & 1) ? d.all : (AT)0;
}

// The activations of a workgroup's V vectors go to LDS, row by row, the vectors of a row next to each other (int8:
// widened to 32 bits, or to 16 where there are several).  Vectors past the batch are zeros.
// A piece is 16 bytes of one float vector (four rows), 16 bytes of one int8 vector, 4 bytes each of several.  A thread
// fetches kAtOnce pieces of every vector together; the caller fetches the first ones before anything else.  Pieces lie wherever the vectors
// begin: the loads take any address (floats are on four bytes, int8 vectors of an odd number of rows are not).
template <class M>
struct Staging {
  using In = typename M::In;
  static constexpr bool kFloat = sizeof(In) == 4;
  static constexpr int kAtOnce = M::V == 1 ? (kFloat ? 4 : 1) : M::V == 2 || !kFloat ? 4 : 2;
  static constexpr int kRows = !kFloat && M::V == 1 ? 16 : 4;    // rows of a piece
  static constexpr int kWords = !kFloat && M::V > 1 ? 1 : 4;
  uint32_t x[kAtOnce][M::V][kWords];

  // Pieces first + lane, first + lane + nt, ... of `n`; vectors from `nv` on are zeros.  Nothing is requested for a wavefront's turn that lies
  // behind the last piece: a load of 16 bytes per lane holds the compute unit's memory pipeline for 16 clocks wherever it reads.  For a vector that is
  // not there the first one is read again: a branch ahead of every vector's load costs full sets 2 % with two float vectors (28 products; up to 7, binary
  // 9001 x 5000, k = 12: 6.53 us and 7.03 for two) and gains sets that are not full nothing, in any pass.
  __device__ __forceinline__ void fetch(const In* __restrict__ v, int vstride, int nv, int first, int lane, int n, int nt) {
#pragma unroll
    for (int a = 0; a < kAtOnce; ++a) {
      if (first + a * nt >= n) break;
      const uint32_t at = (uint32_t)min(first + lane + a * nt, n - 1);
#pragma unroll
      for (int j = 0; j < M::V; ++j) {
        const In* from = v + (j < nv ? (int64_t)j * vstride : 0);
        uint32_t w[kWords];
        __builtin_memcpy(w, reinterpret_cast<const unsigned char*>(from) + at * (kWords * 4), sizeof(w));
#pragma unroll
        for (int c = 0; c < kWords; ++c) x[a][j][c] = w[c];
      }
    }
  }
  __device__ __forceinline__ void put(unsigned char* lds, int nv, int i, int n, int nt) {
#pragma unroll
    for (int j = 1; j < M::V; ++j)
      if (j >= nv)
#pragma unroll
        for (int a = 0; a < kAtOnce; ++a)
#pragma unroll
          for (int c = 0; c < kWords; ++c) x[a][j][c] = 0;
    // (all of them are there ahead of the first store: the compiler would move every load to its store, one wait each)
#pragma unroll
    for (int a = 0; a < kAtOnce; ++a)
#pragma unroll
      for (int j = 0; j < M::V; ++j)
#pragma unroll
        for (int c = 0; c < kWords; ++c) asm volatile("" : "+v"(x[a][j][c]));
#pragma unroll
    for (int a = 0; a < kAtOnce; ++a) {
      const int at = i + a * nt;
      if (at >= n) break;
      uint4* to = reinterpret_cast<uint4*>(lds + ((size_t)at * kRows << M::shift));
      if constexpr (kFloat && M::V == 1) {
        to[0] = make_uint4(x[a][0][0], x[a][0][1], x[a][0][2], x[a][0][3]);
      } else if constexpr (kFloat && M::V == 2) {
        to[0] = make_uint4(x[a][0][0], x[a][1][0], x[a][0][1], x[a][1][1]);
        to[1] = make_uint4(x[a][0][2], x[a][1][2], x[a][0][3], x[a][1][3]);
      } else if constexpr (kFloat) {
#pragma unroll
        for (int r = 0; r < 4; ++r) to[r] = make_uint4(x[a][0][r], x[a][1][r], x[a][2][r], x[a][3][r]);
      } else if constexpr (M::V == 1) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t d = x[a][0][c];
          to[c] = make_uint4((uint32_t)((int32_t)(d << 24) >> 24), (uint32_t)((int32_t)(d << 16) >> 24), (uint32_t)((int32_t)(d << 8) >> 24),
                             (uint32_t)((int32_t)d >> 24));
        }
      } else {
        uint32_t w[4][M::V / 2];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < M::V / 2; ++j)
            w[r][j] = ((uint32_t)((int32_t)(x[a][2 * j][0] << (24 - 8 * r)) >> 24) & 0xffffu) | ((uint32_t)((int32_t)(x[a][2 * j + 1][0] << (24 - 8 * r)) >> 24) << 16);
        if constexpr (M::V == 2) {
          to[0] = make_uint4(w[0][0], w[1][0], w[2][0], w[3][0]);
        } else {
          to[0] = make_uint4(w[0][0], w[0][1], w[1][0], w[1][1]);
          to[1] = make_uint4(w[2][0], w[2][1], w[3][0], w[3][1]);
        }
      }
    }
  }
  // the rows behind the last piece (fewer than kRows)
  __device__ static __forceinline__ void put_rest(unsigned char* lds, const In* __restrict__ v, int vstride, int nv, int first, int rows, int tid) {
    if (first + tid >= rows) return;
    const int r = first + tid;
#pragma unroll
    for (int j = 0; j < M::V; ++j) {
      const In y = j < nv ? v[(int64_t)j * vstride + r] : (In)0;
      if constexpr (kFloat) reinterpret_cast<float*>(lds)[r * M::V + j] = y;
      else if constexpr (M::V == 1) reinterpret_cast<int32_t*>(lds)[r] = y;
      else reinterpret_cast<int16_t*>(lds)[r * M::V + j] = y;
    }
  }
};

// The work of one workgroup: `wg` is its number among the workgroups of this product (a launch may
// carry several products, see rsr_multi_kernel).  The workgroup may have more wavefronts than the
// product has use for (Start::waves): the others help to stage the activations and take no units.
// PLAIN selects step 2 of Algorithm 2 as printed there (the product u . Bin_[k] term by term,
// O(k 2^k)) instead of the RSR++ fold of Algorithm 3: kept for the comparison of Appendix F.2.
template <class M, bool PLAIN>
__device__ __forceinline__ void rsr_body(const unsigned char* __restrict__ stream, const TablePtr unit_words, const TablePtr blk_unit,
                                         const typename M::In* __restrict__ vin, const rsr::Start st,
                                         const KMorePtr more, const int wg) {
  using AT = typename M::Acc;
  constexpr int V = M::V;
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool worker = wave < (int)st.waves();
  const int threads = st.threads(), rows = st.rows(), vstride = st.vstride();

  const rsr::Share mine = rsr::share_of(st, (uint32_t)wg);
  if (mine.first == mine.last) return;
  const int b = (int)mine.set * V, blk_begin = (int)mine.first, blk_end = (int)mine.last;
  const int nv = min(V, st.batch() - b);
  const uint32_t lane16 = (uint32_t)lane * 16u, lane4 = (uint32_t)lane * 4u;

  // Two register buffers: while one unit is summed from one, the next unit's stream arrives in the
  // other.  A unit's stream is read through a buffer descriptor that covers exactly the unit: a load past
  // its end (a granule or a dword row the unit does not have, or a unit that does not exist: npos = 0)
  // returns zeros without touching memory, and an address costs no vector arithmetic.  Every unit
  // issues the same number of loads, so that the wait counts between units are exact and a wait for
  // the current unit never waits for the next one.
  uint32_t eA[NG][4], eB[NG][4];
  uint32_t tA[3], tB[3];  // positions behind the last full granule: up to three rows of dwords
  auto unit_rsrc = [&](uint32_t stream_off, uint32_t npos) {
    unsigned char* us = const_cast<unsigned char*>(stream) + (size_t)stream_off * rsr::kStreamAlign;
    return __builtin_amdgcn_make_buffer_rsrc(us, 0, (int)(npos * rsr::kPositionBytes), 0x00020000);
  };
  // The stream is read once per product (per set of vectors, by siblings that share an L2): non-temporal loads keep
  // it from displacing reused data.
  constexpr int kNonTemporal = 2;
  // (the offsets go into the per-lane offset, which the range check covers; the scalar offset stays 0)
  const uint32_t lane16_hi = lane16 + 4096u;
  auto issue_granule = [&](__amdgpu_buffer_rsrc_t rs, int gq, uint32_t (&e)[NG][4]) {
    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(gq < 4 ? lane16 : lane16_hi) + (gq & 3) * 1024, 0, kNonTemporal);
    e[gq][0] = x.x; e[gq][1] = x.y; e[gq][2] = x.z; e[gq][3] = x.w;
  };
  auto issue_pair = [&](__amdgpu_buffer_rsrc_t rs, uint32_t pair_base, int j, uint32_t (&et)[3]) {
    et[j] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)pair_base + j * 256, 0, kNonTemporal);
  };

  // The start of a launch is a chain of waits for memory - block offsets, descriptor, stream, sums - that every workgroup goes through
  // at the same time, so nothing waits that need not.  The activations go first, so that their loads do not queue behind the (much larger)
  // first stream loads of the other wavefronts; what names them, and the block offsets, is in registers from the start.  The other
  // arguments are asked for together, with the block offsets.  (Stamps of ternary 4096^2, one float vector, before: 0.9 us until the
  // activations were requested, in four waits for arguments, and the staging waited behind the first stream loads.  5.25 us a product then,
  // 4.74 so; a transformer block 26.6 and 24.3.)
  const typename M::In* __restrict__ v = vin + (int64_t)b * vstride + st.row0();
  using Stage = Staging<M>;
  const int pieces = rows / Stage::kRows;
  Stage staged;
  staged.fetch(v, vstride, nv, wave * 64, lane, pieces, threads);
  uint32_t u_begin = blk_unit[blk_begin], u_end = blk_unit[blk_end];
  const KArgs p = more->p;
  const uint16_t* const extra_slots = (const uint16_t*)(const RSR_GLOBAL uint16_t*)more->extra_slots;
  asm volatile("" : "+s"(u_begin), "+s"(u_end) : "s"(p.nbuf), "s"(p.ubytes), "s"(p.off_u), "s"(p.off_done), "s"(p.off_cnt), "s"(p.off_epoch), "s"(p.off_ctr),
               "s"(p.buf_magic), "s"(p.panels), "s"(p.extra_stride), "s"(p.clear), "s"(extra_slots));
  const uint32_t n_tot = u_end - u_begin;  // units of this workgroup, numbered 0 .. n_tot-1
  // The first unit of every wavefront is fixed (its own number); its descriptor and the beginning of its stream are requested before the
  // barrier.  Later units come from a counter.  (Behind the last descriptor there is room for as many as a workgroup has wavefronts.)
  Desc D = load_desc(unit_words, u_begin + (uint32_t)wave);
  uint32_t ix = worker ? (uint32_t)wave : n_tot;
  if (p.clear)  // slots start from zero
    for (uint32_t i = (uint32_t)tid * 16u; i < (uint32_t)p.nbuf * p.ubytes; i += (uint32_t)threads * 16u)
      *reinterpret_cast<uint4*>(lds + p.off_u + i) = make_uint4(0, 0, 0, 0);
  // the counters of records and buffers, and behind them the one that hands out units
  const uint32_t counters = (p.off_ctr - p.off_done) / 4;
  if ((uint32_t)tid <= counters) reinterpret_cast<uint32_t*>(lds + p.off_done)[tid] = (uint32_t)tid == counters ? st.waves() : 0u;
  if (tid < (1 << M::shift) / 4) reinterpret_cast<uint32_t*>(lds + ((size_t)rows << M::shift))[tid] = 0;  // the null row
  if (ix >= n_tot) D.npos = 0;  // (its loads then fall outside the buffer descriptor and read nothing)
  const __amdgpu_buffer_rsrc_t rs0 = unit_rsrc(D.stream_off, D.npos);
  issue_granule(rs0, 0, eA);
  issue_granule(rs0, 1, eA);
  __builtin_amdgcn_sched_barrier(0);  // (they would be moved behind the staging)
  staged.put(lds, nv, tid, pieces, threads);
  for (int i = Stage::kAtOnce * threads; i < pieces; i += Stage::kAtOnce * threads) {
    staged.fetch(v, vstride, nv, i + wave * 64, lane, pieces, threads);
    staged.put(lds, nv, i + tid, pieces, threads);
  }
  Stage::put_rest(lds, v, vstride, nv, pieces * Stage::kRows, rows, tid);
  // The first unit's loads.  A load of 16 bytes per lane holds the compute unit's memory pipeline for 16 clocks, all of sixteen
  // wavefronts' first units for a microsecond: requested together before the barrier they hold up the activations and the
  // barrier, requested together behind it the first sums.  Two granules with the descriptor, one behind the staging where that is
  // long, the rest behind the barrier (granules before the staging + before the barrier, us: binary 16384^2 1+0 13.7, 2+0 13.2, 2+1 12.9,
  // 3+0 13.1, 6+0 13.7; transformer block 1+0 27.0, 2+0 26.1, 2+1 26.5, 3+0 26.5, 6+0 28.3).  Where the line lies, 2+1 against 2+0 at 16 row counts,
  // two matrices each: one float vector +0.6 % up to 48 KB of activations, -0.6 % from 52 to 64 KB, equal above; two and four -0.5 to -2 % from 54 KB; one
  // int8 vector -1 % throughout; two and four, whose staging widens what it reads and waits for it, +1.5 % and +2 % from 80 KB: not there.
  auto first_loads = [&](int from) {
#pragma unroll
    for (int gq = 2; gq < NG; ++gq)
      if (gq >= from) issue_granule(rs0, gq, eA);
#pragma unroll
    for (int j = 0; j < 3; ++j) issue_pair(rs0, lane4 + (D.npos >> 3) * 1024u, j, tA);
  };
  constexpr bool kThird = V == 1 || sizeof(typename M::In) == 4;
  if (kThird && rows << M::shift >= kLongStaging) {
    issue_granule(rs0, 2, eA);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    first_loads(3);
  } else {
    __syncthreads();
    first_loads(2);
  }

  const uint64_t code = M::table();
  const uint32_t panel_begin = (uint32_t)blk_begin * (uint32_t)p.panels;
  uint32_t open_panel = ~0u;  // the panel (counted from panel_begin) that is known to have room

  // ---- the fold of a panel, and the completion of its block, by the wavefront that has summed its last unit ----
  auto fold = [&](const Desc& D, uint32_t buf, uint32_t ubase, uint32_t extra_pair) {
    // (the lane's number has to look new, or the masks made of it below would be kept in scalar registers from the start of the kernel)
    int lane = tid & 63;
    asm volatile("" : "+v"(lane));
    // (The sums in LDS need no fence: LDS operations of a wavefront execute in order, so those of every unit of the panel were
    // stored before its count, and the last count has returned.  A fence would also wait for the stream of the next unit.)
    // (most arguments are fetched again: kept in scalar registers from the start of the kernel they would crowd out what
    // the units need; what the reads of the sums depend on is one word that stays)
    const KMorePtr again = launder(more);
    const KArgs f = again->p;
    RSR_GLOBAL AT* const out = (RSR_GLOBAL AT*)again->out;
    const int pslots = f.pslots; const bool both = f.both, fill = f.fill;
    unsigned char* const u = lds + ubase;
    // Lane l holds the slots 256 i + 4 l + c: value bits 0 and 1 (c) and 8 and up (i) are folded inside the lane: "sum the
    // odd-indexed entries, then add neighbours"; bits 2 to 7 are lane bits.
    const int frows = pslots / rsr::kFoldRow;
    AT hi[V][6], tot[V], pl[V][PLAIN ? 12 : 1];
#pragma unroll
    for (int j = 0; j < V; ++j) {
      tot[j] = (AT)0;
#pragma unroll
      for (int i = 0; i < 6; ++i) hi[j][i] = (AT)0;
      if constexpr (PLAIN)
#pragma unroll
        for (int i = 0; i < 12; ++i) pl[j][i] = (AT)0;
    }
    constexpr int kRowBytes = rsr::kFoldRow * M::slot_bytes;
    unsigned char* const first_quad = u + lane * 4 * M::slot_bytes;
    using Slot = typename M::Slot;
    using Read = SlotRead<M>;
    const int turn = Read::turn(lane);
    // The sums x(0) .. x(G - 1) of vector j in steps i0 .. i0 + G - 1: two steps at a time, in this order, for every G (the sums do not depend on how many
    // vectors share a pass).
    auto add_up = [&]<int G>(auto x, int j, int i0) {
      if constexpr (G == 1) {  // a panel of one step
        tot[j] += x(0);
      } else {
#pragma unroll
        for (int r = 0; r < G; r += 2) {
          const AT g = x(r) + x(r + 1);
          hi[j][2] += x(r + 1);
          if (G == 2 ? ((i0 >> 1) & 1) : ((r >> 1) & 1)) hi[j][3] += g;
          if (G <= 4 ? ((i0 >> 2) & 1) : ((r >> 2) & 1)) hi[j][4] += g;
          if ((i0 >> 3) & 1) hi[j][5] += g;
          tot[j] += g;
        }
      }
    };
    // G steps together, P of them read at a time: reads that are in flight together share the wait (behind the gathers of
    // fifteen other wavefronts the LDS answers after several hundred clocks).  The slots of the second part are read kPart
    // steps at a time (registers).
    auto fold_steps = [&]<int G>(int i0) {
      constexpr int P = M::slot_bytes == 16 ? 1 : V < 4 ? G : G < 2 ? G : 2;
      constexpr int kPart = M::slot_bytes == 4 ? (P < 4 ? P : 4) : M::slot_bytes == 8 ? P : 1;
      AT x[G][V];
      unsigned char* const rows = first_quad + i0 * kRowBytes;
#pragma unroll
      for (int r0 = 0; r0 < G; r0 += P) {
        Read q[P];
        auto add = [&](int r, int j, const AT (&d)[4]) {
          const Quad<AT> s = quad_of<M>(d, turn);
          hi[j][0] += s.odd;
          hi[j][1] += s.high;
          x[r0 + r][j] = s.all;
          if constexpr (PLAIN) plain_sums(pl[j], i0 + r0 + r, lane, s);
        };
        auto add_all = [&](const Read* m) {
#pragma unroll
          for (int r = 0; r < P; ++r)
#pragma unroll
            for (int j = 0; j < V; ++j) {
              AT d[4];
#pragma unroll
              for (int c = 0; c < 4; ++c) d[c] = m ? q[r].get(c, j) - m[r].get(c, j) : q[r].get(c, j);
              add(r, j, d);
            }
        };
#pragma unroll
        for (int r = 0; r < P; ++r) q[r].read(rows + (r0 + r) * kRowBytes, turn);
        // Proposition 2.1, v.B(1) - v.B(2): the fold is linear in u
        unsigned char* const rows1 = rows + (uint32_t)pslots * M::slot_bytes;
        if constexpr (sizeof(Slot) < 4 * V) {  // 16-bit sums, whose differences take 17
          if (both) {
            Read m[P];
#pragma unroll
            for (int r = 0; r < P; ++r) m[r].read(rows1 + (r0 + r) * kRowBytes, turn);
            if (!fill)
#pragma unroll
              for (int r = 0; r < P; ++r) Read::clear(rows1 + (r0 + r) * kRowBytes);
            add_all(m);
          } else {
            add_all(nullptr);
          }
        } else if (both) {
#pragma unroll
          for (int r1 = 0; r1 < P; r1 += kPart) {
            Read m[kPart];
#pragma unroll
            for (int r = 0; r < kPart; ++r) m[r].read(rows1 + (r0 + r1 + r) * kRowBytes, turn);
            if (!fill)
#pragma unroll
              for (int r = 0; r < kPart; ++r) Read::clear(rows1 + (r0 + r1 + r) * kRowBytes);
#pragma unroll
            for (int r = 0; r < kPart; ++r) q[r1 + r].subtract(m[r]);
            if constexpr (kPart < P) asm volatile("" ::: "memory");  // (the next reads stay behind)
          }
        }
        if (!fill)
#pragma unroll
          for (int r = 0; r < P; ++r) Read::clear(rows + (r0 + r) * kRowBytes);
        if constexpr (sizeof(Slot) == 4 * V) add_all(nullptr);
        if constexpr (P < G) asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int j = 0; j < V; ++j) add_up.template operator()<G>([&](int r) { return x[r][j]; }, j, i0);
    };
    // (Slots of 8 bytes: two steps together, and the second part's slots one step at a time, are three waits where one does.  Ternary
    // 7388 x 5593, k = 11, two float vectors: 11.05 us so, 10.24 with four steps and their second part at once; 5215 x 1990, sixteen int8
    // vectors, four per pass: 12.8 and 12.1.)
    constexpr int kTogether = PLAIN || M::slot_bytes > 8 ? 2 : V > 1 ? 4 : 8;
    // Two int8 vectors, panels of one part with several groups of four steps: a group is read while the one before is added up, in the same
    // order, so that the LDS is waited for once.  (Four waits in a panel of 4096 slots are a fifth of its fold, and panels wait for the
    // room that it takes: binary 16384^2, eight vectors, 29.9 us without, 28.9 so.  The others keep their waits, each timed both ways.  One float
    // vector, with two groups of eight steps: 41.0 us and 42.1 for eight, and slower where no panel takes this path, too.  Slots of 8 bytes,
    // whose reads spill registers: two float vectors 7 to 40 % more over 18 products, four int8 21 to 79 % over 15, 14.9 us and 17.4, 14.0 and 18.7
    // for eight at binary 9001 x 5000, k = 12.  Panels of both parts have twice the reads in flight already and were not timed.)
    constexpr bool kAhead = M::slot_bytes == 4 && V > 1;
    if (kAhead && !both && frows % 8 == 0) {
      if constexpr (kAhead) {
        Read even[4], odd[4];
        auto read = [&](Read (&q)[4], int i) {
#pragma unroll
          for (int r = 0; r < 4; ++r) q[r].read(first_quad + (i + r) * kRowBytes, turn);
        };
        auto add = [&](const Read (&q)[4], int i) {
          if (!fill)
#pragma unroll
            for (int r = 0; r < 4; ++r) Read::clear(first_quad + (i + r) * kRowBytes);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            AT x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              AT d[4];
#pragma unroll
              for (int c = 0; c < 4; ++c) d[c] = q[r].get(c, j);
              const Quad<AT> t = quad_of<M>(d, turn);
              hi[j][0] += t.odd;
              hi[j][1] += t.high;
              x[r] = t.all;
            }
            add_up.template operator()<4>([&](int r) { return x[r]; }, j, i);
          }
        };
        read(even, 0);
#pragma unroll 1
        for (int i = 0; i < frows; i += 8) {
          read(odd, i + 4);
          add(even, i);
          if (i + 8 < frows) read(even, i + 8);
          add(odd, i + 4);
        }
      }
    } else if (frows % kTogether == 0)
#pragma unroll 1
      for (int i = 0; i < frows; i += kTogether) fold_steps.template operator()<kTogether>(i);
    else if (frows == 1)
      fold_steps.template operator()<1>(0);
    else if (kTogether == 8 && frows == 4)
      fold_steps.template operator()<4>(0);
    else
#pragma unroll 1
      for (int i = 0; i < frows; i += 2) fold_steps.template operator()<2>(i);
    // The further pieces of segments that were cut: lane l takes the extra sums 2l and 2l + 1, which count under the bits of
    // their segments' values.
    const uint32_t first_extra = (uint32_t)(pslots << (both ? 1 : 0)) + rsr::kDummySlots;
    Slot ex[2] = {Slot{}, Slot{}};
    if (D.extras != 0)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (2u * (uint32_t)lane + i < D.extras) ex[i] = reinterpret_cast<const Slot*>(u)[first_extra + 2 * lane + i];
    // The panel's room is free again as soon as its sums have been read: LDS operations of a wavefront execute in
    // order, so they are read, and the slots cleared, before the epoch moves.
    auto release = [&]() {
      lds_clear(f.off_cnt + buf * 4u);
      lds_bump(f.off_epoch + buf * 4u);
    };
    const bool more = D.extras > (uint32_t)kExtraAhead;
    if (!more) release();
    AT sum[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
      AT items[kItems];
      if constexpr (PLAIN) {
#pragma unroll
        for (int i = 0; i < 12; ++i) items[i] = pl[j][i];
      } else {
#pragma unroll
        for (int i = 0; i < 6; ++i) items[i < 2 ? i : 6 + i] = hi[j][i];
        items[2] = (lane & 1) ? tot[j] : (AT)0;
        items[3] = (lane & 2) ? tot[j] : (AT)0;
        by_lane_bits(tot[j], items[4], items[5], items[6], items[7]);
      }
      items[kTotal] = tot[j];
      items[13] = items[14] = items[15] = (AT)0;
      auto add_extra = [&](uint32_t slot, AT z) {
        const AT y = both && slot >= (uint32_t)pslots ? -z : z;
#pragma unroll
        for (int i = 0; i < 12; ++i) items[i] += ((slot & (uint32_t)(pslots - 1)) >> i) & 1 ? y : (AT)0;
        items[kTotal] += y;
      };
      if (D.extras != 0) {
        uint32_t pair = extra_pair;
        asm volatile("" : "+v"(pair));  // (the masks of its bits are taken anew for every vector: scalar registers)
        add_extra(pair & 0xffffu, M::get(ex[0], j));
        add_extra(pair >> 16, M::get(ex[1], j));
        if (more)
          for (uint32_t e = (uint32_t)kExtraAhead + (uint32_t)lane; e < D.extras; e += 64)
            add_extra(extra_slots[(size_t)D.panel * f.extra_stride + e], M::get(reinterpret_cast<const Slot*>(u)[first_extra + e], j));
      }
      sum[j] = sums_of_sixteen<AT>(items);
    }
    if (more) release();
    // ---- the block: its panels' sums, the parts with their weights, k outputs ----
    const int blk = (int)D.block;
    auto put = [&](int bit, bool here, int j, AT res) {
      // value bit `bit` belongs to column k-1-bit of the block (first column most significant)
      const int width = (blk == f.nblocks - 1) ? f.last_width : f.k;
      const int col = f.k - 1 - bit;
      if (here && bit < f.k && col < width && j < nv) {
        RSR_GLOBAL AT* dst = out + (int64_t)(b + j) * f.cols + (int64_t)blk * f.k + col;
        const AT term = f.scaled ? res * __builtin_bit_cast(AT, f.scale) : res;
        *dst = f.accumulate ? *dst + term : term;  // row tiles add up: the product is linear in the rows
      }
    };
    if (f.nrec == 0) {
#pragma unroll
      for (int j = 0; j < V; ++j) put(lane >> 2, (lane & 3) == 0, j, sum[j]);
    } else {
      const uint32_t bl = (uint32_t)(blk - blk_begin);
      const uint32_t earlier = f.nrec == 1 ? bl : __umulhi(bl, f.rec_magic);  // blocks that have used these records before
      const uint32_t ring = bl - earlier * (uint32_t)f.nrec;
      while (uniform(lds_load(f.off_blocks + ring * 4u)) < earlier) __builtin_amdgcn_s_sleep(1);
      AT* rec = reinterpret_cast<AT*>(lds + f.off_rec) + (size_t)ring * f.panels * V * kItems;
      const int mine = (int)(D.panel - D.block * (uint32_t)f.panels);
      if ((lane & 3) == 0)
#pragma unroll
        for (int j = 0; j < V; ++j) rec[(mine * V + j) * kItems + (lane >> 2)] = sum[j];
      const uint32_t before = lds_count_up(f.off_done + ring * 4u);
      if ((int)before + 1 == f.panels) {  // (the other panels' records were stored before their counts)
        // The four rows of 16 lanes take every fourth panel.  Bits below kc are in the records; a higher bit sees
        // only the totals of the panels whose values have it (the remaining levels of the fold).
        const int bit = lane & 15, word = bit < f.kc ? bit : kTotal;
        const int wbits = f.k - f.kc;  // panel = part << wbits | window
        AT acc[V];
#pragma unroll
        for (int j = 0; j < V; ++j) acc[j] = (AT)0;
        for (int pi = lane >> 4; pi < f.panels; pi += 4) {
          const int part = pi >> wbits, window = pi & ((1 << wbits) - 1);
          const int w = 1 << (part * f.wshift + f.wfirst);
          const bool use = bit < f.kc || ((window >> (bit - f.kc)) & 1);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            const AT t = rec[(pi * V + j) * kItems + word] * (AT)(part == f.wneg ? -w : w);
            acc[j] += use ? t : (AT)0;
          }
        }
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const Swapped hs = swap32(__builtin_bit_cast(uint32_t, acc[j]));
          const AT two = __builtin_bit_cast(AT, hs.x) + __builtin_bit_cast(AT, hs.y);
          const Swapped qs = swap16(__builtin_bit_cast(uint32_t, two));
          put(bit, lane < 16, j, __builtin_bit_cast(AT, qs.x) + __builtin_bit_cast(AT, qs.y));
        }
        lds_clear(f.off_done + ring * 4u);
        lds_bump(f.off_blocks + ring * 4u);
      }
    }
  };

  // One unit from buffer (e, et); the next unit's stream goes into (en, etn) meanwhile.
  auto unit = [&](uint32_t (&e)[NG][4], uint32_t (&et)[3], uint32_t (&en)[NG][4], uint32_t (&etn)[3]) {
    // Panel P of the workgroup uses buffer P mod nbuf, and may start when the sums of panel P - nbuf have been read.  (Units
    // are handed out in panel order and a wavefront sums its units in order, so the oldest unit in flight never waits:
    // no deadlock.)
    const uint32_t panel = D.panel - panel_begin;
    const uint32_t turn = p.nbuf == 1 ? 0u : __umulhi(panel, p.buf_magic);
    const uint32_t buf = panel - turn * (uint32_t)p.nbuf;
    const uint32_t ubase = p.off_u + buf * p.ubytes;
    if (__builtin_expect(turn != 0 && panel != open_panel, 0)) {
      while (uniform(lds_load(p.off_epoch + buf * 4u)) < turn) __builtin_amdgcn_s_sleep(1);
      open_panel = panel;
    }

    // The slots of the panel's extra sums, two per lane, in case this unit is the panel's last: requested here, ahead of the
    // next unit's stream, they are there when the fold wants them.
    const uint16_t* const extra_list = extra_slots + (size_t)D.panel * p.extra_stride;
    const __amdgpu_buffer_rsrc_t rsx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(extra_list), 0, (int)((min(D.extras, (uint32_t)kExtraAhead) + 1u) / 2u * 4u), 0x00020000);
    const uint32_t extra_pair = __builtin_amdgcn_raw_buffer_load_b32(rsx, (int)lane4, 0, 0);
    // ---- step 1: segmented sums (Eq. SS2) into the panel's slots (u of Algorithm 2) ----
    typename M::Sums acc = {};
    const Steps steps{code + (D.wide ? M::kWide : 0u), D.wide ? M::kWideStride : M::kStride, ubase};
    const uint32_t full = D.npos >> 3;
    auto step = [&](int gq) {
      const uint32_t hm = gq < 4 ? D.heads_lo >> (8 * gq) : D.heads_hi >> (8 * (gq - 4));
      if (__builtin_expect((uint32_t)gq < full, 1)) M::template step8<false>(e[gq][0], e[gq][1], e[gq][2], e[gq][3], acc, hm, steps, 0u);
    };
    // The wavefront takes its next unit only here, behind the fold of a panel that it may have had to do and the wait for room: while it
    // folds it holds back one unit of another panel, not two (binary 16384^2, eight vectors: 44.1 us with
    // the next unit taken ahead of the fold, 41.6 so; eight int8 vectors 34.6 and 31.4; transformer block, sixteen vectors 79.2 and 73.8).
    // Several vectors per pass, whose fold is long: in the last step ahead of that unit's loads, so that the last units go to the
    // wavefronts that are furthest on.  In the first step they went to whichever had started first, units of long segments among them, which
    // end last and whose wavefronts then fold: ternary 7672 x 2776, k = 9, two vectors, 9.2 us and 8.6 so.  One vector: in the first step;
    // later, the compiler has the first sums wait for one load more (ternary 4096^2: 5.4 us and 5.6).
    constexpr int kTake = V > 1 ? NG / 2 - 1 : 0;
    uint32_t ix1;
#pragma unroll
    for (int gq = 0; gq < kTake; ++gq) step(gq);
    if (__builtin_expect(full > (uint32_t)kTake, 1)) {
      ix1 = M::template step8<true>(e[kTake][0], e[kTake][1], e[kTake][2], e[kTake][3], acc, D.heads_lo >> (8 * kTake), steps, p.off_ctr);
    } else {
      ix1 = lds_count_up(p.off_ctr);
    }
#pragma unroll
    for (int gq = kTake + 1; gq < NG / 2; ++gq) step(gq);
    // The next unit's loads go out one by one between the later steps: a wavefront that issues a whole unit at once waits
    // for room in the memory pipeline while it could be summing.
    Desc D1 = load_desc(unit_words, ix1 < n_tot ? u_begin + ix1 : 0u);  // past the end it reads unit 0 (unused)
    if (ix1 >= n_tot) D1.npos = 0;
    const __amdgpu_buffer_rsrc_t rs1 = unit_rsrc(D1.stream_off, D1.npos);
    const uint32_t pair_base1 = lane4 + (D1.npos >> 3) * 1024u;
#pragma unroll
    for (int gq = NG / 2; gq < NG; ++gq) {
      step(gq);
      issue_granule(rs1, 2 * (gq - NG / 2), en);
      issue_granule(rs1, 2 * (gq - NG / 2) + 1, en);
    }
    {
      // the positions behind the last full granule, always six: a row that the unit does not have is read as row 0
      // and added to sums that no head stores
      const uint32_t hm = (full < 4 ? D.heads_lo >> (8 * full) : D.heads_hi >> (8 * (full - 4)));
      if (__builtin_expect(D.npos & 7, 1)) M::step6(et[0], et[1], et[2], (uint32_t)rows << M::shift, acc, hm, steps);
#pragma unroll
      for (int j = 0; j < 3; ++j) issue_pair(rs1, pair_base1, j, etn);
    }
    const uint32_t before = lds_count_up(p.off_cnt + buf * 4u);
    if (before + 1 == D.units_in_panel) fold(D, buf, ubase, extra_pair);
    ix = ix1; D = D1;
  };

  while (ix < n_tot) {
    unit(eA, tA, eB, tB);
    if (ix >= n_tot) break;
    unit(eB, tB, eA, tA);
  }
}

template <class M, bool PLAIN>
__global__ void __launch_bounds__(1024)
rsr_matvec_kernel(const unsigned char* __restrict__ stream, const uint32_t* __restrict__ unit_words, const uint32_t* __restrict__ blk_unit,
                  const typename M::In* __restrict__ vin, const uint32_t sets_more, const uint32_t sets_magic, const uint32_t share, const uint32_t rows_stride,
                  const uint32_t row0_g1, const uint32_t shape, const KMore) {
  constexpr size_t at = 4 * sizeof(void*) + sizeof(rsr::Start);  // of the KMore
  static_assert(at == 56);
  rsr_body<M, PLAIN>(stream, (TablePtr)unit_words, (TablePtr)blk_unit, vin, rsr::Start{sets_more, sets_magic, share, rows_stride, row0_g1, shape},
                     (KMorePtr)(argument_memory() + at), (int)blockIdx.x);
}

// Several products in one launch (rsr_matvec_multi): every product owns a range of workgroups and
// brings its own tables, activations, results and LDS layout.  A workgroup finds its product among the first workgroups of the second
// and later ones (there are at most eight products; those that are not there begin behind the grid), which are its leading arguments.
using rsr::kMaxJobs;
struct KJob {
  const unsigned char* stream;
  const uint32_t* unit_words;
  const uint32_t* blk_unit;
  const void* vin;
  rsr::Start start;
  uint32_t wg_begin;  // first workgroup of this product
  KMore more;
};
struct MultiArgs {
  KJob job[kMaxJobs];
};
typedef RSR_CONSTANT KJob* KJobPtr;
static_assert(kMaxJobs == 8);

template <class M>
__global__ void __launch_bounds__(1024) rsr_multi_kernel(const uint32_t b1, const uint32_t b2, const uint32_t b3, const uint32_t b4, const uint32_t b5,
                                                         const uint32_t b6, const uint32_t b7, const uint32_t, const MultiArgs) {
  constexpr size_t at = 8 * sizeof(uint32_t);  // of the MultiArgs
  const uint32_t wg = blockIdx.x;
  uint32_t j = 0;  // (in assembly: the compiler adds up comparisons in vector registers)
#define RSR_BEHIND(b) "s_cmp_ge_u32 %1, " b "\n s_addc_u32 %0, %0, 0\n"
  asm(RSR_BEHIND("%2") RSR_BEHIND("%3") RSR_BEHIND("%4") RSR_BEHIND("%5") RSR_BEHIND("%6") RSR_BEHIND("%7") RSR_BEHIND("%8")
      : "+&s"(j) : "s"(wg), "s"(b1), "s"(b2), "s"(b3), "s"(b4), "s"(b5), "s"(b6), "s"(b7) : "scc");
  const KJobPtr J = (KJobPtr)(argument_memory() + at + (size_t)j * sizeof(KJob));
  // what takes fourteen registers from the start in rsr_matvec_kernel, read together
  typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
  u32x8 pointers, words;
  static_assert(offsetof(KJob, start) == 32 && offsetof(KJob, wg_begin) == 56);
  asm volatile("s_load_dwordx8 %0, %2, 0x0\n s_load_dwordx8 %1, %2, 0x20\n s_waitcnt lgkmcnt(0)" : "=&s"(pointers), "=&s"(words) : "s"(J));
  auto pointer = [&](int i) { return (uint64_t)pointers[2 * i + 1] << 32 | pointers[2 * i]; };
  rsr_body<M, false>((const unsigned char*)(const RSR_GLOBAL unsigned char*)pointer(0), (TablePtr)pointer(1), (TablePtr)pointer(2),
                     (const typename M::In*)(const RSR_GLOBAL typename M::In*)pointer(3),
                     rsr::Start{words[0], words[1], words[2], words[3], words[4], words[5]}, &J->more, (int)(wg - words[6]));
}

// ---------------------------------------------------------------------------------------------
// host code
// ---------------------------------------------------------------------------------------------
template <class M, bool PLAIN>
int enqueue(const DeviceTile& T, const LaunchPlan& plan, const typename M::In* v, void* out, void* stream) {
  const rsr::Start st = rsr::start_of(plan, plan.waves);
  hipLaunchKernelGGL((rsr_matvec_kernel<M, PLAIN>), dim3((unsigned)plan.grid), dim3((unsigned)(plan.waves * 64)), plan.lds,
                     static_cast<hipStream_t>(stream), static_cast<const unsigned char*>(T.d_stream), static_cast<const uint32_t*>(T.d_units),
                     static_cast<const uint32_t*>(T.d_blk_unit), v, st.sets_more, st.sets_magic, st.share, st.rows_stride, st.row0_g1, st.shape,
                     KMore{static_cast<const uint16_t*>(T.d_extras), out, plan.p});
  RSR_HIP_TRY(hipGetLastError());
  return RSR_OK;
}

int plan_failed(int rc, const rsr_handle* h, const DeviceTile& T) {
  if (rc == RSR_ERR_UNSUPPORTED) return fail(rc, "a row tile of " + std::to_string(T.rows) + " rows does not fit in " + std::to_string(h->lds_max) + " bytes of LDS");
  return fail(rc, "batch too large");
}

template <typename VT>
int launch_tile(rsr_handle* h, const DeviceTile& T, bool accumulate, const uint32_t* scale, const VT* v, void* out, int batch, void* stream) {
  constexpr bool i8 = sizeof(VT) == 1;
  Mode mode;
  LaunchPlan plan;
  const int rc = rsr::plan_product(i8, *h, T, accumulate, batch, &mode, &plan);
  if (rc != RSR_OK) return plan_failed(rc, h, T);
  if (scale) { plan.p.scaled = 1; plan.p.scale = *scale; }
  if constexpr (i8) {
    if (h->step2_plain) return enqueue<I1, true>(T, plan, v, out, stream);
    switch (mode) {
      case Mode::four: return enqueue<P4, false>(T, plan, v, out, stream);
      case Mode::two: return enqueue<P2, false>(T, plan, v, out, stream);
      default: return enqueue<I1, false>(T, plan, v, out, stream);
    }
  } else {
    if (h->step2_plain) return enqueue<F1, true>(T, plan, v, out, stream);
    switch (mode) {
      case Mode::four: return enqueue<F4, false>(T, plan, v, out, stream);
      case Mode::two: return enqueue<F2, false>(T, plan, v, out, stream);
      default: return enqueue<F1, false>(T, plan, v, out, stream);
    }
  }
}

// Several products as one launch: every product is planned as if it had its share of the device to itself.
template <class M>
int enqueue_multi(const rsr_job* jobs, int njobs, const LaunchPlan* plans, void* stream) {
  MultiArgs m;
  std::memset(&m, 0, sizeof(m));
  uint32_t begin[kMaxJobs];
  int64_t grid = 0;
  int waves = 1;
  size_t lds = 0;
  for (int j = 0; j < njobs; ++j) waves = std::max(waves, plans[j].waves);
  for (int j = 0; j < kMaxJobs; ++j) {
    begin[j] = 0xffffffffu;
    if (j >= njobs) continue;
    const DeviceTile& T = jobs[j].h->tiles[0];
    KJob& J = m.job[j];
    J.stream = static_cast<const unsigned char*>(T.d_stream);
    J.unit_words = static_cast<const uint32_t*>(T.d_units);
    J.blk_unit = static_cast<const uint32_t*>(T.d_blk_unit);
    J.vin = jobs[j].v;
    J.more = {static_cast<const uint16_t*>(T.d_extras), jobs[j].out, plans[j].p};
    J.start = rsr::start_of(plans[j], waves);
    begin[j] = J.wg_begin = (uint32_t)grid;
    grid += plans[j].grid;  // (a multiple of 8: every product starts on the first XCD of the round-robin)
    lds = std::max(lds, plans[j].lds);
    if (grid > 0x7fffffff) return fail(RSR_ERR_INVALID_ARGUMENT, "batch too large");
  }
  hipLaunchKernelGGL(rsr_multi_kernel<M>, dim3((unsigned)grid), dim3((unsigned)(waves * 64)), lds, static_cast<hipStream_t>(stream), begin[1], begin[2],
                     begin[3], begin[4], begin[5], begin[6], begin[7], 0u, m);
  RSR_HIP_TRY(hipGetLastError());
  return RSR_OK;
}

template <typename VT>
int launch_multi(const rsr_job* jobs, int njobs, int batch, void* stream) {
  if (!jobs || njobs < 1) return fail(RSR_ERR_INVALID_ARGUMENT, "no jobs");
  if (njobs > kMaxJobs) return fail(RSR_ERR_INVALID_ARGUMENT, "at most " + std::to_string(kMaxJobs) + " products per launch");
  if (batch < 1 || batch > 65535) return fail(RSR_ERR_INVALID_ARGUMENT, "batch must be in 1..65535");
  rsr::SharedJob each[kMaxJobs];
  for (int j = 0; j < njobs; ++j) {
    if (!valid(jobs[j].h)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid handle in job " + std::to_string(j));
    if (!jobs[j].v || !jobs[j].out) return fail(RSR_ERR_INVALID_ARGUMENT, "null pointer in job " + std::to_string(j));
    if (jobs[j].h->tiles.size() != 1) return fail(RSR_ERR_UNSUPPORTED, "a matrix with more than 32768 rows takes a launch per row tile: use rsr_matvec");
    if (jobs[j].h->device != jobs[0].h->device) return fail(RSR_ERR_INVALID_ARGUMENT, "the handles belong to different devices");
    each[j] = {jobs[j].h, &jobs[j].h->tiles[0], jobs[j].h->stream_bytes};
  }
  Mode mode;
  LaunchPlan plans[kMaxJobs];
  int failed = 0;
  const int rc = rsr::plan_shared(sizeof(VT) == 1, each, njobs, jobs[0].h->num_cu, batch, &mode, plans, &failed);
  if (rc != RSR_OK) return plan_failed(rc, jobs[failed].h, jobs[failed].h->tiles[0]);
  if constexpr (sizeof(VT) == 4) {
    if (mode == Mode::four) return enqueue_multi<F4>(jobs, njobs, plans, stream);
    if (mode == Mode::two) return enqueue_multi<F2>(jobs, njobs, plans, stream);
    return enqueue_multi<F1>(jobs, njobs, plans, stream);
  } else {
    if (mode == Mode::four) return enqueue_multi<P4>(jobs, njobs, plans, stream);
    if (mode == Mode::two) return enqueue_multi<P2>(jobs, njobs, plans, stream);
    return enqueue_multi<I1>(jobs, njobs, plans, stream);
  }
}

// One launch per row tile, in order, on the caller's stream: the first overwrites `out`, the others add.
template <typename VT>
// With `scale` (rsr_matvec_acc) every launch adds scale * (its tile's product) to `out`.
int launch(rsr_handle* h, const VT* v, void* out, int batch, void* stream, const uint32_t* scale = nullptr) {
  if (!valid(h)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid handle");
  if (!v || !out) return fail(RSR_ERR_INVALID_ARGUMENT, "null pointer");
  if (batch < 1) return fail(RSR_ERR_INVALID_ARGUMENT, "batch must be >= 1");
  if (batch > 65535) return fail(RSR_ERR_INVALID_ARGUMENT, "batch must be <= 65535");
  for (size_t t = 0; t < h->tiles.size(); ++t) {
    const int rc = launch_tile(h, h->tiles[t], t > 0 || scale != nullptr, scale, v, out, batch, stream);
    if (rc != RSR_OK) return rc;
  }
  return RSR_OK;
}

void free_tables(rsr_handle* h) {
  for (DeviceTile& T : h->tiles) {
    if (T.d_tables) (void)hipFree(T.d_tables);
    T = DeviceTile();
  }
}

// A handle for the matrix at A (DEVICE).  plane0 < 0: parts = 1 or 2; otherwise the bit planes plane0 .. plane0 + parts - 1
// of entries with q bits.
rsr_handle* make_handle(const int8_t* A, int64_t rows, int64_t cols, int k, int parts, int plane0, int q, const char* who) {
  std::unique_ptr<rsr_handle> h(new (std::nothrow) rsr_handle());
  if (!h) { fail(RSR_ERR_OUT_OF_MEMORY, "out of host memory"); return nullptr; }
  hipError_t e = hipGetDevice(&h->device);
  int cu = 0, lds = 0;
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, h->device);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, h->device);
  if (e != hipSuccess) { (void)hipGetLastError(); fail(RSR_ERR_HIP, std::string(who) + ": " + hipGetErrorString(e)); return nullptr; }
  h->num_cu = cu;
  h->lds_max = (size_t)lds;
  h->rows = rows; h->cols = cols; h->k = k; h->parts = parts;
  h->qbit = plane0 >= 0;
  h->first_plane = plane0 > 0 ? plane0 : 0;
  h->negative_part = plane0 < 0 ? (parts == 2 ? 1 : -1) : (plane0 + parts == q ? parts - 1 : -1);
  h->nblocks = (cols + k - 1) / k;
  h->last_width = (int)(cols - (h->nblocks - 1) * k);
  // the kernels may use the whole LDS of a compute unit as dynamic shared memory
  for (const void* kern : {reinterpret_cast<const void*>(rsr_matvec_kernel<F1, false>), reinterpret_cast<const void*>(rsr_matvec_kernel<F2, false>),
                           reinterpret_cast<const void*>(rsr_matvec_kernel<F4, false>), reinterpret_cast<const void*>(rsr_matvec_kernel<I1, false>),
                           reinterpret_cast<const void*>(rsr_matvec_kernel<P2, false>), reinterpret_cast<const void*>(rsr_matvec_kernel<P4, false>), reinterpret_cast<const void*>(rsr_matvec_kernel<F1, true>),
                           reinterpret_cast<const void*>(rsr_matvec_kernel<I1, true>), reinterpret_cast<const void*>(rsr_multi_kernel<F1>),
                           reinterpret_cast<const void*>(rsr_multi_kernel<F2>), reinterpret_cast<const void*>(rsr_multi_kernel<F4>),
                           reinterpret_cast<const void*>(rsr_multi_kernel<I1>), reinterpret_cast<const void*>(rsr_multi_kernel<P2>),
                           reinterpret_cast<const void*>(rsr_multi_kernel<P4>)}) {
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) { (void)hipGetLastError(); fail(RSR_ERR_HIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e)); return nullptr; }
  }
  const int64_t ntiles = (rows + rsr::kTileRows - 1) / rsr::kTileRows;
  // equal heights, multiples of 16 rows (a tile's share of an activation vector stays 16-byte aligned)
  const int64_t height = ((rows + ntiles - 1) / ntiles + 15) / 16 * 16;
  std::string err;
  for (int64_t t = 0; t < ntiles; ++t) {
    const int64_t r0 = t * height, r1 = std::min(rows, r0 + height);
    rsr_internal::BuiltTile B;
    int rc;
    try {
      h->tiles.reserve((size_t)ntiles);
      rc = rsr_internal::device_build_tile(A + r0 * cols, r1 - r0, cols, cols, k, parts, plane0, &B, &err);
    } catch (const std::bad_alloc&) {
      rc = RSR_ERR_OUT_OF_MEMORY; err = "out of host memory";
    }
    if (rc != 0) { free_tables(h.get()); fail(rc, std::string(who) + ": " + err); return nullptr; }
    DeviceTile T;
    T.rows = r1 - r0; T.row0 = r0;
    T.shape = B.shape; T.extra_stride = B.extra_stride; T.max_extras = B.max_extras; T.fill = B.fill;
    T.max_units_per_block = B.max_units_per_block; T.nunits = B.nunits;
    T.stream_bytes = B.stream_bytes; T.unit_bytes = B.unit_bytes; T.blk_bytes = B.blk_bytes; T.extra_bytes = B.extra_bytes;
    T.d_tables = B.d_tables;
    T.d_stream = B.d_stream; T.d_units = B.d_units; T.d_blk_unit = B.d_blk_unit; T.d_extras = B.d_extras;
    h->tiles.push_back(T);
    h->stored_rows += B.stored_rows; h->segments += B.segments; h->nunits += B.nunits;
    h->head_bytes += B.head_bytes; h->stream_bytes += (int64_t)B.stream_bytes;
    h->schedule_bytes += (int64_t)(B.unit_bytes + B.blk_bytes + B.extra_bytes);
  }
  h->magic = kMagic;
  return h.release();
}

bool valid_shape(const void* A, int64_t rows, int64_t cols, int k, const char* who) {
  const std::string at = std::string(who) + ": ";
  if (!A) { fail(RSR_ERR_INVALID_ARGUMENT, at + "null pointer"); return false; }
  if (rows < 1 || rows > rsr::kMaxRows) { fail(RSR_ERR_INVALID_ARGUMENT, at + "rows must be in 1..65534"); return false; }
  if (cols < 1) { fail(RSR_ERR_INVALID_ARGUMENT, at + "cols must be >= 1"); return false; }
  if (k < 1 || k > rsr::kMaxK) { fail(RSR_ERR_INVALID_ARGUMENT, at + "k must be in 1..16"); return false; }
  return true;
}

// A host matrix in device memory for the time of a build.
struct DeviceCopy {
  int8_t* p = nullptr;
  ~DeviceCopy() { if (p) (void)hipFree(p); }
  bool fill(const int8_t* A, int64_t count, const char* who) {
    hipError_t e = hipMalloc(&p, (size_t)count);
    if (e == hipSuccess) e = hipMemcpy(p, A, (size_t)count, hipMemcpyHostToDevice);
    if (e != hipSuccess) { (void)hipGetLastError(); fail(RSR_ERR_HIP, std::string(who) + ": " + hipGetErrorString(e)); }
    return e == hipSuccess;
  }
};

}  // namespace

namespace rsr_internal {

int8_t* device_copy(const int8_t* A, int64_t count, const char* who) {
  DeviceCopy d;
  if (!d.fill(A, count, who)) return nullptr;
  int8_t* p = d.p;
  d.p = nullptr;
  return p;
}
void device_release(int8_t* p) { (void)hipFree(p); }

rsr_handle* build_planes(const int8_t* dA, int64_t rows, int64_t cols, int k, int plane0, int planes, int q) {
  return make_handle(dA, rows, cols, k, planes, plane0, q, "rsr_qbit_preprocess");
}

}  // namespace rsr_internal

extern "C" {

rsr_handle* rsr_preprocess(const int8_t* A, int64_t rows, int64_t cols, int k) {
  g_error.clear();
  if (!valid_shape(A, rows, cols, k, "rsr_preprocess")) return nullptr;
  DeviceCopy d;
  if (!d.fill(A, rows * cols, "rsr_preprocess")) return nullptr;
  std::string err;
  int kind = 0;
  const int rc = rsr_internal::device_matrix_kind(d.p, rows * cols, &kind, &err);
  if (rc != 0) { fail(rc, "rsr_preprocess: " + err); return nullptr; }
  if (kind == 0) {
    int64_t i = 0;
    while (i + 1 < rows * cols && A[i] >= -1 && A[i] <= 1) ++i;
    fail(RSR_ERR_INVALID_ARGUMENT, "rsr_preprocess: entry outside {-1,0,1} at row " + std::to_string(i / cols) + ", column " + std::to_string(i % cols));
    return nullptr;
  }
  return make_handle(d.p, rows, cols, k, kind, -1, 0, "rsr_preprocess");
}

rsr_handle* rsr_preprocess_device(const int8_t* A, int64_t rows, int64_t cols, int k) {
  g_error.clear();
  if (!valid_shape(A, rows, cols, k, "rsr_preprocess_device")) return nullptr;
  std::string err;
  int kind = 0;
  const int rc = rsr_internal::device_matrix_kind(A, rows * cols, &kind, &err);
  if (rc != 0) { fail(rc, "rsr_preprocess_device: " + err); return nullptr; }
  if (kind == 0) { fail(RSR_ERR_INVALID_ARGUMENT, "rsr_preprocess_device: an entry lies outside {-1,0,1}"); return nullptr; }
  return make_handle(A, rows, cols, k, kind, -1, 0, "rsr_preprocess_device");
}

int rsr_matvec(rsr_handle* h, const float* v, float* out, int batch, void* stream) {
  return launch<float>(h, v, out, batch, stream);
}

int rsr_matvec_i8(rsr_handle* h, const int8_t* v, int32_t* out, int batch, void* stream) {
  return launch<int8_t>(h, v, out, batch, stream);
}

int rsr_matvec_acc(rsr_handle* h, const float* v, float* out, float scale, int batch, void* stream) {
  if (!(scale == scale) || scale - scale != 0.0f) return fail(RSR_ERR_INVALID_ARGUMENT, "rsr_matvec_acc: scale must be finite");
  const uint32_t bits = __builtin_bit_cast(uint32_t, scale);
  return launch<float>(h, v, out, batch, stream, &bits);
}

int rsr_matvec_acc_i8(rsr_handle* h, const int8_t* v, int32_t* out, int32_t scale, int batch, void* stream) {
  const uint32_t bits = (uint32_t)scale;
  return launch<int8_t>(h, v, out, batch, stream, &bits);
}

int rsr_matvec_multi(const rsr_job* jobs, int njobs, int batch, void* stream) {
  return launch_multi<float>(jobs, njobs, batch, stream);
}

int rsr_matvec_multi_i8(const rsr_job* jobs, int njobs, int batch, void* stream) {
  return launch_multi<int8_t>(jobs, njobs, batch, stream);
}

int rsr_set_step2(rsr_handle* h, int step2) {
  if (!valid(h)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid handle");
  if (step2 != RSR_STEP2_FOLD && step2 != RSR_STEP2_PLAIN) return fail(RSR_ERR_INVALID_ARGUMENT, "unknown step 2 variant");
  h->step2_plain = (step2 == RSR_STEP2_PLAIN);
  return RSR_OK;
}

int rsr_model_k(int64_t rows, int k_min, int k_max) {
  if (rows < 1 || k_min < 1 || k_max > rsr::kMaxK || k_min > k_max) return fail(RSR_ERR_INVALID_ARGUMENT, "rsr_model_k: bad range");
  int best = k_min;
  double best_cost = 0;
  for (int k = k_min; k <= k_max; ++k) {
    const double cost = ((double)rows + (double)(1u << k)) / (double)k;  // per column: (n + 2^k) / k
    if (k == k_min || cost < best_cost) { best = k; best_cost = cost; }
  }
  return best;
}

int rsr_autotune_k(const int8_t* A, int64_t rows, int64_t cols, int batch, int k_min, int k_max, int reps, int cold,
                   int* best_k, double* us_per_k) {
  g_error.clear();
  if (!A || !best_k) return fail(RSR_ERR_INVALID_ARGUMENT, "null pointer");
  if (k_min < 1 || k_max > rsr::kMaxK || k_min > k_max) return fail(RSR_ERR_INVALID_ARGUMENT, "k range must lie in 1..16");
  if (batch < 1 || batch > 65535 || reps < 1) return fail(RSR_ERR_INVALID_ARGUMENT, "batch and reps must be >= 1");
  float* v = nullptr;
  float* out = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  std::vector<rsr_handle*> hs;
  auto cleanup = [&]() {
    (void)hipDeviceSynchronize();
    for (rsr_handle* h : hs) rsr_destroy(h);
    hs.clear();
  };
  auto release = [&]() {
    cleanup();
    if (v) (void)hipFree(v);
    if (out) (void)hipFree(out);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
  };
  auto bail = [&](int code, const std::string& msg) { release(); return fail(code, msg); };
  if (hipMalloc(&v, (size_t)batch * rows * sizeof(float)) != hipSuccess || hipMalloc(&out, (size_t)batch * cols * sizeof(float)) != hipSuccess)
    return bail(RSR_ERR_HIP, "rsr_autotune_k: device allocation failed");
  if (hipMemset(v, 0, (size_t)batch * rows * sizeof(float)) != hipSuccess) return bail(RSR_ERR_HIP, "rsr_autotune_k: hipMemset failed");
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return bail(RSR_ERR_HIP, "rsr_autotune_k: hipEventCreate failed");
  double best_us = 0;
  for (int k = k_min; k <= k_max; ++k) {
    rsr_handle* h = rsr_preprocess(A, rows, cols, k);
    if (!h) { const std::string msg = g_error; return bail(RSR_ERR_INVALID_ARGUMENT, msg); }
    hs.push_back(h);
    if (cold) {  // enough copies that the tables of consecutive calls do not come from the last-level cache
      rsr_info_t info;
      rsr_info(h, &info);
      const int64_t want = ((int64_t)512 << 20) / std::max<int64_t>(1, info.table_bytes) + 1;
      const int copies = (int)std::min<int64_t>(16, std::max<int64_t>(1, want));
      for (int c = 1; c < copies; ++c) {
        rsr_handle* hc = rsr_preprocess(A, rows, cols, k);
        if (!hc) { const std::string msg = g_error; return bail(RSR_ERR_HIP, msg); }
        hs.push_back(hc);
      }
    }
    const int n = (int)hs.size();
    int rc = RSR_OK;
    for (int i = 0; i < std::max(3, n) && rc == RSR_OK; ++i) rc = rsr_matvec(hs[(size_t)(i % n)], v, out, batch, nullptr);
    if (rc == RSR_OK && hipEventRecord(e0, nullptr) != hipSuccess) rc = RSR_ERR_HIP;
    for (int i = 0; i < reps && rc == RSR_OK; ++i) rc = rsr_matvec(hs[(size_t)(i % n)], v, out, batch, nullptr);
    if (rc == RSR_OK && (hipEventRecord(e1, nullptr) != hipSuccess || hipEventSynchronize(e1) != hipSuccess)) rc = RSR_ERR_HIP;
    float ms = 0;
    if (rc == RSR_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = RSR_ERR_HIP;
    if (rc != RSR_OK) { const std::string msg = g_error.empty() ? "rsr_autotune_k: timing failed" : g_error; return bail(rc, msg); }
    const double us = (double)ms * 1e3 / reps;
    if (us_per_k) us_per_k[k - k_min] = us;
    if (k == k_min || us < best_us) { best_us = us; *best_k = k; }
    cleanup();
  }
  release();
  return RSR_OK;
}

void rsr_destroy(rsr_handle* h) {
  if (!valid(h)) return;
  free_tables(h);
  h->magic = 0;
  delete h;
}

const char* rsr_last_error(void) { return g_error.c_str(); }

int rsr_info(const rsr_handle* h, rsr_info_t* info) {
  if (!valid(h) || !info) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid handle or null info");
  std::memset(info, 0, sizeof(*info));
  info->rows = h->rows; info->cols = h->cols; info->k = h->k; info->parts = h->parts;
  info->nblocks = h->nblocks; info->last_block_width = h->last_width;
  info->lo_bits = h->tiles[0].shape.kc; info->hi_bits = h->k - info->lo_bits;
  info->stored_rows = h->stored_rows; info->segments = h->segments; info->work_units = h->nunits;
  info->segment_bytes = h->head_bytes;
  info->index_bytes = h->stream_bytes - h->head_bytes;
  info->schedule_bytes = h->schedule_bytes;
  info->table_bytes = info->index_bytes + info->segment_bytes + info->schedule_bytes;
  info->device = h->device; info->compute_units = h->num_cu;
  info->row_tiles = (int32_t)h->tiles.size();
  return RSR_OK;
}

int rsr_export_block(rsr_handle* h, int part, int64_t block, int32_t* sigma, int32_t* L) {
  if (!valid(h)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid handle");
  if (h->downloaded.empty()) {
    int dev = 0;
    RSR_HIP_TRY(hipGetDevice(&dev));
    RSR_HIP_TRY(hipSetDevice(h->device));
    try {
      std::vector<rsr_internal::TileTables> X(h->tiles.size());
      for (size_t t = 0; t < X.size(); ++t) {
        const DeviceTile& T = h->tiles[t];
        rsr_internal::TileTables& P = X[t];
        P.rows = T.rows; P.row0 = T.row0; P.shape = T.shape; P.extra_stride = T.extra_stride;
        P.stream.resize(T.stream_bytes / sizeof(uint16_t));
        P.units.resize(T.unit_bytes / sizeof(rsr::PUnit));
        P.blk_unit.resize(T.blk_bytes / sizeof(uint32_t));
        P.extras.resize(T.extra_bytes / sizeof(uint16_t));
        if (T.stream_bytes) RSR_HIP_TRY(hipMemcpy(P.stream.data(), T.d_stream, T.stream_bytes, hipMemcpyDeviceToHost));
        if (T.unit_bytes) RSR_HIP_TRY(hipMemcpy(P.units.data(), T.d_units, T.unit_bytes, hipMemcpyDeviceToHost));
        if (T.extra_bytes) RSR_HIP_TRY(hipMemcpy(P.extras.data(), T.d_extras, T.extra_bytes, hipMemcpyDeviceToHost));
        RSR_HIP_TRY(hipMemcpy(P.blk_unit.data(), T.d_blk_unit, T.blk_bytes, hipMemcpyDeviceToHost));
      }
      h->downloaded = std::move(X);
    } catch (const std::bad_alloc&) {
      (void)hipSetDevice(dev);
      return fail(RSR_ERR_OUT_OF_MEMORY, "out of host memory");
    }
    RSR_HIP_TRY(hipSetDevice(dev));
  }
  std::string err;
  int rc;
  try {
    rc = rsr_internal::decode_tables(h->downloaded, h->rows, h->cols, h->k, h->parts, part, block, sigma, L, &err);
  } catch (const std::bad_alloc&) {
    return fail(RSR_ERR_OUT_OF_MEMORY, "out of host memory");
  }
  if (rc != 0) return fail(rc, "rsr_export_block: " + err);
  return RSR_OK;
}

rsr_host_index* rsr_host_pack(const int8_t* A, int64_t rows, int64_t cols, int k) {
  g_error.clear();
  std::unique_ptr<rsr_host_index> x(new (std::nothrow) rsr_host_index());
  if (!x) { fail(RSR_ERR_OUT_OF_MEMORY, "out of host memory"); return nullptr; }
  std::string err;
  int rc;
  try {
    rc = rsr::pack_tiles(A, rows, cols, k, 0, &x->X, &err);
  } catch (const std::bad_alloc&) {
    fail(RSR_ERR_OUT_OF_MEMORY, "out of host memory while packing");
    return nullptr;
  }
  if (rc != 0) { fail(rc, "rsr_host_pack: " + err); return nullptr; }
  x->magic = kHostMagic;
  return x.release();
}

void rsr_host_free(rsr_host_index* x) {
  if (!valid(x)) return;
  x->magic = 0;
  delete x;
}

int rsr_host_info(const rsr_host_index* x, rsr_info_t* info) {
  if (!valid(x) || !info) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid host index or null info");
  fill_info(x->X, info);
  return RSR_OK;
}

int rsr_host_export_block(const rsr_host_index* x, int part, int64_t block, int32_t* sigma, int32_t* L) {
  if (!valid(x)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid host index");
  std::string err;
  const int rc = rsr::decode_block(x->X, part, block, sigma, L, &err);
  if (rc != 0) return fail(rc, "rsr_host_export_block: " + err);
  return RSR_OK;
}

int rsr_host_streams(const rsr_host_index* x, int tile, const uint16_t** stream, int64_t* n_stream, const void** units,
                     int64_t* n_units, const uint32_t** blk_unit, int64_t* tile_row0, int64_t* tile_rows) {
  if (!valid(x)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid host index");
  if (tile < 0 || tile >= (int)x->X.tiles.size()) return fail(RSR_ERR_INVALID_ARGUMENT, "row tile out of range");
  const rsr::Packed& P = x->X.tiles[(size_t)tile];
  if (stream) *stream = P.stream.data();
  if (n_stream) *n_stream = (int64_t)P.stream.size();
  if (units) *units = P.units.data();
  if (n_units) *n_units = (int64_t)P.units.size();
  if (blk_unit) *blk_unit = P.blk_unit.data();
  if (tile_row0) *tile_row0 = x->X.row0[(size_t)tile];
  if (tile_rows) *tile_rows = P.rows;
  return RSR_OK;
}

}  // extern "C"
