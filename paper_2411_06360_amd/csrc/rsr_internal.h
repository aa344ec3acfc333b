// Shared between the translation units of the library (not part of the C ABI).
#ifndef RSR_INTERNAL_H_
#define RSR_INTERNAL_H_

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/rsr.h"
#include "rsr_layout.h"

namespace rsr_internal {

// the calling thread's message for rsr_last_error(); returns `code`
int set_error(int code, const std::string& msg);

// The tables of one row tile, built in device memory by device_build_tile (rsr_prep.hip): one allocation, owned
// by the caller afterwards (hipFree(d_tables)), with the four tables inside.
struct BuiltTile {
  void* d_tables = nullptr;
  void* d_stream = nullptr;
  void* d_units = nullptr;
  void* d_blk_unit = nullptr;
  void* d_extras = nullptr;  // null if no segment is cut
  size_t stream_bytes = 0, unit_bytes = 0, blk_bytes = 0, extra_bytes = 0;
  rsr::Shape shape{};
  int extra_stride = 0;  // entries per panel in d_extras
  int max_extras = 0;    // extra slots of a panel at most
  bool fill = false;     // absent values are stored as zeros (slots need no clearing)
  uint32_t max_units_per_block = 0;
  int64_t nunits = 0, stored_rows = 0, segments = 0, head_bytes = 0;
};

// Algorithm 1 on the device for the rows x cols tile at dA (DEVICE, row-major, `ld` elements between rows):
// row values, counting sort per column block and part, full segmentation, packing into the layout of
// rsr_layout.h.  plane0 < 0: parts = 1 or 2, B(1) and B(2) (decided by the caller for the whole matrix);
// otherwise the parts are the bit planes plane0 .. plane0 + parts - 1 of the entries.  Returns 0 or a negative status.
int device_build_tile(const int8_t* dA, int64_t rows, int64_t cols, int64_t ld, int k, int parts, int plane0, BuiltTile* out, std::string* err);

// Checks the entries of a device matrix: *kind = 0 if an entry lies outside {-1,0,1}, 2 if some entry is -1, else 1.
int device_matrix_kind(const int8_t* dA, int64_t count, int* kind, std::string* err);

// The product of the bit planes plane0 .. plane0 + planes - 1 of the q-bit matrix dA (DEVICE), weighted and added up:
// a handle of rsr.h (rsr_plan.h says how many planes one can hold).
rsr_handle* build_planes(const int8_t* dA, int64_t rows, int64_t cols, int k, int plane0, int planes, int q);

// A host matrix in device memory, for code that is not compiled for the device (null: failed, the message is set).
int8_t* device_copy(const int8_t* A, int64_t count, const char* who);
void device_release(int8_t* p);

// sigma and L of one block from the tables of a tile, copied to the host.
struct TileTables {
  int64_t rows = 0, row0 = 0;
  rsr::Shape shape{};
  int extra_stride = 0;
  std::vector<uint16_t> stream, extras;
  std::vector<rsr::PUnit> units;
  std::vector<uint32_t> blk_unit;
};
int decode_tables(const std::vector<TileTables>& tiles, int64_t rows, int64_t cols, int k, int parts, int part, int64_t block, int32_t* sigma,
                  int32_t* L, std::string* err);

}  // namespace rsr_internal
#endif  // RSR_INTERNAL_H_
