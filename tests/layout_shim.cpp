// The decoder of the device layout (csrc/rsr_export.cpp) and its split into panels behind plain C functions, for
// tests/test_device_layout.py.
#include <cstring>

#include "rsr_internal.h"

extern "C" {

void shim_shape(int64_t rows, int k, int parts, int signed_pair, int32_t* out) {
  const rsr::Shape s = rsr::panel_shape(rows, k, parts, signed_pair != 0);
  const int32_t x[5] = {s.kc, s.both, s.pslots, s.nslots, s.panels};
  std::memcpy(out, x, sizeof(x));
}

// One tile's tables -> sigma and L of a block; the message goes to `message` (256 bytes).
int shim_decode(int64_t rows, int64_t cols, int k, int parts, const uint16_t* stream, int64_t n_stream, const rsr::PUnit* units, int64_t n_units,
                const uint32_t* blk_unit, const uint16_t* extras, int64_t n_extras, int extra_stride, int part, int64_t block, int32_t* sigma,
                int32_t* L, char* message) {
  std::vector<rsr_internal::TileTables> t(1);
  t[0].rows = rows;
  t[0].shape = rsr::panel_shape(rows, k, parts, true);
  t[0].extra_stride = extra_stride;
  t[0].stream.assign(stream, stream + n_stream);
  t[0].extras.assign(extras, extras + n_extras);
  t[0].units.assign(units, units + n_units);
  t[0].blk_unit.assign(blk_unit, blk_unit + (cols + k - 1) / k + 1);
  std::string err;
  const int rc = rsr_internal::decode_tables(t, rows, cols, k, parts, part, block, sigma, L, &err);
  std::strncpy(message, err.c_str(), 255);
  return rc;
}

}  // extern "C"
