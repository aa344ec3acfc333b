// The paper's sigma and L of a column block, recovered from the tables of rsr_layout.h (rsr_export_block).
#include <algorithm>

#include "rsr_internal.h"

namespace rsr_internal {

int decode_tables(const std::vector<TileTables>& tiles, int64_t rows, int64_t cols, int k, int parts, int part, int64_t block, int32_t* sigma,
                  int32_t* L, std::string* err) {
  using namespace rsr;
  const int64_t nblocks = (cols + k - 1) / k;
  if (part < 0 || part >= parts) { *err = "part out of range"; return RSR_ERR_INVALID_ARGUMENT; }
  if (block < 0 || block >= nblocks) { *err = "block out of range"; return RSR_ERR_INVALID_ARGUMENT; }
  const int width = block == nblocks - 1 ? (int)(cols - (nblocks - 1) * k) : k;
  const uint32_t nvals = 1u << width;
  std::vector<std::vector<int32_t>> by_value(nvals);
  std::vector<uint8_t> listed((size_t)rows, 0);
  for (const TileTables& T : tiles) {
    const Shape& S = T.shape;
    const int wbits = k - S.kc;
    std::vector<uint32_t> units_of((size_t)S.panels, 0);
    for (uint32_t ui = T.blk_unit[(size_t)block]; ui < T.blk_unit[(size_t)block + 1]; ++ui) {
      const PUnit& u = T.units[ui];
      if (u.npos > kMaxPositions || u.block != (uint32_t)block) { *err = "corrupt unit"; return RSR_ERR_INVALID_ARGUMENT; }
      const uint32_t pi = u.panel - u.block * (uint32_t)S.panels;
      if (pi >= (uint32_t)S.panels) { *err = "corrupt unit: panel out of range"; return RSR_ERR_INVALID_ARGUMENT; }
      ++units_of[pi];
      const uint16_t* us = &T.stream[(size_t)u.stream_off * (kStreamAlign / 2)];
      const uint64_t heads = (uint64_t)u.heads_lo | ((uint64_t)u.heads_hi << 32);
      const int full = u.npos / kGranulePositions;
      auto at = [&](int p, int lane) {
        if (p < full * kGranulePositions) return us[((p / kGranulePositions) * kLanes + lane) * kGranulePositions + p % kGranulePositions];
        return us[p / 2 * 2 * kLanes + lane * 2 + (p & 1)];
      };
      for (int p0 = 0; p0 < u.npos;) {
        int head = p0;
        while (head < u.npos && !((heads >> head) & 1)) ++head;
        for (int lane = 0; lane < kLanes; ++lane) {
          uint32_t slot = (uint32_t)S.nslots;  // a position behind the last head belongs to no segment
          if (head < u.npos) slot = at(head, u.wide ? lane & ~7 : lane);
          if (slot >= (uint32_t)(S.nslots + kDummySlots)) {  // a piece of a segment that is cut
            const uint32_t e = slot - (uint32_t)(S.nslots + kDummySlots);
            if (e >= u.extras) { *err = "corrupt unit: slot out of range"; return RSR_ERR_INVALID_ARGUMENT; }
            slot = T.extras[(size_t)u.panel * T.extra_stride + e];
          }
          for (int p = p0; p < head; ++p) {
            const uint16_t row = at(p, lane);
            if (row == (uint16_t)T.rows) continue;
            if (row > T.rows || slot >= (uint32_t)S.nslots) { *err = "corrupt unit: row or slot out of range"; return RSR_ERR_INVALID_ARGUMENT; }
            const int of = S.both ? (int)(slot / (uint32_t)S.pslots) : (int)(pi >> wbits);
            if (of != part) continue;
            const uint32_t window = S.both ? 0u : pi & ((1u << wbits) - 1);
            const uint32_t value = ((window << S.kc) | (slot % (uint32_t)S.pslots)) >> (k - width);
            if (value == 0 || value >= nvals || listed[(size_t)(T.row0 + row)]) { *err = "corrupt unit: bad value or repeated row"; return RSR_ERR_INVALID_ARGUMENT; }
            listed[(size_t)(T.row0 + row)] = 1;
            by_value[value].push_back((int32_t)(T.row0 + row));
          }
        }
        p0 = head + 1;
      }
    }
    // (the product waits for exactly this many units of a panel)
    for (uint32_t ui = T.blk_unit[(size_t)block]; ui < T.blk_unit[(size_t)block + 1]; ++ui)
      if (T.units[ui].units_in_panel != units_of[T.units[ui].panel - (uint32_t)block * S.panels]) { *err = "corrupt unit: unit count"; return RSR_ERR_INVALID_ARGUMENT; }
    for (uint32_t n : units_of)
      if (n == 0) { *err = "a panel without units"; return RSR_ERR_INVALID_ARGUMENT; }
  }
  for (int64_t r = 0; r < rows; ++r)
    if (!listed[(size_t)r]) by_value[0].push_back((int32_t)r);  // the rows that are not stored have value 0
  int64_t p = 0;
  for (uint32_t j = 0; j < nvals; ++j) {
    if (L) L[j] = (int32_t)p;
    std::sort(by_value[j].begin(), by_value[j].end());
    for (int32_t r : by_value[j]) {
      if (sigma) sigma[p] = r;
      ++p;
    }
  }
  if (L) L[nvals] = (int32_t)p;
  return RSR_OK;
}

}  // namespace rsr_internal
