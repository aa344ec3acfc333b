// The workgroups' shares of a planned launch (csrc/rsr_plan.h), for tests/test_launch_shares.py.
#include "rsr_plan.h"

extern "C" {

// One launch for `batch` vectors of a matrix of `nblocks` column blocks: writes (set, first block, last block) per workgroup and returns
// their number, -1 if there is no launch.
int64_t shim_shares(int64_t rows, int64_t nblocks, int batch, int vectors, int num_cu, int max_wg_per_cu, int64_t units_per_block, uint32_t* out, int64_t room) {
  using namespace rsr;
  PlanMatrix h;
  PlanTile t;
  h.num_cu = num_cu; h.lds_max = 160 * 1024; h.k = 8;
  h.rows = t.rows = rows; h.nblocks = nblocks; h.cols = nblocks * 8; h.last_width = 8;
  t.shape = panel_shape(rows, 8, 1, true);
  t.max_units_per_block = (uint32_t)units_per_block; t.nunits = nblocks * units_per_block;
  LaunchPlan p;
  if (plan_tile(vectors == 4 ? kF4 : vectors == 2 ? kF2 : kF1, h, t, false, batch, num_cu, max_wg_per_cu, &p) != RSR_OK || p.grid > room) return -1;
  const Start start = start_of(p, p.waves);
  for (int64_t wg = 0; wg < p.grid; ++wg) {
    const Share s = share_of(start, (uint32_t)wg);
    out[3 * wg] = s.set; out[3 * wg + 1] = s.first; out[3 * wg + 2] = s.last;
  }
  return p.grid;
}

}  // extern "C"
