// The words that a launch passes in registers (csrc/rsr_plan.h, start_of), for tests/test_launch_start.py.
#include "rsr_plan.h"

extern "C" {

// Of a planned launch: (planned, as the kernels read it back) for sets, share_more, g1, rows, vstride, row0, waves, threads, batch.
// A negative status if there is no launch.
int shim_start(int64_t rows, int64_t all_rows, int64_t row0, int64_t nblocks, int k, int batch, int vectors, int num_cu, int threads, int64_t* planned,
               int64_t* unpacked) {
  using namespace rsr;
  PlanMatrix h;
  PlanTile t;
  h.num_cu = num_cu; h.lds_max = 160 * 1024; h.k = k;
  h.rows = all_rows; h.nblocks = nblocks; h.cols = nblocks * k; h.last_width = k;
  t.rows = rows; t.row0 = row0; t.shape = panel_shape(rows, k, 1, true);
  t.max_units_per_block = 4; t.nunits = nblocks * 4; t.stream_bytes = (size_t)t.nunits * 40 * kPositionBytes;
  LaunchPlan plan;
  const int rc = plan_tile(vectors == 4 ? kF4 : vectors == 2 ? kF2 : kF1, h, t, false, batch, num_cu, 4, &plan);
  if (rc != RSR_OK) return rc;
  if (!threads) threads = plan.waves * 64;  // (otherwise a launch of several products)
  const int64_t want[9] = {plan.sets, plan.share_more, plan.g1, plan.rows, plan.vstride, plan.row0, plan.waves, threads, plan.batch};
  const Start s = start_of(plan, threads / 64);
  const int64_t got[9] = {s.sets(), s.share_more(), s.g1(), s.rows(), s.vstride(), s.row0(), s.waves(), s.threads(), s.batch()};
  for (int i = 0; i < 9; ++i) { planned[i] = want[i]; unpacked[i] = got[i]; }
  return s.share == plan.share && s.sets_magic == magic((uint32_t)plan.sets) ? 0 : 1;
}

}  // extern "C"
