// The words that a launch passes in registers (csrc/rsr_plan.h, start_of), for tests/test_launch_start.py.
#include "rsr_plan.h"

extern "C" {

// Of a planned launch: (planned, unpacked as rsr_body does it) for sets, share_more, g1, rows, vstride, row0, waves, threads, batch.
// -1 if there is no launch.
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
  if (plan_tile(vectors == 4 ? kF4 : vectors == 2 ? kF2 : kF1, h, t, false, batch, num_cu, 4, &plan) != RSR_OK) return -1;
  KArgs& p = plan.p;
  if (threads) p.threads = threads;  // (a launch of several products)
  const int64_t want[9] = {p.sets, p.share_more, p.g1, p.rows, p.vstride, p.row0, p.waves, p.threads, p.batch};
  const Start s = start_of(p);
  const int64_t got[9] = {s.sets_more & 0xffffu, s.sets_more >> 16, s.row0_g1 >> 16, s.rows_stride & 0xffffu, s.rows_stride >> 16, s.row0_g1 & 0xffffu,
                          s.shape & 0xffu, (s.shape >> 8 & 0xffu) * 64, s.shape >> 16};
  for (int i = 0; i < 9; ++i) { planned[i] = want[i]; unpacked[i] = got[i]; }
  return s.share == p.share && s.sets_magic == p.sets_magic ? 0 : 1;
}

}  // extern "C"
