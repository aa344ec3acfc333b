// The launch planner (csrc/rsr_plan.h) behind plain C functions, for tests/launch_plan.py.
#include "rsr_plan.h"

using namespace rsr;

namespace {
struct Request {  // an index as the builder would make it, and the call
  int64_t rows, cols, units;  // units: of the whole tile
  int32_t k, parts, planes;   // planes > 0: bit planes in place of parts
  int32_t max_extras, batch, i8;
  int64_t stream;  // bytes of the units; 0: 40 positions each
};
struct Answer {
  int64_t grid, lds, vectors, waves, buffers, workgroups, end_of_lds;
};
PlanMatrix matrix_of(const Request& r, int num_cu, int64_t lds_max) {
  PlanMatrix h;
  h.num_cu = num_cu; h.lds_max = (size_t)lds_max;
  h.rows = r.rows; h.cols = r.cols; h.k = r.k; h.nblocks = (r.cols + r.k - 1) / r.k;
  h.last_width = (int)(r.cols - (h.nblocks - 1) * r.k);
  h.qbit = r.planes > 0;
  return h;
}
PlanTile tile_of(const Request& r, const PlanMatrix& h) {
  PlanTile t;
  t.rows = r.rows; t.shape = panel_shape(r.rows, r.k, r.planes ? r.planes : r.parts, r.planes == 0);
  t.max_extras = r.max_extras; t.nunits = r.units; t.stream_bytes = (size_t)(r.stream ? r.stream : r.units * 40 * kPositionBytes);
  t.max_units_per_block = (uint32_t)((r.units + h.nblocks - 1) / h.nblocks);
  return t;
}
void answer(const LaunchPlan& p, const Pass& pass, Answer* a) {
  *a = Answer{p.grid, (int64_t)p.lds, pass.V, p.waves, p.p.nbuf, p.g1, (int64_t)p.p.off_ctr + 4};
}
}  // namespace

extern "C" {

int shim_panels(int64_t rows, int k, int parts, int planes) { return panel_shape(rows, k, planes ? planes : parts, planes == 0).panels; }
int shim_planes_per_handle(int64_t rows, int k, int q) { return planes_per_handle(rows, k, q); }

int shim_product(const Request* r, int num_cu, int64_t lds_max, Answer* a) {
  const PlanMatrix h = matrix_of(*r, num_cu, lds_max);
  const PlanTile t = tile_of(*r, h);
  Mode mode;
  LaunchPlan p;
  const int rc = plan_product(r->i8 != 0, h, t, false, r->batch, &mode, &p);
  if (rc == RSR_OK) answer(p, pass_of(r->i8 != 0, mode), a);
  return rc;
}

int shim_shared(const Request* r, int n, int num_cu, int64_t lds_max, Answer* a) {
  PlanMatrix h[kMaxJobs];
  PlanTile t[kMaxJobs];
  SharedJob jobs[kMaxJobs];
  LaunchPlan p[kMaxJobs];
  for (int j = 0; j < n; ++j) {
    h[j] = matrix_of(r[j], num_cu, lds_max);
    t[j] = tile_of(r[j], h[j]);
    jobs[j] = {&h[j], &t[j], r[j].units * 40 * 128};
  }
  Mode mode;
  int failed = 0;
  const int rc = plan_shared(r[0].i8 != 0, jobs, n, num_cu, r[0].batch, &mode, p, &failed);
  for (int j = 0; rc == RSR_OK && j < n; ++j) answer(p[j], pass_of(r[0].i8 != 0, mode), &a[j]);
  return rc;
}

}  // extern "C"
