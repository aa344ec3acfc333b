// q-bit matrices as weighted sums of binary matrices (include/rsr_qbit.h): host code on top of the
// C ABI of rsr.h; the products themselves are the binary kernel's.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "../../include/rsr_qbit.h"
#include "rsr_internal.h"
#include "rsr_plan.h"

struct rsr_qbit {
  uint64_t magic = 0;
  int q = 0;
  std::vector<rsr_handle*> groups;  // each the weighted sum of some of the bit planes: one, unless their records do not fit in LDS together
  int64_t table_bytes = 0;
};

namespace {
constexpr uint64_t kMagic = 0x7162697452535221ull;
bool valid(const rsr_qbit* h) { return h && h->magic == kMagic; }
int fail(int code, const std::string& msg) { return rsr_internal::set_error(code, msg); }
}  // namespace

extern "C" {

rsr_qbit* rsr_qbit_preprocess(const int8_t* A, int64_t rows, int64_t cols, int k, int q) {
  if (!A) { fail(RSR_ERR_INVALID_ARGUMENT, "rsr_qbit_preprocess: null pointer"); return nullptr; }
  if (q < 2 || q > 8) { fail(RSR_ERR_INVALID_ARGUMENT, "rsr_qbit_preprocess: q must be in 2..8"); return nullptr; }
  if (rows < 1 || cols < 1) { fail(RSR_ERR_INVALID_ARGUMENT, "rsr_qbit_preprocess: rows and cols must be >= 1"); return nullptr; }
  const int lo = -(1 << (q - 1)), hi = (1 << (q - 1)) - 1;
  const int64_t count = rows * cols;
  for (int64_t i = 0; i < count; ++i)
    if (A[i] < lo || A[i] > hi) {
      fail(RSR_ERR_INVALID_ARGUMENT, "rsr_qbit_preprocess: entry " + std::to_string((int)A[i]) + " at flat index " + std::to_string(i) +
                                         " lies outside " + std::to_string(lo) + ".." + std::to_string(hi));
      return nullptr;
    }
  if (rows > 65534 || k < 1 || k > 16) { fail(RSR_ERR_INVALID_ARGUMENT, "rsr_qbit_preprocess: rows must be in 1..65534 and k in 1..16"); return nullptr; }
  std::unique_ptr<rsr_qbit> h(new (std::nothrow) rsr_qbit());
  if (!h) { fail(RSR_ERR_OUT_OF_MEMORY, "out of host memory"); return nullptr; }
  h->q = q;
  int8_t* dA = rsr_internal::device_copy(A, count, "rsr_qbit_preprocess");
  if (!dA) return nullptr;
  const int per = rsr::planes_per_handle(rows, k, q);
  bool ok = true;
  try {
    for (int p0 = 0; ok && p0 < q; p0 += per) {
      h->groups.reserve((size_t)q);
      rsr_handle* p = rsr_internal::build_planes(dA, rows, cols, k, p0, std::min(per, q - p0), q);
      if (!p) { ok = false; break; }  // (its message stands)
      h->groups.push_back(p);
      rsr_info_t info;
      if (rsr_info(p, &info) == RSR_OK) h->table_bytes += info.table_bytes;
    }
  } catch (const std::bad_alloc&) {
    ok = false;
    fail(RSR_ERR_OUT_OF_MEMORY, "out of host memory");
  }
  rsr_internal::device_release(dA);
  if (!ok) {
    for (rsr_handle* x : h->groups) rsr_destroy(x);
    return nullptr;
  }
  h->magic = kMagic;
  return h.release();
}

int rsr_qbit_matvec(rsr_qbit* h, const float* v, float* out, int batch, void* stream) {
  if (!valid(h)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid handle");
  int rc = rsr_matvec(h->groups[0], v, out, batch, stream);
  for (size_t i = 1; i < h->groups.size() && rc == RSR_OK; ++i) rc = rsr_matvec_acc(h->groups[i], v, out, 1.0f, batch, stream);
  return rc;
}

int rsr_qbit_matvec_i8(rsr_qbit* h, const int8_t* v, int32_t* out, int batch, void* stream) {
  if (!valid(h)) return fail(RSR_ERR_INVALID_ARGUMENT, "invalid handle");
  int rc = rsr_matvec_i8(h->groups[0], v, out, batch, stream);
  for (size_t i = 1; i < h->groups.size() && rc == RSR_OK; ++i) rc = rsr_matvec_acc_i8(h->groups[i], v, out, 1, batch, stream);
  return rc;
}

int rsr_qbit_planes(const rsr_qbit* h) { return valid(h) ? h->q : RSR_ERR_INVALID_ARGUMENT; }
int64_t rsr_qbit_table_bytes(const rsr_qbit* h) { return valid(h) ? h->table_bytes : (int64_t)RSR_ERR_INVALID_ARGUMENT; }

void rsr_qbit_destroy(rsr_qbit* h) {
  if (!valid(h)) return;
  for (rsr_handle* p : h->groups) rsr_destroy(p);
  h->magic = 0;
  delete h;
}

}  // extern "C"
