// Device bytes of a plan with absorbing layers: the twelve-field layout B and the damping tables, and the
// full fields and increments only where the x axis runs on the Stockham kernels.  A psatd_pml_set that ran out
// of memory half way allocates nothing twice when it is called again.
#include "psatd.h"
#include "fake_hip.hpp"

#include <cstdio>

void on_launch(const std::string&, void**, dim3, dim3, size_t) {}

static long long bytes_of(psatd_plan* p) {
  long long v = 0;
  psatd_plan_query(p, PSATD_Q_WORKSPACE_BYTES, &v);
  return v;
}

int main() {
  int bad = 0;
  for (int prec : {PSATD_FP32, PSATD_FP64})
    for (int nx : {24, 245}) {
      const long long rs = prec == PSATD_FP64 ? 8 : 4, ny = 6, nz = 10, cells = nx * ny * nz, pts = (nx / 2 + 1) * ny * nz;
      psatd_plan_desc d{};
      d.nx = nx;
      d.ny = (int)ny;
      d.nz = (int)nz;
      d.dx = d.dy = d.dz = d.c = d.eps0 = 1.0;
      d.dt = 0.5;
      d.precision = prec;
      const long long boxes = nx == 245 ? 12 * cells * rs : 0;  // 245 = 5 * 7 * 7: no pair
      const long long want = 12 * pts * 2 * rs + (nx + ny + nz) * rs + boxes;
      const int w[3] = {2, 1, 1};
      psatd_plan* p = nullptr;
      if (psatd_plan_create_ex(&d, &p) != PSATD_OK) return 2;
      const long long before = bytes_of(p);
      // a budget that the first allocations fit and the last does not
      psatd_set_device_budget(psatd_device_bytes_in_use() + want - rs);
      if (psatd_pml_set(p, w, 1.0, 2.0) != PSATD_ENOMEM) ++bad;
      psatd_set_device_budget(-1);
      if (psatd_pml_set(p, w, 1.0, 2.0) != PSATD_OK || psatd_pml_set(p, w, 2.0, 2.0) != PSATD_OK) ++bad;
      if (bytes_of(p) - before != want) {
        std::printf("nx %d: %lld bytes, expected %lld\n", nx, bytes_of(p) - before, want);
        ++bad;
      }
      psatd_plan_destroy(p);
      if (psatd_device_bytes_in_use() != 0) ++bad;
    }
  return bad;
}
