// Every z length: a PML step that psatd_pml_set accepts launches a z pass whose kernel has its tables.
// Both precisions, before and after the autotuner has chosen among the pairs.
#include "internal.hpp"
#include "psatd.h"
#include "fake_hip.hpp"

#include <cstdio>
#include <vector>

using namespace psatd;

static int g_missing, g_stockham, g_pair;

template <typename T>
static void check(const ZPushParams<T>& p, size_t lds) {
  if (p.pair.ra) {
    ++g_pair;
    if (!p.pair.tw || (p.pair.m != p.pair.n && (!p.pair.chirp || !p.pair.filt))) ++g_missing;
  } else {
    ++g_stockham;
    if (!p.fft.tw || (p.fft.blue && (!p.fft.chirp || !p.fft.filt))) ++g_missing;
  }
  if (lds > 160 * 1024) ++g_missing;
}

void on_launch(const std::string& name, void** args, dim3, dim3, size_t lds) {
  if (name.find("zpushIf") != std::string::npos)
    check(*(const ZPushParams<float>*)args[0], lds);
  else if (name.find("zpushId") != std::string::npos)
    check(*(const ZPushParams<double>*)args[0], lds);
}

int main() {
  int bad = 0, accepted = 0;
  std::vector<char> arrays(17);
  void* parts[12];
  const void* src[5];
  for (int f = 0; f < 12; ++f) parts[f] = &arrays[f];
  for (int f = 0; f < 5; ++f) src[f] = &arrays[12 + f];
  for (int prec : {PSATD_FP32, PSATD_FP64})
    for (int nz = 1; nz <= 2048; ++nz) {
      psatd_plan_desc d{};
      d.nx = 4;
      d.ny = 3;
      d.nz = nz;
      d.dx = d.dy = d.dz = d.c = d.eps0 = 1.0;
      d.dt = 0.5;
      d.precision = prec;
      psatd_plan* p = nullptr;
      if (psatd_plan_create_ex(&d, &p) != PSATD_OK) continue;
      const int w[3] = {1, 1, nz > 2 ? 1 : 0};
      for (int order = 0; order < 2; ++order) {  // layers first, then the autotuner; and the reverse
        if (order == 1) {
          psatd_plan_destroy(p);
          psatd_plan_create_ex(&d, &p);
          psatd_plan_autotune(p, nullptr, nullptr);
        }
        if (psatd_pml_set(p, w, 1.0, 2.0) != PSATD_OK) continue;
        ++accepted;
        if (order == 0) psatd_plan_autotune(p, nullptr, nullptr);
        g_missing = g_stockham = g_pair = 0;
        const int rc = psatd_pml_step(p, parts, src, nullptr);
        if (rc != PSATD_OK || g_missing || g_stockham + g_pair != 1) {
          std::printf("%s nz %d order %d: rc %d, %d launches on pairs, %d on Stockham kernels, %d without tables\n",
                      prec == PSATD_FP64 ? "fp64" : "fp32", nz, order, rc, g_pair, g_stockham, g_missing);
          ++bad;
        }
      }
      psatd_plan_destroy(p);
    }
  std::printf("%d steps, %d wrong\n", accepted, bad);
  return bad || accepted < 2000 ? 1 : 0;
}
