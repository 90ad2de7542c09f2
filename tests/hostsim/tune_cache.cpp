// Every edge length on every axis: a plan of one box and then a batch that holds the same box are autotuned
// through one process cache (the batch runs other kernels for many lengths), and every pass
// of the batch runs a compiled kernel over the whole line.
#include "internal.hpp"
#include "psatd.h"
#include "fake_hip.hpp"

#include <cstdio>
#include <vector>

using namespace psatd;

static bool g_watch;
static int g_bad, g_seen;

static bool stockham_radix(int r) {
  for (int k : {2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 16, 17, 18, 20, 24, 32, 36})
    if (r == k) return true;
  return false;
}

template <typename P>
static void check(const std::string& name, const BatchArgs<P>& a) {
  for (int b = 0; b < a.nbox; ++b) {
    const P& p = a.descs[b];
    ++g_seen;
    bool ok;
    if (name.find("k_p") != std::string::npos) {
      ok = p.pair.ra * p.pair.rb == p.pair.m && p.pair.m >= p.pair.n && p.pair.tw;
    } else {
      const LineSchedule& s = p.fft.sch;
      int prod = 1;
      ok = p.fft.tw != nullptr;
      for (int i = 0; i < s.nstages; ++i) {
        prod *= s.radix[i];
        ok = ok && stockham_radix(s.radix[i]);
      }
      ok = ok && prod == s.n && s.n >= p.fft.n;
    }
    if (!ok) {
      std::printf("%s: line of %d points\n", name.c_str(), p.pair.ra ? p.pair.n : p.fft.n);
      ++g_bad;
    }
  }
}

template <typename T>
static void check_kind(const std::string& name, void** args) {
  if (name.find("xfwd") != std::string::npos) check(name, *(const BatchArgs<XFwdParams<T>>*)args[0]);
  if (name.find("ypass") != std::string::npos) check(name, *(const BatchArgs<YPassParams<T>>*)args[0]);
  if (name.find("zpush") != std::string::npos) check(name, *(const BatchArgs<ZPushParams<T>>*)args[0]);
  if (name.find("xinv") != std::string::npos) check(name, *(const BatchArgs<XInvParams<T>>*)args[0]);
}

void on_launch(const std::string& name, void** args, dim3, dim3, size_t) {
  if (!g_watch || name.find("9BatchArgs") == std::string::npos) return;
  const size_t t = name.find("_bI");  // template arguments: T first, or S and T (the y passes)
  const bool is_float = name.compare(t + 3, 1, "f") == 0 || name.compare(t + 3, 5, "Li1Ef") == 0 ||
                        name.compare(t + 3, 6, "Lin1Ef") == 0;
  if (is_float)
    check_kind<float>(name, args);
  else
    check_kind<double>(name, args);
}

int main() {
  std::vector<char> arrays(11);
  void* g1[11];
  for (int f = 0; f < 11; ++f) g1[f] = &arrays[f];
  for (int prec : {PSATD_FP32, PSATD_FP64})
    for (int axis = 0; axis < 3; ++axis)
      for (int n = 1; n <= 1296; ++n) {
        int e[3] = {5, 5, 5};
        e[axis] = n;
        psatd_plan_desc d{};
        d.nx = e[0];
        d.ny = e[1];
        d.nz = e[2];
        d.dx = d.dy = d.dz = d.c = d.eps0 = 1.0;
        d.dt = 0.5;
        d.precision = prec;
        psatd_plan* p = nullptr;
        if (psatd_plan_create_ex(&d, &p) == PSATD_OK) {
          psatd_plan_autotune(p, nullptr, nullptr);
          psatd_plan_destroy(p);
        }
        psatd_batch* b = nullptr;
        const int origin[3] = {0, 0, 0};
        if (psatd_batch_create(1, &d, origin, e, &b) != PSATD_OK) continue;
        g_watch = true;
        if (psatd_batch_autotune(b, nullptr, nullptr) != PSATD_OK || psatd_batch_step(b, g1, nullptr) != PSATD_OK) ++g_bad;
        g_watch = false;
        psatd_batch_destroy(b);
      }
  std::printf("%d passes, %d wrong\n", g_seen, g_bad);
  return g_bad || g_seen < 5 * 3 * 1500 ? 1 : 0;
}
