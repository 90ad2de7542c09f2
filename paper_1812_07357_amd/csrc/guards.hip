// Standalone guard fill / merge between the periodic global grid G1 and box arrays.
//
// Sec. 2.5.2 of arXiv:1812.07357: (1) G1 is copied into G2 including the
// guard cells, which are filled from G1 itself (here: the periodic wrap of the
// global index); (3) after the solve the interior, without guards, is copied
// back from G2 to G1.  The add mode sums every box cell (guards included)
// into its wrapped global cell, for sources deposited on boxes; a thread owns
// one global cell and sums its pre-images in a fixed order (no atomics).

#include "internal.hpp"

namespace psatd {

namespace {

constexpr int kT = 256;
constexpr int kMaxFields = 16;

struct PtrSet {
  const void* in[kMaxFields];
  void* out[kMaxFields];
};

// Fill and interior copy move rows: a row (y, z) of kFields arrays per 1 << sh lanes, so that the
// divisions are made once per row and column and a lane has kFields loads in flight.  With one thread per
// value, each dividing its index four times, the fill of 288x160x160 from 256x128x128 in FP32
// (eleven arrays) took 0.285 ms (now 0.140) and the copy back of six 0.087 (now 0.038).  A row takes the
// lanes of the next power of two and at most a wavefront: with a wavefront for every row, boxes of few cells along x
// left most lanes idle (1x512x512, eleven arrays: 178 us, now 15; 8x256x256: 53 us, now 20).
constexpr int kFields = 4;

int row_lanes(int n) {  // log2
  int sh = 0;
  while (sh < 6 && (1 << sh) < n) ++sh;
  return sh;
}

template <typename T>
__device__ __forceinline__ void move_row(const PtrSet& ps, int nfields, long long src, long long dst, int n, int sx,
                                         int GX, bool wrap_src, int sh) {
  const int f0 = blockIdx.y * kFields, lanes = 1 << sh;
  for (int i = threadIdx.x & (lanes - 1); i < n; i += lanes) {
    const int xg = (int)(((unsigned)sx + (unsigned)i) % (unsigned)GX);
    const long long is = src + (wrap_src ? xg : i), id = dst + (wrap_src ? i : xg);
    T v[kFields];
#pragma unroll
    for (int k = 0; k < kFields; ++k)
      if (f0 + k < nfields) v[k] = ((const T*)ps.in[f0 + k])[is];
#pragma unroll
    for (int k = 0; k < kFields; ++k)
      if (f0 + k < nfields) ((T*)ps.out[f0 + k])[id] = v[k];
  }
}

template <typename T>
__global__ void __launch_bounds__(kT) k_fill(PtrSet ps, int nfields, int BX, int BY, int BZ, int sx, int sy, int sz,
                                             int GX, int GY, int GZ, int sh) {
  const long long r = (long long)blockIdx.x * (kT >> sh) + (threadIdx.x >> sh);
  if (r >= (long long)BY * BZ) return;
  const int k = (int)(r / BY), j = (int)(r - (long long)k * BY);
  const long long yg = ((long long)sy + j) % GY, zg = ((long long)sz + k) % GZ;
  move_row<T>(ps, nfields, (zg * GY + yg) * GX, r * BX, BX, sx, GX, true, sh);
}

template <typename T>
__global__ void __launch_bounds__(kT) k_merge_copy(PtrSet ps, int nfields, int BX, int BY, int gx, int gy, int gz,
                                                   int nx, int ny, int nz, int ox, int oy, int oz, int GX, int GY,
                                                   int GZ, int sh) {
  const long long r = (long long)blockIdx.x * (kT >> sh) + (threadIdx.x >> sh);
  if (r >= (long long)ny * nz) return;
  const int k = (int)(r / ny), j = (int)(r - (long long)k * ny);
  const long long yg = ((long long)oy + j) % GY, zg = ((long long)oz + k) % GZ;
  move_row<T>(ps, nfields, ((long long)(k + gz) * BY + (j + gy)) * BX + gx, (zg * GY + yg) * GX, nx, ox, GX, false, sh);
}

// One thread per global cell covered by the box; pre-images along an axis are a, a+G, a+2G, ... < B.
template <typename T>
__global__ void k_merge_add(PtrSet ps, int BX, int BY, int BZ, int sx, int sy, int sz, int GX, int GY, int GZ) {
  const int cx = BX < GX ? BX : GX;
  const int cy = BY < GY ? BY : GY;
  const int cz = BZ < GZ ? BZ : GZ;
  const long long ncov = (long long)cx * cy * cz;
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= ncov) return;
  const int f = blockIdx.y;
  const int a = (int)(q % cx);
  const long long r = q / cx;
  const int b = (int)(r % cy);
  const int c = (int)(r / cy);
  const T* src = (const T*)ps.in[f];
  T* dst = (T*)ps.out[f];
  T acc = T(0);
  for (int k = c; k < BZ; k += GZ)
    for (int j = b; j < BY; j += GY)
      for (int i = a; i < BX; i += GX) acc += src[((long long)k * BY + j) * BX + i];
  const long long xg = ((long long)sx + a) % GX;
  const long long yg = ((long long)sy + b) % GY;
  const long long zg = ((long long)sz + c) % GZ;
  dst[(zg * GY + yg) * GX + xg] += acc;
}

inline unsigned nblk(long long n) { return (unsigned)((n + kT - 1) / kT); }

}  // namespace

void launch_guard_fill(const void* const* g1, void* const* box, int nfields, int esize, const int bd[3],
                       const int start[3], const int gd[3], hipStream_t s) {
  PtrSet ps{};
  for (int f = 0; f < nfields; ++f) {
    ps.in[f] = g1[f];
    ps.out[f] = box[f];
  }
  const int sh = row_lanes(bd[0]), rows = kT >> sh;
  dim3 grid((unsigned)(((long long)bd[1] * bd[2] + rows - 1) / rows), (unsigned)((nfields + kFields - 1) / kFields));
  if (esize == 8)
    hipLaunchKernelGGL(k_fill<double>, grid, dim3(kT), 0, s, ps, nfields, bd[0], bd[1], bd[2], start[0], start[1], start[2],
                       gd[0], gd[1], gd[2], sh);
  else
    hipLaunchKernelGGL(k_fill<float>, grid, dim3(kT), 0, s, ps, nfields, bd[0], bd[1], bd[2], start[0], start[1], start[2],
                       gd[0], gd[1], gd[2], sh);
}

void launch_guard_merge(const void* const* box, void* const* g1, int nfields, int esize, const int bd[3],
                        const int guard[3], const int interior[3], const int origin[3], const int gd[3], int mode,
                        hipStream_t s) {
  PtrSet ps{};
  for (int f = 0; f < nfields; ++f) {
    ps.in[f] = box[f];
    ps.out[f] = g1[f];
  }
  if (mode == 0) {
    const int sh = row_lanes(interior[0]), rows = kT >> sh;
    dim3 grid((unsigned)(((long long)interior[1] * interior[2] + rows - 1) / rows),
              (unsigned)((nfields + kFields - 1) / kFields));
    if (esize == 8)
      hipLaunchKernelGGL(k_merge_copy<double>, grid, dim3(kT), 0, s, ps, nfields, bd[0], bd[1], guard[0], guard[1], guard[2],
                         interior[0], interior[1], interior[2], origin[0], origin[1], origin[2], gd[0], gd[1], gd[2], sh);
    else
      hipLaunchKernelGGL(k_merge_copy<float>, grid, dim3(kT), 0, s, ps, nfields, bd[0], bd[1], guard[0], guard[1], guard[2],
                         interior[0], interior[1], interior[2], origin[0], origin[1], origin[2], gd[0], gd[1], gd[2], sh);
  } else {
    int start[3];
    for (int a = 0; a < 3; ++a) start[a] = (int)((((long long)origin[a] - guard[a]) % gd[a] + gd[a]) % gd[a]);
    const long long n = (long long)(bd[0] < gd[0] ? bd[0] : gd[0]) * (bd[1] < gd[1] ? bd[1] : gd[1]) *
                        (bd[2] < gd[2] ? bd[2] : gd[2]);
    dim3 grid(nblk(n), (unsigned)nfields);
    if (esize == 8)
      hipLaunchKernelGGL(k_merge_add<double>, grid, dim3(kT), 0, s, ps, bd[0], bd[1], bd[2], start[0], start[1],
                         start[2], gd[0], gd[1], gd[2]);
    else
      hipLaunchKernelGGL(k_merge_add<float>, grid, dim3(kT), 0, s, ps, bd[0], bd[1], bd[2], start[0], start[1],
                         start[2], gd[0], gd[1], gd[2]);
  }
}

}  // namespace psatd
