// Particle side of the PIC cycle around the PSATD step (gfx950): field gather +
// relativistic Boris push, and current / charge deposition through D1 tiles.
//
// arXiv:1812.07357, Sec. 2.5.1 (Fig. 4): particles are pushed with the fields at
// their positions, their current and charge are deposited with linear
// interpolation, Maxwell's equations are solved, and the fields are gathered
// back.  Sec. 2.5.2: particle-mesh work runs on the grid G1 split into
// sub-domains D1 whose guard cells are as wide as the interpolation stencil,
// while the FFTs run on the boxes of G2 (decomposition D2, psatd_step_g1 /
// psatd_batch_*), coupled by guard fill and interior copy.
//
// Here a D1 sub-domain is a tile of T^3 cells of G1 worked on by one workgroup:
// the particles are counted per tile (by their start position), the tile
// offsets scanned, the particles listed per tile, and each workgroup deposits its
// tile's particles into LDS over the tile plus its guard cells (Reach<K>::lo below,
// Reach<K>::hi above, per axis), then adds that LDS block into G1 (the guard cells land
// on the neighbouring tiles' cells: the additive guard merge of the D1
// decomposition).  The guards hold the stencil of a particle that started in
// the tile and moved less than one cell during the step, which the host ensures
// (c dt below the smallest cell size, with a margin for rounding).  The LDS block sums in
// 64-bit fixed point with a power-of-two scale per tile, so a tile's sums are exact and do
// not depend on the order of the atomics.
//
// Weights: a quantity of a component with half-cell offset o sits at grid point
// (i + o/2) d; a particle at x spreads over the (K+1)^3 points around it with the
// product of the 1D centred B-spline weights of degree K (Sec. 2.5.1 allows linear or
// higher-order interpolation: K = 1 cloud in cell, 2 triangular-shaped cloud, 3 cubic),
// and the gather uses the same weights.  rho = q S / (dx dy dz)
// at the start and end positions, J = q v S / (dx dy dz) at the mid-point with
// the half-step velocity.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <vector>

#include "../../include/psatd.h"
#include "internal.hpp"
#include "row_run.hpp"

namespace psatd {
namespace {

constexpr int kPicThreads = 256;
constexpr int kXcds = 8;  // workgroups go round the chiplets in this order
// Threads of a deposit workgroup.  Its LDS block (53 KB linear, 88 KB above) leaves one to three
// workgroups per CU, and the particle reads through the list wait on memory: with 256 threads
// the deposit of 33.5 M cubic particles in random order took 11.6 ms, with 1024 9.5 ms; 67 M
// linear ones 4.77 ms, with 512 4.50 ms.
template <int K>
constexpr int kDepositThreads = K == 1 ? 512 : 1024;
// Stencil reach of a particle that starts in cell c and moves less than one cell, for
// weights of degree K: the points of rho_new and of J (mid-point, half a cell away) span
// [c - 1, c + 2] (K = 1) or [c - 2, c + 3] (K = 2, 3).
template <int K>
struct Reach {
  static constexpr int lo = K == 1 ? 1 : 2, hi = K == 1 ? 2 : 3;
};
constexpr int kMaxShape = 3;
// c dt may reach this fraction of the smallest cell (the rest absorbs rounding).
constexpr double kMaxCourant = 0.999;
constexpr int kTileMax = 12;

template <typename T>
struct PicArgs {
  int gx, gy, gz;
  T dx, dy, dz;   // cell sizes
  T idx, idy, idz;  // 1 / cell sizes
  T lx, ly, lz;   // periodic lengths
  T dt, c, q, qm;
  T inv_vol;
  int stag;
  int tile, tx, ty, tz, ntiles;  // D1 tiles: edge, tiles per axis, total
  int n;
};

// Centred B-spline weights of degree K of coordinate s (in cells): the K + 1 points
// first, ..., first + K and their weights.
template <int K, typename T>
__device__ __forceinline__ void shape1d(T s, int& first, T* w) {
  if constexpr (K == 1) {
    const T f = floor(s), t = s - f;
    first = (int)f;
    w[0] = T(1) - t;
    w[1] = t;
  } else if constexpr (K == 2) {
    const T r = floor(s + T(0.5)), t = s - r;
    first = (int)r - 1;
    w[0] = T(0.5) * (T(0.5) - t) * (T(0.5) - t);
    w[1] = T(0.75) - t * t;
    w[2] = T(0.5) * (T(0.5) + t) * (T(0.5) + t);
  } else {
    const T f = floor(s), t = s - f, t2 = t * t, t3 = t2 * t, u = T(1) - t;
    first = (int)f - 1;
    w[0] = u * u * u / T(6);
    w[1] = (T(4) - T(6) * t2 + T(3) * t3) / T(6);
    w[2] = (T(1) + T(3) * t + T(3) * t2 - T(3) * t3) / T(6);
    w[3] = t3 / T(6);
  }
}


// Index i of an axis of n cells folded into [0, n): positions in [0, L) need at most one
// add or subtract; the clamp keeps out-of-contract positions inside the array.
__device__ __forceinline__ int fold(int i, int n) {
  if (i < 0) i += n;
  if (i >= n) i -= n;
  return min(max(i, 0), n - 1);
}

// The (K+1)^3 G1 points around (x, y, z) (lengths) of a quantity with half-cell offsets
// (ox, oy, oz), periodic G1, as per-axis folded indices and weights.
template <int K, typename T>
struct Points {
  int xs[K + 1], ys[K + 1], zs[K + 1];
  T wx[K + 1], wy[K + 1], wz[K + 1];
};

template <int K, typename T>
__device__ __forceinline__ void grid_points(Points<K, T>& g, const PicArgs<T>& a, T x, T y, T z, int ox, int oy,
                                            int oz) {
  int fx, fy, fz;
  shape1d<K>(x * a.idx - T(0.5) * ox, fx, g.wx);
  shape1d<K>(y * a.idy - T(0.5) * oy, fy, g.wy);
  shape1d<K>(z * a.idz - T(0.5) * oz, fz, g.wz);
#pragma unroll
  for (int c = 0; c <= K; ++c) {
    g.xs[c] = fold(fx + c, a.gx);
    g.ys[c] = fold(fy + c, a.gy) * a.gx;
    g.zs[c] = fold(fz + c, a.gz) * a.gy * a.gx;
  }
}

template <int K, typename T>
__device__ __forceinline__ T gather_at(const T* __restrict__ f, const Points<K, T>& g) {
  T acc = 0;
  // the x points are consecutive unless the stencil wraps around the periodic edge
  const bool run = g.xs[K] == g.xs[0] + K;
#pragma unroll
  for (int cz = 0; cz <= K; ++cz)
#pragma unroll
    for (int cy = 0; cy <= K; ++cy) {
      const T wyz = g.wy[cy] * g.wz[cz];
      const T* row = f + g.zs[cz] + g.ys[cy];
      RowRun<K, T> r;
      if (run) {
        r = load_run<K>(row + g.xs[0]);
      } else {
#pragma unroll
        for (int cx = 0; cx <= K; ++cx) r.v[cx] = row[g.xs[cx]];
      }
#pragma unroll
      for (int cx = 0; cx <= K; ++cx) acc += r.v[cx] * (g.wx[cx] * wyz);
    }
  return acc;
}

// The six components of every G1 cell side by side ([cell][6]) for the gather of k_pic_push:
// four (FP32) or two (FP64) cells per thread, in 16-byte loads and stores.  Particles that are no
// longer in cell order find nothing of their stencil in the caches: gathered from six arrays
// one cubic particle touched 96 rows in as many cache lines, and the push was bound by
// the lines moved (7 TB/s out of the 256 MB cache).  Side by side its stencil is 16 rows of
// 96 bytes.  33.5 M cubic particles in random order on 256x128x128, FP32: 61.1 -> 15.9 ms
// (linear 14.8 -> 3.5); 67 M linear ones in cell order on 512x256x256 1.63 -> 1.59 ms, 44
// steps later 10.8 -> 4.3 ms; 16.8 M cubic ones in FP64 33.6 -> 11.6 ms.
template <typename T>
struct Six {
  const T* f[6];
};
template <typename T>
__global__ void __launch_bounds__(kPicThreads) k_interleave(Six<T> a, T* __restrict__ out, long long ncell) {
  constexpr int V = 16 / sizeof(T);  // cells per thread
  typedef T vec_t __attribute__((ext_vector_type(V)));
  const long long i = ((long long)blockIdx.x * kPicThreads + threadIdx.x) * V;
  if (i >= ncell) return;
  // the arrays are the caller's: vectors only where every one of them is 16-byte aligned
  bool whole = i + V <= ncell;
#pragma unroll
  for (int k = 0; k < 6; ++k) whole = whole && ((uintptr_t)a.f[k] & 15) == 0;
  if (whole) {
    T v[6 * V];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const vec_t w = *reinterpret_cast<const vec_t*>(a.f[k] + i);
#pragma unroll
      for (int c = 0; c < V; ++c) v[c * 6 + k] = w[c];
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      vec_t w;
#pragma unroll
      for (int c = 0; c < V; ++c) w[c] = v[k * V + c];
      *reinterpret_cast<vec_t*>(out + i * 6 + k * V) = w;
    }
  } else {
    for (long long c = i; c < ncell && c < i + V; ++c)
#pragma unroll
      for (int k = 0; k < 6; ++k) out[c * 6 + k] = a.f[k][c];
  }
}

// All six components at a particle from the interleaved cells: a row of K + 1 points is one run of
// 6 (K + 1) values.  Above degree 1 one plane of rows is in flight at a time (a loop that is not
// unrolled): the loads of all planes together took 424 registers at degree 3 and left one wavefront
// per SIMD (67 M particles in cell order, FP32: 10.4 ms against 5.3; 16.8 M in random order, FP64: 28.5 against 11.6).
template <int K, typename T>
__device__ __forceinline__ void gather_six(T* eb, const T* __restrict__ cells, Points<K, T>& g) {
  // 16-byte loads; FP32 rows of three points are 18 values, in 8-byte loads
  constexpr int V = sizeof(T) == 8 || K == 2 ? 2 : 4, NV = 6 * (K + 1) / V;
  typedef T vec_t __attribute__((ext_vector_type(V), aligned(alignof(T))));
#pragma unroll
  for (int k = 0; k < 6; ++k) eb[k] = 0;
  const bool run = g.xs[K] == g.xs[0] + K;
#pragma unroll(K == 1 ? 2 : 1)
  for (int cz = 0; cz <= K; ++cz) {
#pragma unroll
    for (int cy = 0; cy <= K; ++cy) {
      const T wyz = g.wy[cy] * g.wz[0];
      const long long row = (long long)g.zs[0] + g.ys[cy];
      T v[6 * (K + 1)];
      if (run) {
        const vec_t* p = reinterpret_cast<const vec_t*>(cells + (row + g.xs[0]) * 6);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          const vec_t w = p[q];
#pragma unroll
          for (int c = 0; c < V; ++c) v[q * V + c] = w[c];
        }
      } else {
#pragma unroll
        for (int cx = 0; cx <= K; ++cx)
#pragma unroll
          for (int k = 0; k < 6; ++k) v[cx * 6 + k] = cells[(row + g.xs[cx]) * 6 + k];
      }
#pragma unroll
      for (int cx = 0; cx <= K; ++cx) {
        const T w = g.wx[cx] * wyz;
#pragma unroll
        for (int k = 0; k < 6; ++k) eb[k] += v[cx * 6 + k] * w;
      }
    }
    // the next plane moves to the front (no index that varies at run time into the registers)
#pragma unroll
    for (int c = 0; c < K; ++c) {
      g.wz[c] = g.wz[c + 1];
      g.zs[c] = g.zs[c + 1];
    }
  }
}

template <typename T>
struct PushPtrs {
  const T* f[6];  // Ex Ey Ez Bx By Bz on G1
  const T* cells; // the same interleaved (collocated grid), or NULL
  T* x[3];
  T* u[3];
  T* x_old[3];
};

// Gather E, B at x, relativistic Boris push of u = gamma v, x moved by dt u / gamma (wrapped).
// STAG: staggered grid (each component at its own half-cell offsets); otherwise the six
// components share one set of points and weights.  SIX: from interleaved cells.
template <typename T, bool STAG, int K, bool SIX>
__global__ void __launch_bounds__(kPicThreads) __attribute__((amdgpu_waves_per_eu(2))) k_pic_push(PicArgs<T> a, PushPtrs<T> p) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  // the particle arrays stream through once (non-temporal), which leaves the caches to the
  // field rows that neighbouring particles gather again
  const T x = __builtin_nontemporal_load(&p.x[0][i]), y = __builtin_nontemporal_load(&p.x[1][i]),
          z = __builtin_nontemporal_load(&p.x[2][i]);
  T E[3], B[3];
  Points<K, T> g;
  if constexpr (SIX) {
    T eb[6];
    grid_points<K>(g, a, x, y, z, 0, 0, 0);
    gather_six<K>(eb, p.cells, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      E[c] = eb[c];
      B[c] = eb[3 + c];
    }
  } else if constexpr (K > 1) {
    // one field at a time (a loop that is not unrolled), so that the (K+1)^3 loads of one
    // field are in flight together without the registers of all six
    T eb[6];
    if constexpr (!STAG) grid_points<K>(g, a, x, y, z, 0, 0, 0);
#pragma unroll 1
    for (int k = 0; k < 6; ++k) {
      if constexpr (STAG) {
        // E_a half a cell up along a; B_a along the two other axes
        const int c = k < 3 ? k : k - 3;
        const bool e = k < 3;
        grid_points<K>(g, a, x, y, z, (c == 0) == e, (c == 1) == e, (c == 2) == e);
      }
      const T v = gather_at<K>(p.f[k], g);
#pragma unroll
      for (int j = 0; j < 6; ++j)
        if (j == k) eb[j] = v;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      E[c] = eb[c];
      B[c] = eb[3 + c];
    }
  } else if constexpr (STAG) {
    // E_a half a cell up along a; B_a along the two other axes
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      grid_points<K>(g, a, x, y, z, k == 0, k == 1, k == 2);
      E[k] = gather_at<K>(p.f[k], g);
      grid_points<K>(g, a, x, y, z, k != 0, k != 1, k != 2);
      B[k] = gather_at<K>(p.f[3 + k], g);
    }
  } else {
    grid_points<K>(g, a, x, y, z, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      E[k] = gather_at<K>(p.f[k], g);
      B[k] = gather_at<K>(p.f[3 + k], g);
    }
  }
  const T h = T(0.5) * a.qm * a.dt;
  const T ic2 = T(1) / (a.c * a.c);
  T um[3] = {__builtin_nontemporal_load(&p.u[0][i]) + h * E[0], __builtin_nontemporal_load(&p.u[1][i]) + h * E[1],
             __builtin_nontemporal_load(&p.u[2][i]) + h * E[2]};
  const T gm = sqrt(T(1) + (um[0] * um[0] + um[1] * um[1] + um[2] * um[2]) * ic2);
  const T t[3] = {h * B[0] / gm, h * B[1] / gm, h * B[2] / gm};
  const T t2 = t[0] * t[0] + t[1] * t[1] + t[2] * t[2];
  const T s[3] = {T(2) * t[0] / (T(1) + t2), T(2) * t[1] / (T(1) + t2), T(2) * t[2] / (T(1) + t2)};
  const T up[3] = {um[0] + um[1] * t[2] - um[2] * t[1], um[1] + um[2] * t[0] - um[0] * t[2],
                   um[2] + um[0] * t[1] - um[1] * t[0]};
  const T un[3] = {um[0] + up[1] * s[2] - up[2] * s[1] + h * E[0], um[1] + up[2] * s[0] - up[0] * s[2] + h * E[1],
                   um[2] + up[0] * s[1] - up[1] * s[0] + h * E[2]};
  const T gn = sqrt(T(1) + (un[0] * un[0] + un[1] * un[1] + un[2] * un[2]) * ic2);
  const T L[3] = {a.lx, a.ly, a.lz};
  const T xs[3] = {x, y, z};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T xn = xs[k] + a.dt * un[k] / gn;
    xn -= L[k] * floor(xn / L[k]);
    if (xn >= L[k]) xn -= L[k];  // rounding at the upper edge
    __builtin_nontemporal_store(xs[k], &p.x_old[k][i]);
    __builtin_nontemporal_store(xn, &p.x[k][i]);
    __builtin_nontemporal_store(un[k], &p.u[k][i]);
  }
}

// D1 tile of a start position.
template <typename T>
__device__ __forceinline__ int tile_of(const PicArgs<T>& a, T x, T y, T z) {
  // clamped, so that a position outside [0, L) cannot index past the tile arrays
  const int cx = min(max((int)(x * a.idx), 0), a.gx - 1), cy = min(max((int)(y * a.idy), 0), a.gy - 1),
            cz = min(max((int)(z * a.idz), 0), a.gz - 1);
  return ((cz / a.tile) * a.ty + cy / a.tile) * a.tx + cx / a.tile;
}

template <typename T>
struct DepPtrs {
  const T* xo[3];
  const T* xn[3];
  const T* u[3];
  T* g[5];  // Jx Jy Jz rho_old rho_new on G1
  int* count;   // ntiles
  int* offset;  // ntiles + 1
  int* cursor;  // ntiles
  int* list;    // n particle indices, tile by tile
};

// (Indices of tiles are unsigned where they step past the last one: a grid may have almost 2^31.)
__global__ void k_zero_int(int* a, unsigned n) {
  const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0;
}

template <typename T>
__global__ void k_zero_fields(DepPtrs<T> p, long long ncell) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ncell)
#pragma unroll
    for (int f = 0; f < 5; ++f) p.g[f][i] = T(0);
}

// Runs of equal keys in consecutive lanes of a wave: whether this lane leads its run,
// the run's leading lane and (at the leader) its length.  Inactive lanes carry
// distinct keys, so they never join a run.  Every lane of the wave must call it.
struct WaveRun {
  bool head;
  int leader, len;
};
__device__ __forceinline__ WaveRun wave_run(int key, bool active) {
  const int lane = __lane_id();
  const int k = active ? key : -1 - lane;
  const int prev = __shfl_up(k, 1);
  const bool head = lane == 0 || prev != k;
  const unsigned long long heads = __ballot(head);
  const unsigned long long upto = (2ull << lane) - 1ull;  // lanes 0..lane (all for lane 63)
  const unsigned long long after = heads & ~upto;
  WaveRun r;
  r.head = head;
  r.leader = 63 - __clzll(heads & upto);
  r.len = (after ? __ffsll((long long)after) - 1 : 64) - lane;
  return r;
}

// A table in LDS that gathers what a workgroup adds to the tiles' counters: particles that have left
// their cell order make few runs, and one global atomic for each of them bound the count and
// the list (67 M particles on 65536 tiles, 62 steps after cell order: 1.23 -> 0.26 and 2.22 -> 0.39
// ms; in cell order 0.24 and 0.34 ms before and after; 33.5 M in random order on 8192 tiles
// 1.13 -> 0.24 and 1.14 -> 0.82 ms).  A tile is entered in one of kProbes slots from its hash on;
// a tile that finds them taken stays outside for good, and its particles go to the
// global counter one by one.  Grids of up to kSlots tiles never collide.
constexpr int kTileThreads = 1024;  // two workgroups per CU with the table's 64 KB
constexpr int kSlots = 8192, kProbes = 4;
// Particles of a thread in one fill of the list's table: many meet in a table only if it is filled
// with many, few leave no CU without a workgroup where there are few in all.
constexpr int kListRun = 16, kListRunFew = 4;
constexpr int kListMany = 256 * kTileThreads * kListRun;
struct TileTable {
  int tag[kSlots], n[kSlots];
};
__device__ __forceinline__ void table_clear(TileTable& t) {
  for (int i = threadIdx.x; i < kSlots; i += kTileThreads) {
    t.tag[i] = -1;
    t.n[i] = 0;
  }
}
// multiplied by an odd number: a bijection of the low bits that parts the tiles of a plane
__device__ __forceinline__ int table_hash(int tile) { return (tile * 2531) & (kSlots - 1); }
__device__ __forceinline__ int table_enter(TileTable& t, int tile) {
  int s = table_hash(tile);
  for (int k = 0; k < kProbes; ++k, s = (s + 1) & (kSlots - 1)) {
    const int was = atomicCAS(&t.tag[s], -1, tile);
    if (was == -1 || was == tile) return s;
  }
  return -1;
}
__device__ __forceinline__ int table_find(const TileTable& t, int tile) {
  int s = table_hash(tile);
  for (int k = 0; k < kProbes; ++k, s = (s + 1) & (kSlots - 1))
    if (t.tag[s] == tile) return s;
  return -1;
}

// Particles per D1 tile: each workgroup counts one contiguous range of `chunk` particles in its
// table; particles of one tile in consecutive lanes (cell-ordered input) add their count at once.
template <typename T>
__global__ void __launch_bounds__(kTileThreads) k_tile_count(PicArgs<T> a, DepPtrs<T> p, int chunk) {
  __shared__ TileTable table;
  table_clear(table);
  __syncthreads();
  const long long lo = (long long)blockIdx.x * chunk, hi = min((long long)a.n, lo + chunk);
  for (long long b = lo; b < hi; b += kTileThreads) {
    const long long i = b + threadIdx.x;
    const bool active = i < hi;
    const int t = active ? tile_of(a, p.xo[0][i], p.xo[1][i], p.xo[2][i]) : 0;
    const WaveRun r = wave_run(t, active);
    if (active && r.head) {
      const int s = table_enter(table, t);
      atomicAdd(s >= 0 ? &table.n[s] : &p.count[t], r.len);
    }
  }
  __syncthreads();
  for (int s = threadIdx.x; s < kSlots; s += kTileThreads)
    if (table.n[s]) atomicAdd(&p.count[table.tag[s]], table.n[s]);
}

// Exclusive scan of the tile counts by one workgroup (offset[ntiles] = n); cursors start at the
// offsets.  Four counts per thread and round, the next round's loaded before this one is summed
// (65536 tiles: 0.152 -> 0.048 ms; the threads walked ranges of their own before).
__global__ void __launch_bounds__(1024) k_tile_scan(const int* count, int* offset, int* cursor, unsigned ntiles) {
  __shared__ int wsum[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int next[4], carry = 0;
  auto load = [&](unsigned i0) {
#pragma unroll
    for (unsigned k = 0; k < 4; ++k) next[k] = i0 + k < ntiles ? count[i0 + k] : 0;
  };
  load(tid * 4);
  int par = 0;
  for (unsigned base = 0; base < ntiles; base += 4096, par ^= 1) {
    const unsigned i0 = base + tid * 4;
    int c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = next[k];
    load(i0 + 4096);
    const int mine = c[0] + c[1] + c[2] + c[3];
    int inc = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int v = __shfl_up(inc, d);
      if (lane >= d) inc += v;
    }
    if (lane == 63) wsum[par][wave] = inc;
    __syncthreads();  // one per round: the other half of wsum is the last round's
    int run = carry + inc - mine;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int v = wsum[par][w];
      if (w < wave) run += v;
      carry += v;
    }
#pragma unroll
    for (unsigned k = 0; k < 4; ++k) {
      if (i0 + k < ntiles) {
        offset[i0 + k] = run;
        cursor[i0 + k] = run;
      }
      run += c[k];
    }
  }
  if (tid == 0) offset[ntiles] = carry;
}

// Particle indices listed tile by tile: a workgroup counts RUN particles per thread in its
// table, takes the tiles' slots with one atomic each and fills them; a run of one tile's
// particles in consecutive lanes lies in lane order.
template <typename T, int RUN>
__global__ void __launch_bounds__(kTileThreads) k_tile_list(PicArgs<T> a, DepPtrs<T> p) {
  __shared__ TileTable table;
  table_clear(table);
  const long long lo = (long long)blockIdx.x * (kTileThreads * RUN) + threadIdx.x;
  int t[RUN];
#pragma unroll
  for (int k = 0; k < RUN; ++k) {
    const long long i = lo + k * kTileThreads;
    t[k] = i < a.n ? tile_of(a, p.xo[0][i], p.xo[1][i], p.xo[2][i]) : -1;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < RUN; ++k) {
    const WaveRun r = wave_run(t[k], t[k] >= 0);
    if (t[k] >= 0 && r.head) {
      const int s = table_enter(table, t[k]);
      if (s >= 0) atomicAdd(&table.n[s], r.len);
    }
  }
  __syncthreads();
  for (int s = threadIdx.x; s < kSlots; s += kTileThreads)
    if (table.n[s]) table.n[s] = atomicAdd(&p.cursor[table.tag[s]], table.n[s]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < RUN; ++k) {
    const WaveRun r = wave_run(t[k], t[k] >= 0);
    int base = 0;
    if (t[k] >= 0 && r.head) {
      const int s = table_find(table, t[k]);
      base = atomicAdd(s >= 0 ? &table.n[s] : &p.cursor[t[k]], r.len);
    }
    base = __shfl(base, r.leader);
    if (t[k] >= 0) p.list[base + (int)__lane_id() - r.leader] = (int)(lo + k * kTileThreads);
  }
}

// The stencil of one particle position inside the LDS block of a tile, in separable form: the
// block-local index of its first point and the 1D weights per axis.  The block spans
// E = T + Reach<K>::lo + Reach<K>::hi cells per axis from the tile's first cell (bx, by, bz)
// minus Reach<K>::lo.
template <int K, typename T>
struct Axes {
  int l0;
  T wx[K + 1];
  double wyz[(K + 1) * (K + 1)];
};

template <int K, typename T>
__device__ __forceinline__ void stencil_axes(Axes<K, T>& s, int E, const PicArgs<T>& a, int ox, int oy, int oz, T x,
                                             T y, T z, int bx, int by, int bz) {
  int ix, iy, iz;
  T wy[K + 1], wz[K + 1];
  shape1d<K>(x * a.idx - T(0.5) * ox, ix, s.wx);
  shape1d<K>(y * a.idy - T(0.5) * oy, iy, wy);
  shape1d<K>(z * a.idz - T(0.5) * oz, iz, wz);
#pragma unroll
  for (int c = 0; c < (K + 1) * (K + 1); ++c) s.wyz[c] = (double)wy[c % (K + 1)] * (double)wz[c / (K + 1)];
  // local indices relative to the block origin (tile origin - guard); positions near the
  // periodic edge are taken on the tile's side of the edge.  For positions in [0, L) whose
  // particle started in the tile the first point lies in [0, E - 1 - K]; the clamp only
  // keeps positions that break that contract inside the block.
  auto local = [&](int i, int b, int n) {
    int l = i - (b - Reach<K>::lo);
    if (l < 0) l += n;
    if (l >= n) l -= n;
    return min(max(l, 0), E - 1 - K);
  };
  s.l0 = (local(iz, bz, a.gz) * E + local(iy, by, a.gy)) * E + local(ix, bx, a.gx);
}

// The LDS block accumulates in 64-bit fixed point: each weighted value times a power of two
// (its scale), rounded to an integer, added with an integer LDS atomic (floating-point LDS
// atomics are several times slower).  Integer sums are exact and independent of their order;
// the scale keeps every sum below 2^62 in magnitude (see k_deposit_tiles).
//
// The tile kernel was bound by vector instructions (0.82 per cycle and CU of at most 1 for linear
// shapes), most of them the conversion to an integer: without it and with one stencil for the three
// components of J the cubic kernel went from 6.1 to 5.1 ms (33.5 M particles in random order,
// FP32), then bound by the bank conflicts of its atomics, the linear one from 4.20 to 4.04
// (67 M, 62 steps after cell order).  A product p = w wyz of two doubles becomes one here by
// the addition of kMagic = 1.5 * 2^52, whose sum holds p rounded to the nearest integer in its
// low bits: with |p| < 2^51 (WORDS 1) one fma and one subtraction from the high word.  Larger p
// (WORDS 2, w given in units of 2^32) are split exactly into a multiple of 2^32 and a rest.
using fixed_t = unsigned long long;
constexpr double kMagic = 6755399441055744.0;         // 1.5 * 2^52
constexpr unsigned kMagicHi = 0x43380000u;            // its high word (the low one is 0)
constexpr double kOneWord = 0.999 * 2251799813685248.0;  // 2^51 less a margin for the rounding of the weights

template <int WORDS>
__device__ __forceinline__ fixed_t to_fixed(double w, double wyz) {
  const double t = fma(w, wyz, kMagic);
  if constexpr (WORDS == 1) {
    return (fixed_t)__double_as_longlong(t) - ((fixed_t)kMagicHi << 32);
  } else {
    const double r = fma(w, wyz, kMagic - t);
    const fixed_t l = (fixed_t)__double_as_longlong(fma(r, 4294967296.0, kMagic));
    const unsigned hi = (unsigned)__double_as_longlong(t) + (unsigned)(l >> 32) - kMagicHi;
    return ((fixed_t)hi << 32) | (unsigned)l;
  }
}

// The stencil times `value` (times the scale) into one quantity's block, (K + 1)^3 atomics.
template <int K, int WORDS, typename T>
__device__ __forceinline__ void stencil_add(fixed_t* blk, int E, const Axes<K, T>& s, T value, double scale) {
  double w[K + 1];
#pragma unroll
  for (int c = 0; c <= K; ++c) w[c] = (double)(s.wx[c] * value) * scale;
#pragma unroll
  for (int cz = 0; cz <= K; ++cz)
#pragma unroll
    for (int cy = 0; cy <= K; ++cy) {
      fixed_t* row = blk + s.l0 + (cz * E + cy) * E;
#pragma unroll
      for (int cx = 0; cx <= K; ++cx) atomicAdd(&row[cx], to_fixed<WORDS>(w[cx], s.wyz[cz * (K + 1) + cy]));
    }
}

// The particles [e0, e1) of a tile's list into its LDS block: J at the mid-point of the step, rho_old
// at its start and rho_new at its end.  On a collocated grid the components of J share one stencil.
template <int K, bool STAG, int WORDS, typename T>
__device__ __forceinline__ void deposit_run(fixed_t* lds, int E, int ncl, const PicArgs<T>& a, const DepPtrs<T>& p,
                                            int e0, int e1, double sj, double sr, int bx, int by, int bz) {
  const T ic2 = T(1) / (a.c * a.c);
  const T qv = a.q * a.inv_vol;
  for (int e = e0; e < e1; ++e) {
    const int i = p.list[e];
    const T u0 = p.u[0][i], u1 = p.u[1][i], u2 = p.u[2][i];
    const T x0 = p.xo[0][i], y0 = p.xo[1][i], z0 = p.xo[2][i];
    const T x1 = p.xn[0][i], y1 = p.xn[1][i], z1 = p.xn[2][i];
    const T ig = T(1) / sqrt(T(1) + (u0 * u0 + u1 * u1 + u2 * u2) * ic2);
    const T v[3] = {u0 * ig, u1 * ig, u2 * ig};
    // mid-point (unwrapped from the start position; stencil_axes() folds the periodic edge)
    T xm = x0 + T(0.5) * a.dt * v[0], ym = y0 + T(0.5) * a.dt * v[1], zm = z0 + T(0.5) * a.dt * v[2];
    xm -= a.lx * floor(xm / a.lx);
    ym -= a.ly * floor(ym / a.ly);
    zm -= a.lz * floor(zm / a.lz);
    Axes<K, T> g;
    if constexpr (!STAG) stencil_axes<K>(g, E, a, 0, 0, 0, xm, ym, zm, bx, by, bz);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if constexpr (STAG)  // half a cell up along its own axis
        stencil_axes<K>(g, E, a, k == 0, k == 1, k == 2, xm, ym, zm, bx, by, bz);
      stencil_add<K, WORDS>(lds + k * ncl, E, g, qv * v[k], sj);
    }
    // both charge densities live on the cell corners, staggered or not
    stencil_axes<K>(g, E, a, 0, 0, 0, x0, y0, z0, bx, by, bz);
    stencil_add<K, WORDS>(lds + 3 * ncl, E, g, qv, sr);
    stencil_axes<K>(g, E, a, 0, 0, 0, x1, y1, z1, bx, by, bz);
    stencil_add<K, WORDS>(lds + 4 * ncl, E, g, qv, sr);
  }
}

// One workgroup per D1 tile: its particles' J (mid-point), rho_old (start) and rho_new
// (end) into LDS over the tile and its guard cells, then the block either added into G1
// with global atomics (blocks == nullptr) or stored whole, tile by tile, into `blocks`
// ([tile][quantity][z][y][x], E^3 values per quantity) for k_gather_blocks.
template <typename T, int K, bool STAG>
__global__ void __launch_bounds__(kDepositThreads<K>) k_deposit_tiles(PicArgs<T> a, DepPtrs<T> p, T* __restrict__ blocks) {
  extern __shared__ double2 pic_smem[];
  fixed_t* lds = reinterpret_cast<fixed_t*>(pic_smem);
  constexpr int GL = Reach<K>::lo;
  const int E = a.tile + GL + Reach<K>::hi;
  const int ncl = E * E * E;
  const int tid = threadIdx.x;
  // merge walk: thread (row r0, column lx) of R = blockDim / E rows per round
  const int R = blockDim.x / E, r0 = tid / E, lx = tid - r0 * E;
  const int dy = R % E, dz = (R / E) % E, df = R / (E * E);
  for (unsigned next = blockIdx.x; next < (unsigned)a.ntiles; next += gridDim.x) {
    const int t = (int)next;
    const int tz = t / (a.tx * a.ty), rem = t - tz * a.tx * a.ty, ty = rem / a.tx, tx = rem - ty * a.tx;
    const int bx = tx * a.tile, by = ty * a.tile, bz = tz * a.tile;
    for (int i = tid; i < 5 * ncl; i += blockDim.x) lds[i] = 0;
    __syncthreads();
    // each thread takes a contiguous run of the tile's list, so the lanes of a wave work in
    // different cells: no two lanes add to one LDS word in the same instruction
    const int first = p.offset[t], count = p.offset[t + 1] - first;
    // fixed-point scales of J and rho: a particle adds at most |q| c / V (|v| < c) to a J
    // point and |q| / V to a rho point, so with count particles every sum stays below
    // count * bound * scale < 2^62.  Powers of two: scaling and unscaling are exact.
    const double bv = fabs((double)a.q) * (double)a.inv_vol * 1.0000001, bj = bv * (double)a.c;
    const double nmax = (double)max(count, 1);
    // (capped where the bound is tiny: then bound * 2^120 is below 2^62 anyway)
    const int ejc = min(61 - ilogb(fmax(bj * nmax, 1e-300)), 120), erc = min(61 - ilogb(fmax(bv * nmax, 1e-300)), 120);
    const int per = (count + (int)blockDim.x - 1) / (int)blockDim.x;
    const int e0 = first + min(count, tid * per), e1 = first + min(count, (tid + 1) * per);
    // one word where a single value stays below 2^51, which is from about 2050 particles on
    if (ldexp(bj, ejc) < kOneWord && ldexp(bv, erc) < kOneWord)
      deposit_run<K, STAG, 1>(lds, E, ncl, a, p, e0, e1, ldexp(1.0, ejc), ldexp(1.0, erc), bx, by, bz);
    else
      deposit_run<K, STAG, 2>(lds, E, ncl, a, p, e0, e1, ldexp(1.0, ejc - 32), ldexp(1.0, erc - 32), bx, by, bz);
    __syncthreads();
    if (blocks) {
      // the whole block, unscaled, in the tile's slot (consecutive threads, consecutive words)
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        const double sc = ldexp(1.0, -(f < 3 ? ejc : erc));
        T* dst = blocks + ((long long)t * 5 + f) * ncl;
        for (int i = tid; i < ncl; i += blockDim.x) dst[i] = (T)((double)(long long)lds[f * ncl + i] * sc);
      }
    } else if (r0 < R) {
      // the block (tile and guards) added into G1: guard cells are the neighbours' cells.
      // Rows (f, z, y) are walked with carries, so no element needs a division.
      auto wrap_near = [](int v, int n) {  // v in [-n, ...): one add or subtract except on tiny grids
        if (v < 0) v += n;
        if (v >= n) {
          v -= n;
          if (v >= n) v %= n;
        }
        return v;
      };
      const int gxi = wrap_near(bx - GL + lx, a.gx);
      int y = r0 % E, z = (r0 / E) % E, f = r0 / (E * E);
      while (f < 5) {
        const long long iv = (long long)lds[((f * E + z) * E + y) * E + lx];
        if (iv != 0) {
          const T v = (T)((double)iv * ldexp(1.0, -(f < 3 ? ejc : erc)));
          const int gyi = wrap_near(by - GL + y, a.gy), gzi = wrap_near(bz - GL + z, a.gz);
          unsafeAtomicAdd(&p.g[f][((long long)gzi * a.gy + gyi) * a.gx + gxi], v);
        }
        y += dy;
        if (y >= E) {
          y -= E;
          ++z;
        }
        z += dz;
        if (z >= E) {
          z -= E;
          ++f;
        }
        f += df;
      }
    }
    __syncthreads();
  }
}

// The blocks stored by k_deposit_tiles summed into G1: one workgroup per tile, one thread
// per cell of the tile (x fastest), so that a wave reads rows of several block rows at once.
// A cell lies in the block of its own tile and, within Reach<K>::hi cells of the tile's
// lower face or Reach<K>::lo cells of its upper face, in the block of the neighbour across
// it.  Requires tiles that divide the grid, at least two tiles per axis and guards no wider
// than a tile, so that along each axis a cell is reached by its own tile and at most one
// neighbour (with two tiles per axis both neighbours are the same tile, reached through one
// face or the other).  Every cell is written (no zeroing first), with a fixed order of the
// sums.  Each chiplet takes one range of tiles, so that neighbours along x find their common lines in
// one L2 (4.2 M cells, FP32: 0.206 -> 0.143 ms).
template <typename T, int K>
__global__ void __launch_bounds__(256) k_gather_blocks(PicArgs<T> a, DepPtrs<T> p, const T* __restrict__ blocks) {
  constexpr int GL = Reach<K>::lo, GH = Reach<K>::hi;
  const int T_ = a.tile, E = T_ + GL + GH, T2 = T_ * T_;
  const long long ncl = (long long)E * E * E;
  const int per = gridDim.x / kXcds, tile = blockIdx.x % kXcds * per + blockIdx.x / kXcds;
  if (tile >= a.ntiles) return;
  const int tz = tile / (a.tx * a.ty), ty = (tile - tz * a.tx * a.ty) / a.tx, tx = tile - (tz * a.ty + ty) * a.tx;
  // per axis: the tiles whose block covers local cell c, and the cell's index in each
  auto reach = [&](int c, int t, int nt, int* ts, int* ls) {
    ts[0] = t;
    ls[0] = c + GL;
    int m = 1;
    if (c < GH) {  // in the upper guard of the tile below
      ts[1] = t == 0 ? nt - 1 : t - 1;
      ls[1] = c + T_ + GL;
      m = 2;
    } else if (c >= T_ - GL) {  // in the lower guard of the tile above
      ts[1] = t == nt - 1 ? 0 : t + 1;
      ls[1] = c - T_ + GL;
      m = 2;
    }
    return m;
  };
  for (int q = threadIdx.x; q < T2 * T_; q += blockDim.x) {
    const int lz = q / T2, ly = (q - lz * T2) / T_, lx = q - lz * T2 - ly * T_;
    int tsx[2], lsx[2], tsy[2], lsy[2], tsz[2], lsz[2];
    const int mx = reach(lx, tx, a.tx, tsx, lsx), my = reach(ly, ty, a.ty, tsy, lsy),
              mz = reach(lz, tz, a.tz, tsz, lsz);
    T acc[5] = {0, 0, 0, 0, 0};
    for (int iz = 0; iz < mz; ++iz)
      for (int iy = 0; iy < my; ++iy) {
        const long long row = ((long long)tsz[iz] * a.ty + tsy[iy]) * a.tx;
        const int r = (lsz[iz] * E + lsy[iy]) * E;
        const T* b0 = blocks + (row + tsx[0]) * 5 * ncl + r + lsx[0];
        T v[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) v[f] = b0[f * ncl];
        if (mx == 2) {
          const T* b1 = blocks + (row + tsx[1]) * 5 * ncl + r + lsx[1];
          T w[5];
#pragma unroll
          for (int f = 0; f < 5; ++f) w[f] = b1[f * ncl];
#pragma unroll
          for (int f = 0; f < 5; ++f) v[f] += w[f];
        }
#pragma unroll
        for (int f = 0; f < 5; ++f) acc[f] += v[f];
      }
    const long long cell = ((long long)(tz * T_ + lz) * a.gy + (ty * T_ + ly)) * a.gx + (tx * T_ + lx);
#pragma unroll
    for (int f = 0; f < 5; ++f) p.g[f][cell] = acc[f];
  }
}

}  // namespace
}  // namespace psatd

using namespace psatd;

struct psatd_pic {
  psatd_pic_desc d{};
  int fp64 = 0;
  int tx = 0, ty = 0, tz = 0, ntiles = 0;
  int* count = nullptr;
  int* offset = nullptr;
  int* cursor = nullptr;
  int* list = nullptr;
  void* blocks = nullptr;  // per-tile deposit blocks (NULL: blocks merged with atomics)
  // E and B of every cell side by side, filled by each push that uses them (collocated grid; NULL:
  // pushes gather from the six arrays).  A push on another stream than the last one takes
  // them only once that one has finished, and gathers from the arrays otherwise; so does a
  // push under capture, whose replays nothing here could order.
  void* cells = nullptr;
  std::mutex mu;
  hipEvent_t cells_done = nullptr;
  hipStream_t cells_stream = nullptr;
  bool cells_used = false;

  bool claim_cells(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      return false;
    }
    if (!cells_used) return true;
    // (the same handle may be a new stream, whose predecessor still runs: ordered by the event)
    const hipError_t e = cells_stream == s ? hipStreamWaitEvent(s, cells_done, 0) : hipEventQuery(cells_done);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
  }
  int release_cells(hipStream_t s) {
    if (hipEventRecord(cells_done, s) != hipSuccess)
      return report_error(PSATD_EHIP, "psatd_pic_push: %s", hipGetErrorString(hipGetLastError()));
    cells_stream = s;
    cells_used = true;
    return PSATD_OK;
  }
};

namespace {

template <typename T>
PicArgs<T> pic_args(const psatd_pic* o, int n) {
  PicArgs<T> a{};
  const psatd_pic_desc& d = o->d;
  a.gx = d.gx;
  a.gy = d.gy;
  a.gz = d.gz;
  a.dx = T(d.dx);
  a.dy = T(d.dy);
  a.dz = T(d.dz);
  a.idx = T(1.0 / d.dx);
  a.idy = T(1.0 / d.dy);
  a.idz = T(1.0 / d.dz);
  a.lx = T(d.gx * d.dx);
  a.ly = T(d.gy * d.dy);
  a.lz = T(d.gz * d.dz);
  a.dt = T(d.dt);
  a.c = T(d.c);
  a.q = T(d.q);
  a.qm = T(d.q_over_m);
  a.inv_vol = T(1.0 / (d.dx * d.dy * d.dz));
  a.stag = (d.flags & PSATD_FLAG_STAGGERED) ? 1 : 0;
  a.tile = d.tile;
  a.tx = o->tx;
  a.ty = o->ty;
  a.tz = o->tz;
  a.ntiles = o->ntiles;
  a.n = n;
  return a;
}

// LDS of one deposit workgroup: five fixed-point quantities over the tile and its guard
// cells, for particle shapes of degree `shape`.
size_t pic_lds_bytes(int tile, int shape) {
  const size_t e = (size_t)tile + (shape == 1 ? Reach<1>::lo + Reach<1>::hi : Reach<2>::lo + Reach<2>::hi);
  return 5 * e * e * e * sizeof(fixed_t);
}

// Interleaving moves 12 values per cell and takes a launch: it is done where there is a particle
// for every kCellsPerParticle cells (one per cell: 0.12 -> 0.15 ms while in perfect order, 0.42
// -> 0.23 ms 22 steps later) and the arrays are larger than what an L2 holds anyway.
constexpr int kCellsPerParticle = 2;
constexpr long long kCellsBytes = 8 << 20;
long long ncell_of(const psatd_pic* o) { return (long long)o->d.gx * o->d.gy * o->d.gz; }

// degree of the particle shape of a descriptor (0 means linear)
int shape_of(const psatd_pic_desc& d) { return d.shape == 0 ? 1 : d.shape; }

unsigned blocks_for(long long n, int th) { return (unsigned)((n + th - 1) / th); }

template <typename T>
int pic_push(psatd_pic* o, void* const* g1, void* const* x, void* const* u, void* const* x_old, int n,
             hipStream_t s) {
  if (n == 0) return PSATD_OK;
  PushPtrs<T> p{};
  for (int k = 0; k < 6; ++k) p.f[k] = (const T*)g1[k];
  for (int k = 0; k < 3; ++k) {
    p.x[k] = (T*)x[k];
    p.u[k] = (T*)u[k];
    p.x_old[k] = (T*)x_old[k];
  }
  const PicArgs<T> a = pic_args<T>(o, n);
  const dim3 grid(blocks_for(n, kPicThreads)), block(kPicThreads);
  const int shape = shape_of(o->d);
  // Interleaved cells where there are enough particles to pay for the interleaving and no call
  // on another stream may still be reading them.
  std::unique_lock<std::mutex> lock(o->mu, std::defer_lock);
  if (o->cells && (long long)n * kCellsPerParticle >= ncell_of(o) &&
      6 * ncell_of(o) * (long long)sizeof(T) >= kCellsBytes) {
    lock.lock();
    if (o->claim_cells(s)) {
      Six<T> six{};
      for (int k = 0; k < 6; ++k) six.f[k] = p.f[k];
      const long long per = 16 / sizeof(T);
      hipLaunchKernelGGL(k_interleave<T>, dim3(blocks_for((ncell_of(o) + per - 1) / per, kPicThreads)),
                         dim3(kPicThreads), 0, s, six, (T*)o->cells, ncell_of(o));
      p.cells = (const T*)o->cells;
      switch (shape) {
        case 1: hipLaunchKernelGGL((k_pic_push<T, false, 1, true>), grid, block, 0, s, a, p); break;
        case 2: hipLaunchKernelGGL((k_pic_push<T, false, 2, true>), grid, block, 0, s, a, p); break;
        default: hipLaunchKernelGGL((k_pic_push<T, false, 3, true>), grid, block, 0, s, a, p); break;
      }
      return o->release_cells(s);
    }
    lock.unlock();
  }
  switch (shape * 2 + a.stag) {
    case 2: hipLaunchKernelGGL((k_pic_push<T, false, 1, false>), grid, block, 0, s, a, p); break;
    case 3: hipLaunchKernelGGL((k_pic_push<T, true, 1, false>), grid, block, 0, s, a, p); break;
    case 4: hipLaunchKernelGGL((k_pic_push<T, false, 2, false>), grid, block, 0, s, a, p); break;
    case 5: hipLaunchKernelGGL((k_pic_push<T, true, 2, false>), grid, block, 0, s, a, p); break;
    case 6: hipLaunchKernelGGL((k_pic_push<T, false, 3, false>), grid, block, 0, s, a, p); break;
    default: hipLaunchKernelGGL((k_pic_push<T, true, 3, false>), grid, block, 0, s, a, p); break;
  }
  return PSATD_OK;
}

template <typename T, int K, bool STAG>
void launch_tiles(const PicArgs<T>& a, const DepPtrs<T>& p, T* blocks, size_t lds, hipStream_t s) {
  if (lds > 64 * 1024)
    (void)hipFuncSetAttribute((const void*)k_deposit_tiles<T, K, STAG>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
  // one tile per workgroup (the loop inside covers grids beyond the cap)
  const unsigned grid = (unsigned)std::min(a.ntiles, 1 << 20);
  hipLaunchKernelGGL((k_deposit_tiles<T, K, STAG>), dim3(grid), dim3(kDepositThreads<K>), lds, s, a, p, blocks);
}
template <typename T, int K>
void launch_deposit(const PicArgs<T>& a, const DepPtrs<T>& p, T* blocks, size_t lds, hipStream_t s) {
  if (a.stag)
    launch_tiles<T, K, true>(a, p, blocks, lds, s);
  else
    launch_tiles<T, K, false>(a, p, blocks, lds, s);
  if (blocks) hipLaunchKernelGGL((k_gather_blocks<T, K>), dim3((a.ntiles + kXcds - 1) / kXcds * kXcds), dim3(256), 0, s, a, p,
                                 (const T*)blocks);
}

template <typename T>
int pic_deposit(psatd_pic* o, void* const* g1, const void* const* x_old, const void* const* x, const void* const* u,
                int n, hipStream_t s) {
  DepPtrs<T> p{};
  for (int k = 0; k < 3; ++k) {
    p.xo[k] = (const T*)x_old[k];
    p.xn[k] = (const T*)x[k];
    p.u[k] = (const T*)u[k];
  }
  for (int f = 0; f < 5; ++f) p.g[f] = (T*)g1[6 + f];
  p.count = o->count;
  p.offset = o->offset;
  p.cursor = o->cursor;
  p.list = o->list;
  const PicArgs<T> a = pic_args<T>(o, n);
  const long long ncell = (long long)o->d.gx * o->d.gy * o->d.gz;
  T* blocks = (T*)o->blocks;
  // with per-tile blocks every cell is written by the gather; otherwise the atomics add
  // into zeroed arrays
  if (!blocks || n == 0) hipLaunchKernelGGL(k_zero_fields<T>, dim3(blocks_for(ncell, 256)), dim3(256), 0, s, p, ncell);
  if (n == 0) return PSATD_OK;
  hipLaunchKernelGGL(k_zero_int, dim3(blocks_for(o->ntiles, 256)), dim3(256), 0, s, o->count, o->ntiles);
  // two workgroups per CU, each with at least two particles per thread
  const int chunk = std::max(2 * kTileThreads, (int)blocks_for(n, 512));
  hipLaunchKernelGGL(k_tile_count<T>, dim3(blocks_for(n, chunk)), dim3(kTileThreads), 0, s, a, p, chunk);
  hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(1024), 0, s, o->count, o->offset, o->cursor, o->ntiles);
  if (n >= kListMany)
    hipLaunchKernelGGL((k_tile_list<T, kListRun>), dim3(blocks_for(n, kTileThreads * kListRun)), dim3(kTileThreads), 0,
                       s, a, p);
  else
    hipLaunchKernelGGL((k_tile_list<T, kListRunFew>), dim3(blocks_for(n, kTileThreads * kListRunFew)),
                       dim3(kTileThreads), 0, s, a, p);
  const int shape = shape_of(o->d);
  const size_t lds = pic_lds_bytes(o->d.tile, shape);
  if (shape == 1)
    launch_deposit<T, 1>(a, p, blocks, lds, s);
  else if (shape == 2)
    launch_deposit<T, 2>(a, p, blocks, lds, s);
  else
    launch_deposit<T, 3>(a, p, blocks, lds, s);
  return PSATD_OK;
}

}  // namespace

extern "C" {

int psatd_pic_create(const psatd_pic_desc* d, psatd_pic** out) {
  if (!out) return report_error(PSATD_EINVAL, "out is NULL");
  *out = nullptr;
  if (!d) return report_error(PSATD_EINVAL, "descriptor is NULL");
  if (d->gx <= 0 || d->gy <= 0 || d->gz <= 0) return report_error(PSATD_EINVAL, "grid sizes must be positive");
  if (!(d->dx > 0) || !(d->dy > 0) || !(d->dz > 0) || !(d->dt > 0) || !(d->c > 0))
    return report_error(PSATD_EINVAL, "cell sizes, dt and c must be > 0");
  if (d->precision != PSATD_FP32 && d->precision != PSATD_FP64) return report_error(PSATD_EINVAL, "unknown precision");
  if (d->flags & ~PSATD_FLAG_STAGGERED) return report_error(PSATD_EINVAL, "unknown flags 0x%x", d->flags);
  if (d->tile < 1 || d->tile > kTileMax) return report_error(PSATD_EINVAL, "tile must be in [1, %d]", kTileMax);
  if (d->max_particles < 0) return report_error(PSATD_EINVAL, "max_particles must be >= 0");
  if (d->shape < 0 || d->shape > kMaxShape)
    return report_error(PSATD_EINVAL, "shape must be 0 (linear), 1, 2 or %d", kMaxShape);
  // a particle moves less than c dt per step; the margin covers the rounding of positions
  if (d->c * d->dt > kMaxCourant * std::min(d->dx, std::min(d->dy, d->dz)))
    return report_error(PSATD_EUNSUPPORTED,
                        "c dt = %g exceeds %g of the smallest cell size: a particle could leave its tile's guard "
                        "cells", d->c * d->dt, kMaxCourant);
  if ((double)d->gx * d->gy * d->gz >= 2147483647.0) return report_error(PSATD_EUNSUPPORTED, "grid too large");
  {
    int dev = 0, lim = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&lim, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || lim <= 0) {
      (void)hipGetLastError();
      lim = 64 * 1024;
    }
    const size_t need = pic_lds_bytes(d->tile, shape_of(*d));
    if (need > (size_t)lim)
      return report_error(PSATD_EUNSUPPORTED, "tile %d with shape degree %d needs %zu bytes of LDS per workgroup "
                          "(limit %d)", d->tile, shape_of(*d), need, lim);
  }
  psatd_pic* o = new psatd_pic;
  o->d = *d;
  o->fp64 = d->precision == PSATD_FP64;
  o->tx = (d->gx + d->tile - 1) / d->tile;
  o->ty = (d->gy + d->tile - 1) / d->tile;
  o->tz = (d->gz + d->tile - 1) / d->tile;
  o->ntiles = o->tx * o->ty * o->tz;
  const size_t bytes[4] = {(size_t)o->ntiles * 4, (size_t)(o->ntiles + 1) * 4, (size_t)o->ntiles * 4,
                           (size_t)std::max(1, d->max_particles) * 4};
  int** ptrs[4] = {&o->count, &o->offset, &o->cursor, &o->list};
  for (int k = 0; k < 4; ++k)
    if (hipMalloc((void**)ptrs[k], bytes[k]) != hipSuccess) {
      (void)hipGetLastError();
      for (int j = 0; j < k; ++j) (void)hipFree(*ptrs[j]);
      delete o;
      return report_error(PSATD_ENOMEM, "particle workspace allocation failed");
    }
  // Per-tile blocks for the atomic-free merge (see k_gather_blocks) for shapes of degree 2
  // and 3, where the tiling allows it: their blocks hold 13^3 cells per 8^3 tile, and
  // storing and gathering them beats adding them with global atomics.  For degree 1 (11^3
  // cells per 8^3 tile) the atomics are faster.  Without the memory the blocks are merged
  // with atomics.
  {
    const int shape = shape_of(*d), T = d->tile;
    const int reach = shape == 1 ? Reach<1>::lo + Reach<1>::hi : Reach<2>::lo + Reach<2>::hi;
    const bool tiled = shape >= 2 && d->gx % T == 0 && d->gy % T == 0 && d->gz % T == 0 && o->tx >= 2 &&
                       o->ty >= 2 && o->tz >= 2 && reach <= T;
    if (tiled) {
      const size_t e = (size_t)T + reach;
      const size_t b = (size_t)o->ntiles * 5 * e * e * e * (o->fp64 ? sizeof(double) : sizeof(float));
      if (hipMalloc(&o->blocks, b) != hipSuccess) {
        (void)hipGetLastError();
        o->blocks = nullptr;
      }
    }
  }
  const long long cell_bytes = 6 * ncell_of(o) * (long long)(o->fp64 ? sizeof(double) : sizeof(float));
  if (!(d->flags & PSATD_FLAG_STAGGERED) && (long long)d->max_particles * kCellsPerParticle >= ncell_of(o) &&
      cell_bytes >= kCellsBytes) {
    if (hipMalloc(&o->cells, (size_t)cell_bytes) != hipSuccess ||
        hipEventCreateWithFlags(&o->cells_done, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      if (o->cells) (void)hipFree(o->cells);
      o->cells = nullptr;
      o->cells_done = nullptr;
    }
  }
  *out = o;
  return PSATD_OK;
}

void psatd_pic_destroy(psatd_pic* o) {
  if (!o) return;
  for (int* q : {o->count, o->offset, o->cursor, o->list})
    if (q) (void)hipFree(q);
  if (o->blocks) (void)hipFree(o->blocks);
  if (o->cells) (void)hipFree(o->cells);
  if (o->cells_done) (void)hipEventDestroy(o->cells_done);
  delete o;
}

int psatd_pic_push(psatd_pic* o, void* const* g1, void* const* x, void* const* u, void* const* x_old, int n,
                   void* stream) {
  if (!o || !g1 || !x || !u || !x_old) return report_error(PSATD_EINVAL, "NULL argument");
  if (n < 0 || n > o->d.max_particles) return report_error(PSATD_EINVAL, "n = %d outside [0, max_particles]", n);
  if (n == 0) return PSATD_OK;
  for (int k = 0; k < 6; ++k)
    if (!g1[k]) return report_error(PSATD_EINVAL, "field pointer %d is NULL", k);
  for (int k = 0; k < 3; ++k)
    if (!x[k] || !u[k] || !x_old[k]) return report_error(PSATD_EINVAL, "particle array %d is NULL", k);
  const int rc = o->fp64 ? pic_push<double>(o, g1, x, u, x_old, n, (hipStream_t)stream)
                         : pic_push<float>(o, g1, x, u, x_old, n, (hipStream_t)stream);
  if (rc) return rc;
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PSATD_OK : report_error(PSATD_EHIP, "psatd_pic_push: %s", hipGetErrorString(e));
}

int psatd_pic_deposit(psatd_pic* o, void* const* g1, const void* const* x_old, const void* const* x,
                      const void* const* u, int n, void* stream) {
  if (!o || !g1 || !x_old || !x || !u) return report_error(PSATD_EINVAL, "NULL argument");
  if (n < 0 || n > o->d.max_particles) return report_error(PSATD_EINVAL, "n = %d outside [0, max_particles]", n);
  for (int k = 6; k < 11; ++k)
    if (!g1[k]) return report_error(PSATD_EINVAL, "field pointer %d is NULL", k);
  for (int k = 0; n > 0 && k < 3; ++k)
    if (!x[k] || !u[k] || !x_old[k]) return report_error(PSATD_EINVAL, "particle array %d is NULL", k);
  const int rc = o->fp64 ? pic_deposit<double>(o, g1, x_old, x, u, n, (hipStream_t)stream)
                         : pic_deposit<float>(o, g1, x_old, x, u, n, (hipStream_t)stream);
  if (rc) return rc;
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PSATD_OK : report_error(PSATD_EHIP, "psatd_pic_deposit: %s", hipGetErrorString(e));
}

}  // extern "C"
