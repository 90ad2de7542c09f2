// Line transforms in two register stages around one LDS exchange (gfx950).
//
// A transform length m = RA * RB (RA >= RB, both with a compiled DFT) is split as
//   stage A, butterfly j < RB of a line:  Y[j][k] = sum_t w_RA^(t k) x[j + RB t],
//   stage B, column k < RA:               X[k + RA t'] = sum_j w_RB^(j t') w_m^(j k) Y[j][k].
// Every butterfly is one thread's: its points go from memory into registers, through a
// compile-time DFT and into a padded LDS row (A), or from an LDS column through the
// twiddles and the DFT to the output (B).  One transform is one LDS round trip and one
// barrier, whatever the length; the radices are chosen at run time by a switch over the
// compiled DFTs, so every length with such a pair runs the same kernel, alone or in a batch.
//
// Lengths n with a prime factor above 17 use the chirp-z form (see LineFFT): a cyclic
// convolution of length m >= 2n - 1 with the chirp filter.  Stage B leaves frequency
// k + RA t' of the forward transform in the thread that needs it for the backward one, so
// the filter product and the backward stage B run in the same registers: a chirp-z
// line is stage A, exchange, stage B . filter . inverse stage B, exchange, inverse stage A
// (two exchanges; as separate Stockham transforms and products it takes eleven).
#pragma once

#include "fft_lds.hpp"

#include <utility>

namespace psatd {

// Run-time description of one axis on the pair kernels.
template <typename T>
struct PairFFT {
  int n = 0, m = 0;     // line length, transform length
  int ra = 0, rb = 0;   // m = ra * rb, ra >= rb; 0: the axis runs on the Stockham kernels
  int pb = 0, ld = 0;   // LDS slots per column and per line (pair_pitch, pair_line)
  FastDiv fa, fb;       // division by ra, rb
  const Tw<T>* tw = nullptr;     // w_m^(j k) at [k * pair_tw_pitch(rb) + j - 1], 1 <= j < rb
  const Tw<T>* chirp = nullptr;  // m entries: exp(-i pi j^2 / n) below n, zero from n on
  const Tw<T>* filt = nullptr;   // m entries
};

// Stage A leaves Y[j][k] of a line at LDS slot k * pitch + j: its lanes of consecutive j write
// consecutive slots, and stage B reads its column k from consecutive slots, 16 bytes (one
// FP64 or two FP32 values) at a time.  A 16-byte access serves 8 lanes per cycle, so the lanes'
// columns have to lie an odd number of 16 bytes apart.  (With FP32 columns an odd number of
// 8-byte slots apart, conflict-free for single values, the paired reads of the x and z
// passes took two cycles for one.)
template <typename T>
__host__ __device__ constexpr int pair_pitch(int rb) {
  return sizeof(T) == 8 ? rb | 1 : ((rb + 1) & ~3) + 2 >= rb ? ((rb + 1) & ~3) + 2 : rb;
}
// The twiddles of a column are consecutive 16-byte entries, columns an odd number apart.
__host__ __device__ constexpr int pair_tw_pitch(int rb) { return (rb - 1) | 1; }

// Compiled radices, by kernel class: 0 direct pairs up to 24 points (a butterfly and its
// temporaries fit 128 FP32 registers), 1 direct pairs with a radix of 25 to 36 points (lengths
// up to 1296), 2 and 3 chirp-z lines.  Chirp-z has classes of its own because its stage B,
// with two DFTs and the filter between them, would set the registers of every length.
template <int... R>
using radix_list = std::integer_sequence<int, R...>;
template <int CLASS>
struct radices;
template <>
struct radices<0> {
  using a = radix_list<1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 20, 21, 22, 24>;
  using b = radix_list<1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 20, 21, 22, 24>;
};
template <>
struct radices<1> {
  using a = radix_list<25, 26, 27, 28, 30, 32, 33, 34, 36>;
  using b = radix_list<4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 20, 21, 22, 24, 25, 26, 27, 28, 30, 32, 33, 34, 36>;
};
template <>
struct radices<2> {
  using a = radix_list<8, 10, 12, 16, 18, 20, 24>;
  using b = radix_list<2, 4, 6, 8, 10, 12, 16, 18, 20, 24>;
};
template <>
struct radices<3> {
  using a = radix_list<32>;
  using b = radix_list<20, 24, 32>;
};
constexpr bool chirp_class(int cls) { return cls >= 2; }
constexpr int kPairClasses = 4;

// f(integral_constant<R>) for the radix of the list that equals r (uniform over the block).
template <typename F, int... R>
__host__ __device__ __forceinline__ void with_radix(int r, radix_list<R...>, F&& f) {
  (void)((r == R ? (f(std::integral_constant<int, R>{}), true) : false) || ...);
}
template <int... R>
constexpr int max_of(radix_list<R...>) {
  int m = 0;
  ((m = R > m ? R : m), ...);
  return m;
}
template <int... R>
constexpr bool in_list(int r, radix_list<R...>) {
  return ((r == R) || ...);
}

#define PSATD_INLINE __attribute__((always_inline))

// x, opaque to the optimiser: multiples of a run-time stride would otherwise be computed
// ahead of the tile loop for every radix of the switch, far more than the scalar registers
// hold (their spills, through vector registers, made the y pass 25 % slower).
__device__ __forceinline__ int opaque(int x) {
  int r = __builtin_amdgcn_readfirstlane(x);
  asm volatile("" : "+s"(r));
  return r;
}

// The same for a per-lane value: the lanes' LDS addresses do not change from tile to tile, and
// would be kept in registers for every radix.
__device__ __forceinline__ int opaque_lane(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Copies an axis's twiddles to LDS (every thread of the block; the caller synchronises).
template <typename T>
__device__ __forceinline__ void pair_stage_twiddles(Tw<T>* dst, const PairFFT<T>& P) {
  for (int i = threadIdx.x; i < P.ra * pair_tw_pitch(P.rb); i += blockDim.x) dst[i] = P.tw[i];
}

// v * w^(S j k) of column k for the points j >= 1 (k = 0: factors of exactly 1).
template <int R, int S, typename T>
__device__ __forceinline__ void pair_twiddle(cx<T>* v, const Tw<T>* tw, int k) {
  const Tw<T>* w = tw + k * pair_tw_pitch(R);
#pragma unroll
  for (int t = 1; t < R; ++t) v[t] = twmul<S>(v[t], w[t - 1]);
}

// A column's R values, in 16-byte reads.
template <int R>
__device__ __forceinline__ void pair_take(cx<float>* v, const cx<float>* y) {
  const float4* q = reinterpret_cast<const float4*>(y);
#pragma unroll
  for (int t = 0; t + 1 < R; t += 2) {
    const float4 w = q[t / 2];
    v[t] = {w.x, w.y};
    v[t + 1] = {w.z, w.w};
  }
  if constexpr (R % 2 == 1) v[R - 1] = y[R - 1];
}
template <int R>
__device__ __forceinline__ void pair_take(cx<double>* v, const cx<double>* y) {
#pragma unroll
  for (int t = 0; t < R; ++t) v[t] = y[t];
}

// A butterfly's outputs into its LDS slots: point k of butterfly j at k * pitch + j.
template <int R, typename T>
__device__ __forceinline__ void pair_put(cx<T>* y, int pb, const cx<T>* v) {
#pragma unroll
  for (int t = 0; t < R; ++t) {
    *y = v[t];
    y += pb;
  }
}

// Stage A of butterfly (line, j): load(radix constant, t) gives point j + RB t of the line.  LDSIN: the points
// come from the natural-order LDS line itself (a barrier between the reads and the writes).  AHEAD: from that
// many points on all loads are issued before the DFT begins (0: where the compiler places them).
template <int CLASS, int S, bool LDSIN, int AHEAD = 0, typename T, typename Load>
__device__ __forceinline__ void pair_stage_a(cx<T>* lds, const PairFFT<T>& P, int line, int j, bool active,
                                             Load&& load) {
  with_radix(P.ra, typename radices<CLASS>::a{}, [&](auto rc) PSATD_INLINE {
    constexpr int R = decltype(rc)::value;
    cx<T> v[R];
    if (active) {
#pragma unroll
      for (int t = 0; t < R; ++t) v[t] = load(rc, t);
      if constexpr (AHEAD > 0 && R >= AHEAD) __builtin_amdgcn_sched_barrier(0);
      dft<R, S, T>::run(v);
    }
    if constexpr (LDSIN) __syncthreads();
    if (active) pair_put<R>(lds + line * P.ld + j, opaque(P.pb), v);
  });
}

// Stage B of column (line, k): store(t, value) receives point k + RA t.  SYNC: a barrier
// before the stores (they go back into the LDS lines).
template <int CLASS, int S, bool SYNC, typename T, typename Store>
__device__ __forceinline__ void pair_stage_b(const cx<T>* lds, const Tw<T>* tw, const PairFFT<T>& P, int line, int k,
                                             bool active, Store&& store) {
  with_radix(P.rb, typename radices<CLASS>::b{}, [&](auto rc) PSATD_INLINE {
    constexpr int R = decltype(rc)::value;
    cx<T> v[R];
    if (active) {
      pair_take<R>(v, lds + line * P.ld + k * pair_pitch<T>(R));
      pair_twiddle<R, S>(v, tw, k);
      dft<R, S, T>::run(v);
    }
    if constexpr (SYNC) __syncthreads();
    if (active) {
#pragma unroll
      for (int t = 0; t < R; ++t) store(t, v[t]);
    }
  });
}

// Chirp-z: point j + RB t of the line times the chirp, stage A.  With n <= (m + 1) / 2 and RA even
// the points of t >= RA / 2 lie past the line: they are zeros of the code, and the DFT is
// cut accordingly.  load(radix constant, t) is asked for t < RA / 2 only; from n on it may give any finite value (the chirp is zero).
template <int CLASS, int S, bool LDSIN, typename T, typename Load>
__device__ __forceinline__ void chirp_stage_a(cx<T>* lds, const PairFFT<T>& P, int line, int j, bool active,
                                              Load&& load) {
  with_radix(P.ra, typename radices<CLASS>::a{}, [&](auto rc) PSATD_INLINE {
    constexpr int R = decltype(rc)::value;
    static_assert(R % 2 == 0, "chirp-z stage A radices are even");
    cx<T> v[R];
    if (active) {
      const Tw<T>* c = P.chirp + j;
      const int rb = opaque(P.rb);
#pragma unroll
      for (int t = 0; t < R / 2; ++t) v[t] = load(rc, t);
#pragma unroll
      for (int t = 0; t < R / 2; ++t) {
        v[t] = twmul<S>(v[t], c[rb * t]);
        v[R / 2 + t] = {T(0), T(0)};
      }
      dft<R, -1, T>::run(v);
    }
    if constexpr (LDSIN) __syncthreads();
    if (active) pair_put<R>(lds + line * P.ld + j, opaque(P.pb), v);
  });
}

// Chirp-z: forward stage B, filter, backward stage B of column (line, k), in place.
template <int CLASS, int S, typename T>
__device__ __forceinline__ void chirp_stage_b(cx<T>* lds, const Tw<T>* tw, const PairFFT<T>& P, int line, int k,
                                              bool active) {
  with_radix(P.rb, typename radices<CLASS>::b{}, [&](auto rc) PSATD_INLINE {
    constexpr int R = decltype(rc)::value;
    if (active) {
      cx<T> v[R];
      cx<T>* y = lds + line * P.ld + k * pair_pitch<T>(R);
      pair_take<R>(v, y);
      pair_twiddle<R, -1>(v, tw, k);
      dft<R, -1, T>::run(v);
      const Tw<T>* f = P.filt + k;
      const int ra = opaque(P.ra);
#pragma unroll
      for (int t = 0; t < R; ++t) v[t] = twmul<S>(v[t], f[ra * t]);
      dft<R, 1, T>::run(v);
      pair_twiddle<R, 1>(v, tw, k);
#pragma unroll
      for (int t = 0; t < R; ++t) y[t] = v[t];
    }
  });
}

// Chirp-z: backward stage A of butterfly (line, j); store(t, value) receives point
// j + RB t of the transform, t < RA / 2 (zero from n on).  SYNC: a barrier before the stores.
template <int CLASS, int S, bool SYNC, typename T, typename Store>
__device__ __forceinline__ void chirp_stage_c(const cx<T>* lds, const PairFFT<T>& P, int line, int j, bool active,
                                              Store&& store) {
  with_radix(P.ra, typename radices<CLASS>::a{}, [&](auto rc) PSATD_INLINE {
    constexpr int R = decltype(rc)::value;
    cx<T> v[R];
    if (active) {
      const cx<T>* y = lds + line * P.ld + j;
      const int pb = opaque(P.pb);
#pragma unroll
      for (int t = 0; t < R; ++t) {
        v[t] = *y;
        y += pb;
      }
      dft<R, 1, T>::run(v);
      const Tw<T>* c = P.chirp + j;
      const int rb = opaque(P.rb);
#pragma unroll
      for (int t = 0; t < R / 2; ++t) v[t] = twmul<S>(v[t], c[rb * t]);
    }
    if constexpr (SYNC) __syncthreads();
    if (active) {
#pragma unroll
      for (int t = 0; t < R / 2; ++t) store(t, v[t]);
    }
  });
}

}  // namespace psatd
