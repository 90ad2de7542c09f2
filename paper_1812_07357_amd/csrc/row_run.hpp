// K + 1 consecutive values of a field row in as few multi-word loads as cover them exactly (gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace psatd {

// V values as a vector aligned like one of them.
template <int V, typename T>
struct RowVec {
  typedef T type __attribute__((ext_vector_type(V), aligned(alignof(T))));
};
template <typename T>
struct RowVec<1, T> {
  typedef T type;
};

template <int K, typename T>
struct RowRun {
  T v[K + 1];
};

// One load, except for three doubles: the compiler reads a vector of three of them as four, and
// the fourth of the last row of an array is past its end (three floats are one 12-byte load).
template <int K, typename T>
__device__ __forceinline__ RowRun<K, T> load_run(const T* p) {
  constexpr int N = K + 1, V = N == 3 && sizeof(T) == 8 ? 2 : N;
  typedef typename RowVec<V, T>::type head_t;
  const head_t x = *reinterpret_cast<const head_t*>(p);
  RowRun<K, T> r;
#pragma unroll
  for (int c = 0; c < V; ++c) r.v[c] = x[c];
  if constexpr (V < N) r.v[V] = p[V];
  return r;
}

}  // namespace psatd
