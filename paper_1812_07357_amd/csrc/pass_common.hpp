// What the pass kernels share (gfx950): parameter sources, the k-space push, persistent launches.
#pragma once

#include "internal.hpp"

namespace psatd {

namespace {

constexpr uint32_t kOOB = 0x3fffffffu;  // element index past the end of every array

template <typename T>
__device__ inline cx<T>* lds_base() {
  extern __shared__ double2 psatd_smem[];
  return reinterpret_cast<cx<T>*>(psatd_smem);
}

// x mod d for 0 <= x < 2^31
__device__ __forceinline__ int fmod_i(int x, const FastDiv& f) { return x - fdiv(x, f) * (int)f.d; }
// x mod d for 0 <= x < 2 d
__device__ __forceinline__ int wrap_once(int x, int d) { return x - (x >= d ? d : 0); }
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// ------------------------------------------------------------------ parameter sources
// A single box's parameters are the kernel's only argument, so they sit at
// offset 0 of the kernel-argument segment.  They are read from there through a
// pointer: binding a reference to the by-value argument makes the compiler keep
// a private (scratch) copy of the whole block, because the transform schedules
// inside it are indexed with run-time stage numbers.
template <typename P>
struct SingleSrc {
  const P* p;
  __device__ __forceinline__ SingleSrc()
      : p((const P*)__builtin_amdgcn_kernarg_segment_ptr()) {}
  __device__ __forceinline__ int ntiles() const { return p->ntiles; }
  __device__ __forceinline__ const P& box(int tile, int& local) const {
    local = tile;
    return *p;
  }
};

// The descriptors of a batch are constant while its kernels run: they are read through the
// constant address space, so that box parameters arrive by scalar loads and stay uniform
// (through plain global loads every buffer resource was per lane, a loop around each access).
template <typename P>
__device__ __forceinline__ const P* as_constant(const P* p) {
  return (const P*)(const __attribute__((address_space(4))) P*)(uintptr_t)p;
}

template <typename P>
struct BatchSrc {
  BatchArgs<P> a;
  __device__ __forceinline__ int ntiles() const { return a.total; }
  // box b with starts[b] <= tile < starts[b + 1] (binary search on uniform values)
  __device__ __forceinline__ const P& box(int tile, int& local) const {
    const int* starts = as_constant(a.starts);
    int lo = 0, hi = a.nbox;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (starts[mid] <= tile)
        lo = mid;
      else
        hi = mid;
    }
    local = tile - starts[lo];
    return *as_constant(a.descs + lo);
  }
};

// Cache policy of the x passes' stores: streamed (non-temporal) in FP32, where it made the
// step about 3 % faster; FP64 was slower with it and keeps the default.
template <typename T>
constexpr int kXStore = sizeof(T) == 4 ? kStream : kKeep;

// ------------------------------------------------------------------ k-space push
// The push at one k-space point: column col, z index kz, its field-0 value at LDS
// slot s and field f at s + f * fs; k_x, k_y of the column given.
// Staggered grid: the same update with the complex symbols kappa = k_s exp(i k d / 2)
// (kp, from nodes to the half points above) and their conjugates (back down):
//   E' = C E + i c^2 S1 (kappa^* x B) - (S1/eps0) J + i (c^2/eps0) kappa (X3 rho_old - X2 rho_new)
//   B' = C B - i S1 (kappa x E) + i (X1/eps0) (kappa x J)
// (E and J sit half a cell up along their own axis, B along the other two, rho on
// the nodes; C, S1, X1..X3 are functions of |k_s|).

// What the push of one point needs besides the fields: the five coefficients (requested before
// the transforms, they come from memory) and the wavenumbers of its column and kz (staggered
// grid: kappa; small tables, read when the point is pushed).
template <typename T>
struct PushPoint {
  T cc[5];
  cx<T> kx, ky, kz;  // collocated grid: real
  // point e (kz fastest) of the columns from col0 on; past npt: zeros from out-of-range loads
  __device__ __forceinline__ void load(const ZPushParams<T>& p, int col0, int e, int npt) {
    const uint32_t idx = e < npt ? (uint32_t)(col0 * p.NZ + e) : kOOB;
#pragma unroll
    for (int k = 0; k < 5; ++k) cc[k] = gm<T>::ld(make_rsrc(p.coef + (i64)k * p.npts, p.coef_bytes), idx);
  }
  // its wavenumbers: column `col`, index kzi
  __device__ __forceinline__ void wavenumbers(const ZPushParams<T>& p, int col, int kzi) {
    const int kxi = fdiv(col, p.fd_NY), kyi = col - kxi * p.NY;
    if (p.stag) {
      kx = p.kxc[kxi];
      ky = p.kyc[kyi];
      kz = p.kzc[kzi];
    } else {
      kx.re = p.kx[kxi];
      ky.re = p.ky[kyi];
      kz.re = p.kz[kzi];
    }
  }
};

template <typename T>
__device__ __forceinline__ void push_point_staggered(const ZPushParams<T>& p, cx<T>* lds, int fs, int s,
                                                     const PushPoint<T>& q) {
  const T c2 = p.c2, ie = p.inv_eps0;
  const T C = q.cc[0], S1 = q.cc[1], X1 = q.cc[2], X2 = q.cc[3], X3 = q.cc[4];
  const cx<T> kx = q.kx, ky = q.ky, kz_ = q.kz;
  const cx<T> kxm = cconj(kx), kym = cconj(ky), kzm = cconj(kz_);
  const cx<T> ex = lds[0 * fs + s], ey = lds[1 * fs + s], ez = lds[2 * fs + s];
  const cx<T> bx = lds[3 * fs + s], by = lds[4 * fs + s], bz = lds[5 * fs + s];
  const cx<T> jx = lds[6 * fs + s], jy = lds[7 * fs + s], jz = lds[8 * fs + s];
  const cx<T> ro = lds[9 * fs + s], rn = lds[10 * fs + s];
  // kappa^* x B, kappa x E, kappa x J
  const cx<T> kbx = csub(cmul(kym, bz), cmul(kzm, by));
  const cx<T> kby = csub(cmul(kzm, bx), cmul(kxm, bz));
  const cx<T> kbz = csub(cmul(kxm, by), cmul(kym, bx));
  const cx<T> kex = csub(cmul(ky, ez), cmul(kz_, ey));
  const cx<T> key = csub(cmul(kz_, ex), cmul(kx, ez));
  const cx<T> kez = csub(cmul(kx, ey), cmul(ky, ex));
  const cx<T> kjx = csub(cmul(ky, jz), cmul(kz_, jy));
  const cx<T> kjy = csub(cmul(kz_, jx), cmul(kx, jz));
  const cx<T> kjz = csub(cmul(kx, jy), cmul(ky, jx));
  const cx<T> rr = csub(cscale(ro, X3), cscale(rn, X2));
  const T a = c2 * S1, g = c2 * ie, sj = S1 * ie, xj = X1 * ie;
  const cx<T> ux = cadd(cscale(kbx, a), cscale(cmul(kx, rr), g));
  const cx<T> uy = cadd(cscale(kby, a), cscale(cmul(ky, rr), g));
  const cx<T> uz = cadd(cscale(kbz, a), cscale(cmul(kz_, rr), g));
  lds[0 * fs + s] = {C * ex.re - sj * jx.re - ux.im, C * ex.im - sj * jx.im + ux.re};
  lds[1 * fs + s] = {C * ey.re - sj * jy.re - uy.im, C * ey.im - sj * jy.im + uy.re};
  lds[2 * fs + s] = {C * ez.re - sj * jz.re - uz.im, C * ez.im - sj * jz.im + uz.re};
  const cx<T> wx = csub(cscale(kjx, xj), cscale(kex, S1));
  const cx<T> wy = csub(cscale(kjy, xj), cscale(key, S1));
  const cx<T> wz = csub(cscale(kjz, xj), cscale(kez, S1));
  lds[3 * fs + s] = {C * bx.re - wx.im, C * bx.im + wx.re};
  lds[4 * fs + s] = {C * by.re - wy.im, C * by.im + wy.re};
  lds[5 * fs + s] = {C * bz.re - wz.im, C * bz.im + wz.re};
}

template <typename T>
__device__ __forceinline__ void push_point_c(const ZPushParams<T>& p, cx<T>* lds, int fs, int s, const PushPoint<T>& q) {
  const T c2 = p.c2, ie = p.inv_eps0;
  if (p.stag) {
    push_point_staggered(p, lds, fs, s, q);
    return;
  }
  const T kx = q.kx.re, ky = q.ky.re, kzz = q.kz.re;
  const T C = q.cc[0], S1 = q.cc[1], X1 = q.cc[2], X2 = q.cc[3], X3 = q.cc[4];
  const cx<T> ex = lds[0 * fs + s], ey = lds[1 * fs + s], ez = lds[2 * fs + s];
  const cx<T> bx = lds[3 * fs + s], by = lds[4 * fs + s], bz = lds[5 * fs + s];
  const cx<T> jx = lds[6 * fs + s], jy = lds[7 * fs + s], jz = lds[8 * fs + s];
  const cx<T> ro = lds[9 * fs + s], rn = lds[10 * fs + s];
  // K x B, K x E, K x J (K real)
  const cx<T> kbx = csub(cscale(bz, ky), cscale(by, kzz));
  const cx<T> kby = csub(cscale(bx, kzz), cscale(bz, kx));
  const cx<T> kbz = csub(cscale(by, kx), cscale(bx, ky));
  const cx<T> kex = csub(cscale(ez, ky), cscale(ey, kzz));
  const cx<T> key = csub(cscale(ex, kzz), cscale(ez, kx));
  const cx<T> kez = csub(cscale(ey, kx), cscale(ex, ky));
  const cx<T> kjx = csub(cscale(jz, ky), cscale(jy, kzz));
  const cx<T> kjy = csub(cscale(jx, kzz), cscale(jz, kx));
  const cx<T> kjz = csub(cscale(jy, kx), cscale(jx, ky));
  const cx<T> rr = csub(cscale(ro, X3), cscale(rn, X2));
  const T a = c2 * S1;   // multiplies K x B
  const T g = c2 * ie;   // multiplies K r
  const T sj = S1 * ie;  // multiplies J
  const T xj = X1 * ie;  // multiplies K x J
  // E' = C E - sj J + i (a K x B + g K r)
  const cx<T> ux = cadd(cscale(kbx, a), cscale(rr, g * kx));
  const cx<T> uy = cadd(cscale(kby, a), cscale(rr, g * ky));
  const cx<T> uz = cadd(cscale(kbz, a), cscale(rr, g * kzz));
  lds[0 * fs + s] = {C * ex.re - sj * jx.re - ux.im, C * ex.im - sj * jx.im + ux.re};
  lds[1 * fs + s] = {C * ey.re - sj * jy.re - uy.im, C * ey.im - sj * jy.im + uy.re};
  lds[2 * fs + s] = {C * ez.re - sj * jz.re - uz.im, C * ez.im - sj * jz.im + uz.re};
  // B' = C B + i (xj K x J - S1 K x E)
  const cx<T> wx = csub(cscale(kjx, xj), cscale(kex, S1));
  const cx<T> wy = csub(cscale(kjy, xj), cscale(key, S1));
  const cx<T> wz = csub(cscale(kjz, xj), cscale(kez, S1));
  lds[3 * fs + s] = {C * bx.re - wx.im, C * bx.im + wx.re};
  lds[4 * fs + s] = {C * by.re - wy.im, C * by.im + wy.re};
  lds[5 * fs + s] = {C * bz.re - wz.im, C * bz.im + wz.re};
}

// Two-step PML (Sec. 2.6): the twelve split parts of E and B (component a split into set
// A, driven by the derivative along axis a+1, and set B, along a+2) advance over the step
// by the integral of their own right-hand side along the exact evolution of the full
// fields, with the sources constant.  Set B of E_a gains -i c^2 K_{a+2} IB_{a+1}, set B of
// B_a gains +i K_{a+2} IE_{a+1}, where
//   IB = S1 B_T + dt B_L - i X1 (K x E) + i (dt X2/eps0) (K x J),
//   IE = S1 E_T + dt E_L + i c^2 X1 (K x B) - (X1/eps0) J_T - (dt^2/(2 eps0)) J_L
// are the integrals of B(t) and E(t) over the step (T, L: parts transverse and parallel
// to K); set A takes the rest of the increment of the ordinary push, so the two sets
// always add up to it.  Writes the increments (scaled by 1/N like the tables) of set A
// to slots 0..5 and of set B to slots 6..11 (in the split-part order E_xz E_yx E_zy
// B_xz B_yx B_zy); the sources in slots 6..10 are read first.  Collocated grid.
template <typename T>
__device__ __forceinline__ void push_point_pml(const ZPushParams<T>& p, cx<T>* lds, int fs, int s,
                                               const PushPoint<T>& q) {
  const T c2 = p.c2, ie = p.inv_eps0, invn = p.inv_n, dt = p.dt;
  const T K[3] = {q.kx.re, q.ky.re, q.kz.re};
  const T C = q.cc[0], S1 = q.cc[1], X1 = q.cc[2], X2 = q.cc[3], X3 = q.cc[4];
  cx<T> E[3], B[3], J[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    E[a] = lds[a * fs + s];
    B[a] = lds[(3 + a) * fs + s];
    J[a] = lds[(6 + a) * fs + s];
  }
  const cx<T> ro = lds[9 * fs + s], rn = lds[10 * fs + s];
  const T k2 = K[0] * K[0] + K[1] * K[1] + K[2] * K[2];
  const T ik2 = k2 > T(0) ? T(1) / k2 : T(0);
  auto dot = [&](const cx<T>* v) {
    return cadd(cadd(cscale(v[0], K[0]), cscale(v[1], K[1])), cscale(v[2], K[2]));
  };
  auto cross = [&](const cx<T>* v, int a) {  // (K x v)_a
    const int b = a == 2 ? 0 : a + 1, c = a == 0 ? 2 : a - 1;
    return csub(cscale(v[c], K[b]), cscale(v[b], K[c]));
  };
  const cx<T> kE = cscale(dot(E), ik2), kB = cscale(dot(B), ik2), kJ = cscale(dot(J), ik2);
  const cx<T> rr = csub(cscale(ro, X3), cscale(rn, X2));
  cx<T> IB[3], IE[3], dE[3], dB[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cx<T> kxe = cross(E, a), kxb = cross(B, a), kxj = cross(J, a);
    const cx<T> EL = cscale(kE, K[a]), BL = cscale(kB, K[a]), JL = cscale(kJ, K[a]);
    // IB_a = S1 (B - B_L) + dt/N B_L + (X1 K x E + dt X2/eps0 K x J) * (-i, +i)
    const cx<T> ib_r = cadd(cscale(csub(B[a], BL), S1), cscale(BL, dt * invn));
    const cx<T> ib_i = csub(cscale(kxj, dt * X2 * ie), cscale(kxe, X1));  // times i
    IB[a] = {ib_r.re - ib_i.im, ib_r.im + ib_i.re};
    const cx<T> ie_r = csub(cadd(cscale(csub(E[a], EL), S1), cscale(EL, dt * invn)),
                            cadd(cscale(csub(J[a], JL), X1 * ie), cscale(JL, T(0.5) * dt * dt * invn * ie)));
    const cx<T> ie_i = cscale(kxb, c2 * X1);  // times i
    IE[a] = {ie_r.re - ie_i.im, ie_r.im + ie_i.re};
    // ordinary push (tables scaled by 1/N) minus E/N: the whole increment
    const cx<T> ux = cadd(cscale(kxb, c2 * S1), cscale(rr, c2 * ie * K[a]));
    dE[a] = {C * E[a].re - S1 * ie * J[a].re - ux.im - invn * E[a].re,
             C * E[a].im - S1 * ie * J[a].im + ux.re - invn * E[a].im};
    const cx<T> w = csub(cscale(kxj, X1 * ie), cscale(kxe, S1));
    dB[a] = {C * B[a].re - w.im - invn * B[a].re, C * B[a].im + w.re - invn * B[a].im};
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int b = a == 2 ? 0 : a + 1, c = a == 0 ? 2 : a - 1;  // a+1, a+2
    // set B: -i c^2 K_c IB_b and +i K_c IE_b
    const cx<T> eb = {c2 * K[c] * IB[b].im, -c2 * K[c] * IB[b].re};
    const cx<T> bb = {-K[c] * IE[b].im, K[c] * IE[b].re};
    lds[a * fs + s] = csub(dE[a], eb);
    lds[(3 + a) * fs + s] = csub(dB[a], bb);
    lds[(6 + a) * fs + s] = eb;
    lds[(9 + a) * fs + s] = bb;
  }
}

// ------------------------------------------------------------------ launches
template <typename T>
size_t cx_bytes() {
  return sizeof(cx<T>);
}

int num_cus() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      n = v;
    else
      n = 256;
  }
  return n;
}

// Persistent grid: as many blocks as can be resident at once (capped by the tile count).
// Opts in to more than 64 KB of dynamic LDS when needed (the plan checked the device limit).
template <typename K>
unsigned persistent_grid(K kernel, int threads, size_t lds, int ntiles) {
  if (lds > 64 * 1024)
    (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds) != hipSuccess || per_cu < 1) {
    (void)hipGetLastError();
    per_cu = 1;
  }
  const long long g = (long long)per_cu * num_cus();
  return (unsigned)(g < ntiles ? g : ntiles);
}

template <typename K, typename A>
void launch_persistent(K kernel, const A& arg, int threads, size_t lds, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return;
  const unsigned g = persistent_grid(kernel, threads, lds, ntiles);
  hipLaunchKernelGGL(kernel, dim3(g), dim3(threads), lds, s, arg);
}

}  // namespace

}  // namespace psatd
