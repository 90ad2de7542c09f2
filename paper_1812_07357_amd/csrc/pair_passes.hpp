// The five passes of one PSATD step on the pair kernels (gfx950): see passes.hip for what
// each pass computes and pair_fft.hpp for the line transform.  Every axis whose length
// has a radix pair runs here, in single boxes and in batches; the Stockham kernels of
// passes.hip keep the lengths without one.
//
// A tile is a few lines; every stage gives one butterfly to one thread, so a block has
// lines * RA threads (rounded to whole wavefronts) and no stage loops.  Blocks are
// persistent: the twiddles (and P1's column table) are copied to LDS once per box, then
// the block walks its tiles, each waiting only on its own loads while the other blocks of
// the CU transform theirs.

#pragma once

#include "internal.hpp"
#include "pass_common.hpp"

namespace psatd {
namespace {

// Tiles are taken in runs of kRun consecutive ones per block: a batch block changes box (and
// copies that box's tables) less often than with single tiles.
template <bool BATCH>
struct TileWalk {
  static constexpr int kRun = BATCH ? 4 : 1;
  int i = 0;
  __device__ __forceinline__ int tile() const {
    return ((i / kRun) * (int)gridDim.x + (int)blockIdx.x) * kRun + i % kRun;
  }
  // false: past the end (a run may start inside the range and end outside it)
  __device__ __forceinline__ bool in_range(int ntiles) const {
    return ((i / kRun) * (int)gridDim.x + (int)blockIdx.x) * kRun < ntiles;
  }
};

template <typename T>
__device__ __forceinline__ Tw<T>* tables_after(cx<T>* lds, int lines, const PairFFT<T>& P) {
  return reinterpret_cast<Tw<T>*>(lds + lines * P.ld + (lines * P.ld & 1));
}

// ------------------------------------------------------------------ P1
// A block's tile waits for its own loads, and its LDS leaves nine wavefronts per CU to cover them.  Left to
// itself the compiler takes a load when the DFT needs it.  With all loads first P1 of 576x320x320 takes 0.868
// instead of 0.925 ms (kernels compiled for 24 * 24 alone: 0.844), lines of 180 to 1056 points up to 12 % less;
// those up to 160 up to 5 % more (101 registers: four wavefronts per SIMD, not five).  Held to five
// wavefronts (two registers spilled) the box takes 0.888 ms.  The same costs the large radices in FP64 up to
// 36 %, the x inverse 5 %, the y passes in FP64 4 %.
template <typename T, int CLASS>
constexpr int kAhead = sizeof(T) == 4 ? 14 : 0;
// PML: a full field is the sum of its two split parts, added as they are loaded (the sources have
// one array: an empty buffer reads as zero).
template <int CLASS, bool BATCH, bool PML, typename T, typename Src>
__device__ __forceinline__ void pair_xfwd_body(const Src& S) {
  cx<T>* lds = lds_base<T>();
  const int nth = blockDim.x;
  const XFwdParams<T>* last = nullptr;
  for (TileWalk<BATCH> w; w.in_range(S.ntiles()); ++w.i) {
    const int tid = opaque_lane(threadIdx.x);
    const int tile = w.tile();
    if (tile >= S.ntiles()) continue;
    int lt;
    const XFwdParams<T>& p = S.box(tile, lt);
    const PairFFT<T>& P = p.pair;
    const int nc = p.pnl, N = P.n, RA = opaque(P.ra), RB = opaque(P.rb);
    Tw<T>* tw = tables_after(lds, nc, P);
    int* xoff = reinterpret_cast<int*>(tw + RA * pair_tw_pitch(RB));  // source column of each box x (G1 wrap applied)
    if (last != &p) {
      pair_stage_twiddles(tw, P);
      for (int i = tid; i < N; i += nth) xoff[i] = p.gather ? fmod_i(p.x0 + i, p.fd_GX) : i;
      last = &p;
      __syncthreads();
    }
    const int NY = p.NY, NXH = p.NXH;
    const int rowlen = p.gather ? p.GX : N;
    const int q = fdiv(lt, p.fd_ytiles);
    const int ybase = (lt - q * p.ytiles) * (2 * nc);
    const int f = fdiv(q, p.fd_NZ);
    const int z = q - f * p.NZ;
    const int zrow = p.gather ? fmod_i(p.z0 + z, p.fd_GZ) * p.GY : z * NY;
    // stage A: rows a = ybase + 2c, b = a + 1 of line c as one complex line, straight from the source
    {
      const int c = fdiv(tid, P.fb), j = tid - c * RB;
      const int ya = ybase + 2 * c;
      // Lines past the last row are left out (nothing of them is stored).  The last row of an odd NY is its own
      // partner: a row of zeros would take a select after each load (P1 of 576x320x320 FP32 0.918 -> 0.930
      // ms, of 128-point lines 25.6 -> 28.1 us), and kOOB with a column added wraps back into the array.
      const bool active = c < nc && ya < NY;
      int ra = ya, rb = min(ya + 1, NY - 1);
      if (p.gather) {
        ra = fmod_i(p.y0 + ra, p.fd_GY);
        rb = fmod_i(p.y0 + rb, p.fd_GY);
      }
      const uint32_t oa = (uint32_t)((zrow + ra) * rowlen), ob = (uint32_t)((zrow + rb) * rowlen);
      const rsrc_t src = make_rsrc(p.src[f], p.src_bytes);
      rsrc_t add = src;
      if constexpr (PML) add = make_rsrc(p.add[f < 6 ? f : 0], f < 6 ? p.src_bytes : 0u);
      auto load = [&](uint32_t i) PSATD_INLINE {
        if constexpr (PML)
          return gm<T>::ld(src, i) + gm<T>::ld(add, i);
        else
          return gm<T>::ld(src, i);
      };
      const int* xo = xoff + j;
      const int cb = fdiv(tid, P.fa), kb = tid - cb * RA;
      if constexpr (chirp_class(CLASS)) {
        chirp_stage_a<CLASS, -1, false>(lds, P, c, j, active, [&](auto, int t) PSATD_INLINE {
          const bool in = j + RB * t < N;
          const uint32_t xs = in ? (uint32_t)xo[RB * t] : 0u;
          return cx<T>{load(in ? oa + xs : kOOB), load(in ? ob + xs : kOOB)};
        });
        __syncthreads();
        chirp_stage_b<CLASS, -1>(lds, tw, P, cb, kb, cb < nc);
        __syncthreads();
        chirp_stage_c<CLASS, -1, true>(lds, P, c, j, active, [&](int t, cx<T> v) PSATD_INLINE {
          lds[c * P.ld + j + RB * t] = v;
        });
      } else {
        pair_stage_a<CLASS, -1, false, kAhead<T, CLASS>>(lds, P, c, j, active, [&](auto, int t) PSATD_INLINE {
          const uint32_t xs = (uint32_t)xo[RB * t];
          return cx<T>{load(oa + xs), load(ob + xs)};
        });
        __syncthreads();
        pair_stage_b<CLASS, -1, true>(lds, tw, P, cb, kb, cb < nc, [&](int t, cx<T> v) PSATD_INLINE {
          lds[cb * P.ld + kb + RA * t] = v;
        });
      }
    }
    __syncthreads();
    // split each complex line into the half spectra of its two real rows, written as pairs
    const rsrc_t dst = make_rsrc(p.dst + (i64)f * p.fsA, p.dst_bytes);
    const int ny_t = min(2 * nc, NY - ybase);
    const int sh = p.pnl_sh;
    for (int e = tid; e < NXH * nc; e += nth) {
      const int kx = e >> sh, c = e & (nc - 1);
      const cx<T> za = lds[c * P.ld + kx];
      const cx<T> zb = cconj(lds[c * P.ld + (kx == 0 ? 0 : N - kx)]);
      const cx<T> sum = cadd(za, zb), dif = csub(za, zb);
      const cx<T> va = cscale(sum, T(0.5));
      const cx<T> vb = {T(0.5) * dif.im, T(-0.5) * dif.re};
      const int t = 2 * c;
      const uint32_t o = (uint32_t)((z * NXH + kx) * NY + ybase + t);
      if (t + 1 < ny_t)
        gm<T>::template stc2<kXStore<T>>(dst, o, va, vb);
      else if (t < ny_t)
        gm<T>::template stc<kXStore<T>>(dst, o, va);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ P2 / P4
// P2 (S_ = -1) reads lines with contiguous positions and writes consecutive lines
// contiguously; P4 (S_ = +1) the reverse.  Lanes walk the contiguous direction of each side.
template <int CLASS, bool BATCH, int S_, typename T, typename Src>
__device__ __forceinline__ void pair_ypass_body(const Src& S) {
  cx<T>* lds = lds_base<T>();
  const YPassParams<T>* last = nullptr;
  for (TileWalk<BATCH> w; w.in_range(S.ntiles()); ++w.i) {
    const int tid = opaque_lane(threadIdx.x);
    const int tile = w.tile();
    if (tile >= S.ntiles()) continue;
    int lt;
    const YPassParams<T>& p = S.box(tile, lt);
    const PairFFT<T>& P = p.pair;
    const int NL = p.pnl, sh = p.pnl_sh, RA = opaque(P.ra), RB = opaque(P.rb);
    Tw<T>* tw = tables_after(lds, NL, P);
    if (last != &p) {
      pair_stage_twiddles(tw, P);
      last = &p;
      __syncthreads();
    }
    const int q = fdiv(lt, p.fd_utiles);
    const int ut = lt - q * p.utiles;
    const int f = fdiv(q, p.fd_nouter);
    const int o = q - f * p.nouter;
    const int u0 = p.u_lo + ut * NL;
    const int nlt = min(NL, p.u_hi - u0);
    const rsrc_t in = make_rsrc(p.in + (i64)f * p.fs_in + (i64)o * p.ob_in, p.in_bytes);
    const rsrc_t out = make_rsrc(p.out + (i64)f * p.fs_out + (i64)o * p.ob_out, p.out_bytes);
    // stage A mapping: along the line where positions are contiguous, across lines otherwise
    int line, j;
    if (S_ < 0) {
      line = fdiv(tid, P.fb);
      j = tid - line * RB;
    } else {
      line = tid & (NL - 1);
      j = tid >> sh;
    }
    const bool active = S_ < 0 ? line < NL : j < RB;
    const uint32_t ibase =
        active && line < nlt ? (uint32_t)(o * p.os_in + (u0 + line) * p.ls_in + j * p.ps_in) : kOOB;
    const uint32_t istep = (uint32_t)opaque(RB * p.ps_in * (int)sizeof(cx<T>));  // bytes between a butterfly's points
    if constexpr (chirp_class(CLASS)) {
      chirp_stage_a<CLASS, S_, false>(lds, P, line, j, active, [&](auto, int t) PSATD_INLINE {
        return gm<T>::ldc_s(in, j + RB * t < P.n ? ibase : kOOB, (uint32_t)t * istep);
      });
      __syncthreads();
      const int lb = fdiv(tid, P.fa), kb = tid - lb * RA;
      chirp_stage_b<CLASS, S_>(lds, tw, P, lb, kb, lb < NL);
      __syncthreads();
      // backward stage A and the stores: lanes along the contiguous direction of the output
      int lc, jc;
      if (S_ > 0) {
        lc = fdiv(tid, P.fb);
        jc = tid - lc * RB;
      } else {
        lc = tid & (NL - 1);
        jc = tid >> sh;
      }
      const bool ac = S_ > 0 ? lc < NL : jc < RB;
      const bool ok = ac && lc < nlt;
      const uint32_t obase = (uint32_t)(o * p.os_out + (u0 + lc) * p.ls_out + jc * p.ps_out);
      const uint32_t ostep = (uint32_t)opaque(RB * p.ps_out * (int)sizeof(cx<T>));
      chirp_stage_c<CLASS, S_, false>(lds, P, lc, jc, ac, [&](int t, cx<T> v) PSATD_INLINE {
        const int pos = jc + RB * t;
        gm<T>::stc_if(out, ok && pos >= p.p_lo && pos < p.p_hi, obase, (uint32_t)t * ostep, v);
      });
    } else {
      pair_stage_a<CLASS, S_, false>(lds, P, line, j, active, [&](auto, int t) PSATD_INLINE {
        return gm<T>::ldc_s(in, ibase, (uint32_t)t * istep);
      });
      __syncthreads();
      int lb, kb;
      if (S_ > 0) {
        lb = fdiv(tid, P.fa);
        kb = tid - lb * RA;
      } else {
        lb = tid & (NL - 1);
        kb = tid >> sh;
      }
      const bool ab = S_ > 0 ? lb < NL : kb < RA;
      const bool ok = ab && lb < nlt;
      const uint32_t obase = (uint32_t)(o * p.os_out + (u0 + lb) * p.ls_out + kb * p.ps_out);
      const uint32_t ostep = (uint32_t)opaque(RA * p.ps_out * (int)sizeof(cx<T>));
      pair_stage_b<CLASS, S_, false>(lds, tw, P, lb, kb, ab, [&](int t, cx<T> v) PSATD_INLINE {
        const int pos = kb + RA * t;
        gm<T>::stc_if(out, ok && pos >= p.p_lo && pos < p.p_hi, obase, (uint32_t)t * ostep, v);
      });
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ P3
// A tile is pnl consecutive (kx, ky) columns, contiguous in layout B ([kx][ky][field][z]):
// line l of the tile is field l % 11 of column l / 11.  The forward results are left in
// LDS in natural order for the push; the lines of E and B (PML: all twelve) then go back.
template <int CLASS, bool BATCH, bool PML, typename T, typename Src>
__device__ __forceinline__ void pair_zpush_body(const Src& S) {
  constexpr int F = PML ? 12 : 11, kOut = PML ? 12 : 6;
  constexpr int NPRE = 2;  // rounds of push coefficients requested before the transforms
  cx<T>* lds = lds_base<T>();
  const int nth = blockDim.x;
  const ZPushParams<T>* last = nullptr;
  for (TileWalk<BATCH> w; w.in_range(S.ntiles()); ++w.i) {
    const int tid = opaque_lane(threadIdx.x);
    const int tile = w.tile();
    if (tile >= S.ntiles()) continue;
    int lt;
    const ZPushParams<T>& p = S.box(tile, lt);
    const PairFFT<T>& P = p.pair;
    const int ncol = p.pnl, N = P.n, RA = opaque(P.ra), RB = opaque(P.rb);
    Tw<T>* tw = tables_after(lds, F * ncol, P);
    if (last != &p) {
      pair_stage_twiddles(tw, P);
      last = &p;
      __syncthreads();
    }
    const int col0 = lt * ncol;
    const int nct = min(ncol, p.NXH * p.NY - col0);
    const int npt = nct * N;
    const rsrc_t col = make_rsrc(p.b + (i64)col0 * F * N, (uint32_t)(nct * F * N * (int)sizeof(cx<T>)));
    // forward: line (c, f) of 11 per column
    const int la = fdiv(tid, P.fb), ja = tid - la * RB, ca = la / 11, lla = ca * F + la - ca * 11;
    const int lb = fdiv(tid, P.fa), kb = tid - lb * RA, cb = lb / 11, llb = cb * F + lb - cb * 11;
    const uint32_t ibase = ca < nct ? (uint32_t)(lla * N + ja) : kOOB;
    const uint32_t istep = (uint32_t)opaque(RB * (int)sizeof(cx<T>));
    auto point = [&](auto, int t) PSATD_INLINE {
      return gm<T>::ldc_s(col, chirp_class(CLASS) && ja + RB * t >= N ? kOOB : ibase, (uint32_t)t * istep);
    };
    if constexpr (chirp_class(CLASS))
      chirp_stage_a<CLASS, -1, false>(lds, P, lla, ja, ca < nct, point);
    else
      pair_stage_a<CLASS, -1, false>(lds, P, lla, ja, ca < nct, point);
    PushPoint<T> pt[NPRE];
#pragma unroll
    for (int u = 0; u < NPRE; ++u) pt[u].load(p, col0, u * nth + tid, npt);
    __syncthreads();
    if constexpr (chirp_class(CLASS)) {
      chirp_stage_b<CLASS, -1>(lds, tw, P, llb, kb, cb < nct);
      __syncthreads();
      chirp_stage_c<CLASS, -1, true>(lds, P, lla, ja, ca < nct, [&](int t, cx<T> v) PSATD_INLINE {
        lds[lla * P.ld + ja + RB * t] = v;
      });
    } else {
      pair_stage_b<CLASS, -1, true>(lds, tw, P, llb, kb, cb < nct, [&](int t, cx<T> v) PSATD_INLINE {
        lds[llb * P.ld + kb + RA * t] = v;
      });
    }
    __syncthreads();
    // push, point by point
    auto push = [&](int e, PushPoint<T>& q) PSATD_INLINE {
      const int c = fdiv(e, p.fd_NZ), kz = e - c * N;
      q.wavenumbers(p, col0 + c, kz);
      if constexpr (PML)
        push_point_pml(p, lds, P.ld, c * F * P.ld + kz, q);
      else
        push_point_c(p, lds, P.ld, c * F * P.ld + kz, q);
    };
#pragma unroll
    for (int u = 0; u < NPRE; ++u)
      if (u * nth + tid < npt) push(u * nth + tid, pt[u]);
    for (int e = NPRE * nth + tid; e < npt; e += nth) {
      PushPoint<T> q;
      q.load(p, col0, e, npt);
      push(e, q);
    }
    __syncthreads();
    // back: the first kOut lines of every column
    {
      const int l = fdiv(tid, P.fb), j = tid - l * RB;
      const int c = l / kOut, ll = c * F + l - c * kOut;
      const bool active = c < nct;
      const int lo = fdiv(tid, P.fa), ko = tid - lo * RA;
      const int co = lo / kOut, llo = co * F + lo - co * kOut;
      const cx<T>* x = lds + ll * P.ld + j;
      if constexpr (chirp_class(CLASS)) {
        chirp_stage_a<CLASS, 1, true>(lds, P, ll, j, active, [&](auto, int t) PSATD_INLINE {
          const cx<T> v = x[RB * t];
          return j + RB * t < N ? v : cx<T>{T(0), T(0)};
        });
        __syncthreads();
        chirp_stage_b<CLASS, 1>(lds, tw, P, llo, ko, co < nct);
        __syncthreads();
        const uint32_t base = (uint32_t)(ll * N + j), step = (uint32_t)opaque(RB * (int)sizeof(cx<T>));
        chirp_stage_c<CLASS, 1, false>(lds, P, ll, j, active, [&](int t, cx<T> v) PSATD_INLINE {
          const int z = j + RB * t;
          gm<T>::stc_if(col, z >= p.z_lo && z < p.z_hi, base, (uint32_t)t * step, v);
        });
      } else {
        pair_stage_a<CLASS, 1, true>(lds, P, ll, j, active, [&](auto, int t) PSATD_INLINE { return x[RB * t]; });
        __syncthreads();
        const uint32_t base = (uint32_t)(llo * N + ko), step = (uint32_t)opaque(RA * (int)sizeof(cx<T>));
        pair_stage_b<CLASS, 1, false>(lds, tw, P, llo, ko, co < nct, [&](int t, cx<T> v) PSATD_INLINE {
          const int z = ko + RA * t;
          gm<T>::stc_if(col, z >= p.z_lo && z < p.z_hi, base, (uint32_t)t * step, v);
        });
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ P5
// Stage A rebuilds the full line Z = A + i B from the half spectra of rows 2c, 2c + 1 as it
// loads: point i is X + i Y of bin i up to N/2 and conj X + i conj Y of bin N - i above
// (each bin is read twice, the second time from the caches, which costs less than the LDS
// round trip and the barrier of a rebuilt line).
// PML: the increment of one split set goes straight into its parts, damped (kPmlRows values of each row
// in flight: a read per store would leave the stores waiting for one read each).
constexpr int kPmlRows = 4;
template <int CLASS, bool BATCH, bool PML, typename T, typename Src>
__device__ __forceinline__ void pair_xinv_body(const Src& S) {
  cx<T>* lds = lds_base<T>();
  const int nth = blockDim.x;
  const XInvParams<T>* last = nullptr;
  for (TileWalk<BATCH> w; w.in_range(S.ntiles()); ++w.i) {
    const int tid = opaque_lane(threadIdx.x);
    const int tile = w.tile();
    if (tile >= S.ntiles()) continue;
    int lt;
    const XInvParams<T>& p = S.box(tile, lt);
    const PairFFT<T>& P = p.pair;
    const int nc = p.pnl, sh = p.pnl_sh, N = P.n, RA = opaque(P.ra), RB = opaque(P.rb);
    Tw<T>* tw = tables_after(lds, nc, P);
    if (last != &p) {
      pair_stage_twiddles(tw, P);
      last = &p;
      __syncthreads();
    }
    const int NY = p.NY, NXH = p.NXH;
    const int q = fdiv(lt, p.fd_ytiles);
    const int ybase = p.y_lo + (lt - q * p.ytiles) * (2 * nc);
    const int f = fdiv(q, p.fd_nz);
    const int zs = q - f * p.nzs;  // plane of the interior
    const int z = p.zfirst + zs;
    {
      // lanes across the lines: the rows of a bin are contiguous
      const int c = tid & (nc - 1), j = tid >> sh;
      const bool active = j < RB;
      const int ya = ybase + 2 * c;
      const rsrc_t src = make_rsrc(p.src + (i64)f * p.npts, p.src_bytes);
      const bool hasa = ya < p.y_hi, hasb = ya + 1 < p.y_hi;
      // Without a mask the compiler takes a load when its point is needed: fewer registers (FP32 150 -> 104,
      // 223 -> 149 for the large radices) and more wavefronts, P5 of 288 points 23.9 -> 22.0 us, of 600 points
      // 46 -> 38.  The large radices in FP64 have one wavefront per SIMD either way and want their loads in flight
      // together, which the mask brings about (1056 points: 200 us, without it 288).
      constexpr bool kMasked = sizeof(T) == 8 && CLASS == 1;
      const uint32_t base = (uint32_t)(zs * NXH * NY + ya);
      auto load = [&](auto, int t) PSATD_INLINE {
        // Chirp-z points past the line read bin 0 of their own rows (the chirp is zero there); lines past
        // the interior read whatever follows, and nothing of them is stored.
        const int i = j + RB * t;
        const bool up = 2 * i > N;
        const int kx = up ? (chirp_class(CLASS) ? max(N - i, 0) : N - i) : i;
        cx<T> x, y;
        if constexpr (kMasked)
          gm<T>::ldc2(src, hasa ? base + __umul24((uint32_t)kx, (uint32_t)NY) : kOOB, x, y);
        else
          gm<T>::ldc2(src, base + __umul24((uint32_t)kx, (uint32_t)NY), x, y);
        if (!hasb) y = {T(0), T(0)};  // the row past an odd interior
        // +1, -1 for the conjugate, 0 where the bin is its own conjugate (imaginary part dropped)
        const T s = (i == 0 || 2 * i == N) ? T(0) : (up ? T(-1) : T(1));
        return cx<T>{x.re - s * y.im, y.re + s * x.im};
      };
      const int cb = fdiv(tid, P.fa), kb = tid - cb * RA;
      if constexpr (chirp_class(CLASS)) {
        chirp_stage_a<CLASS, 1, false>(lds, P, c, j, active, load);
        __syncthreads();
        chirp_stage_b<CLASS, 1>(lds, tw, P, cb, kb, cb < nc);
        __syncthreads();
        const int cc = fdiv(tid, P.fb), jc = tid - cc * RB;
        chirp_stage_c<CLASS, 1, true>(lds, P, cc, jc, cc < nc, [&](int t, cx<T> v) PSATD_INLINE {
          lds[cc * P.ld + jc + RB * t] = v;
        });
      } else {
        pair_stage_a<CLASS, 1, false>(lds, P, c, j, active, load);
        __syncthreads();
        pair_stage_b<CLASS, 1, true>(lds, tw, P, cb, kb, cb < nc, [&](int t, cx<T> v) PSATD_INLINE {
          lds[cb * P.ld + kb + RA * t] = v;
        });
      }
    }
    __syncthreads();
    // the two real rows of each line (box, or interior of G1), written along x so that
    // a wave's stores cover whole rows
    if constexpr (PML) {
      const rsrc_t dst = make_rsrc(p.dst[f], p.dst_bytes);
      const int f3 = f < 3 ? f : f - 3, axis = f3 + p.pml < 3 ? f3 + p.pml : f3 + p.pml - 3;
      const T* dm = p.damp[axis];
      for (int e0 = tid; e0 < nc * N; e0 += kPmlRows * nth) {
        uint32_t ia[kPmlRows], ib[kPmlRows];
        cx<T> val[kPmlRows], part[kPmlRows], damp[kPmlRows];
#pragma unroll
        for (int u = 0; u < kPmlRows; ++u) {
          const int e = min(e0 + u * nth, nc * N - 1), c = fdiv(e, p.fd_nx), n = e - c * N;
          const bool in = e0 + u * nth < nc * N;
          const int ya = ybase + 2 * c;
          ia[u] = in && ya < NY ? (uint32_t)((z * NY + ya) * N + n) : kOOB;
          ib[u] = in && ya + 1 < NY ? (uint32_t)((z * NY + ya + 1) * N + n) : kOOB;
          part[u] = {gm<T>::ld(dst, ia[u]), gm<T>::ld(dst, ib[u])};
          damp[u] = {dm[axis == 0 ? n : axis == 1 ? min(ya, NY - 1) : z],
                     dm[axis == 0 ? n : axis == 1 ? min(ya + 1, NY - 1) : z]};
          val[u] = lds[c * P.ld + n];
        }
#pragma unroll
        for (int u = 0; u < kPmlRows; ++u) {
          gm<T>::template st<kXStore<T>>(dst, ia[u], (part[u].re + val[u].re) * damp[u].re);
          gm<T>::template st<kXStore<T>>(dst, ib[u], (part[u].im + val[u].im) * damp[u].im);
        }
      }
    } else {
      const rsrc_t dst = make_rsrc(p.dst[f], p.dst_bytes);
      const int zrow = p.scatter ? fmod_i(p.oz + z - p.gz, p.fd_GZ) * p.GY : z * NY;
      const int rowlen = p.scatter ? p.GX : N;
      const int x_lo = p.scatter ? p.gx : 0, nx = p.scatter ? p.nx : N;
      for (int e = tid; e < nc * nx; e += nth) {
        const int c = fdiv(e, p.fd_nx), n = e - c * nx;
        const cx<T> val = lds[c * P.ld + x_lo + n];
        const int ya = ybase + 2 * c;
        uint32_t ia = kOOB, ib = kOOB;
        if (!p.scatter) {
          if (ya < p.y_hi) ia = (uint32_t)((zrow + ya) * rowlen + n);
          if (ya + 1 < p.y_hi) ib = (uint32_t)((zrow + ya + 1) * rowlen + n);
        } else {
          // the interior is no larger than the grid and its origin lies in it: one wrap at most
          const int xg = wrap_once(p.ox + n, p.GX);
          const int ra = wrap_once(p.oy + ya - p.gy, p.GY);
          if (ya < p.y_hi) ia = (uint32_t)((zrow + ra) * rowlen + xg);
          if (ya + 1 < p.y_hi) ib = (uint32_t)((zrow + wrap_once(ra + 1, p.GY)) * rowlen + xg);
        }
        // streamed: G1 is read back by the next step's fill
        gm<T>::template st<kXStore<T>>(dst, ia, val.re);
        gm<T>::template st<kXStore<T>>(dst, ib, val.im);
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ kernels
// Wavefronts per SIMD the registers are cut for.  FP32: 4 (128 registers) for the small radices,
// 3 (168) for the chirp-z y and z passes and the large radices; FP64: 2 (256) and, for the large
// radices, 1.
template <typename T, int CLASS>
constexpr int kPairWaves = sizeof(T) == 4 ? (CLASS % 2 == 0 ? 4 : 3) : (CLASS % 2 == 0 ? 2 : 1);
template <typename T, int CLASS>
constexpr int kPairWavesY = sizeof(T) == 4 ? (CLASS == 0 ? 5 : CLASS == 2 ? 4 : 3) : kPairWaves<T, CLASS>;
template <typename T, int CLASS>
constexpr int kPairWavesZ = sizeof(T) == 4 ? (CLASS == 0 ? 4 : CLASS == 1 ? 2 : 3) : 2;
// x inverse: a point is loaded as the 16 bytes of a bin's two rows, so a butterfly in flight
// takes twice the registers (the LDS of its blocks leaves three wavefronts per SIMD anyway)
template <typename T, int CLASS>
constexpr int kPairWavesXInv = sizeof(T) == 4 ? (CLASS == 2 ? 4 : CLASS == 1 ? 2 : 3) : kPairWaves<T, CLASS>;
template <typename T, int CLASS>
constexpr int kPairThreads = pair_threads_max(sizeof(T) == 8, CLASS, false);

#define PSATD_PAIR_ATTR(T, C, W) \
  __global__ void __launch_bounds__((kPairThreads<T, C>)) __attribute__((amdgpu_waves_per_eu(W<T, C>)))

template <typename T, int C, bool PML>
PSATD_PAIR_ATTR(T, C, kPairWaves) k_pxfwd(XFwdParams<T>) {
  pair_xfwd_body<C, false, PML, T>(SingleSrc<XFwdParams<T>>{});
}
template <typename T, int C>
PSATD_PAIR_ATTR(T, C, kPairWaves) k_pxfwd_b(BatchArgs<XFwdParams<T>> a) {
  pair_xfwd_body<C, true, false, T>(BatchSrc<XFwdParams<T>>{a});
}
template <int S, typename T, int C>
PSATD_PAIR_ATTR(T, C, kPairWavesY) k_pypass(YPassParams<T>) {
  pair_ypass_body<C, false, S, T>(SingleSrc<YPassParams<T>>{});
}
template <int S, typename T, int C>
PSATD_PAIR_ATTR(T, C, kPairWavesY) k_pypass_b(BatchArgs<YPassParams<T>> a) {
  pair_ypass_body<C, true, S, T>(BatchSrc<YPassParams<T>>{a});
}
template <typename T, int C, bool PML>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(kPairWavesZ<T, C>))) k_pzpush(ZPushParams<T>) {
  pair_zpush_body<C, false, PML, T>(SingleSrc<ZPushParams<T>>{});
}
template <typename T, int C>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(kPairWavesZ<T, C>))) k_pzpush_b(BatchArgs<ZPushParams<T>> a) {
  pair_zpush_body<C, true, false, T>(BatchSrc<ZPushParams<T>>{a});
}
template <typename T, int C, bool PML>
PSATD_PAIR_ATTR(T, C, kPairWavesXInv) k_pxinv(XInvParams<T>) {
  pair_xinv_body<C, false, PML, T>(SingleSrc<XInvParams<T>>{});
}
template <typename T, int C>
PSATD_PAIR_ATTR(T, C, kPairWavesXInv) k_pxinv_b(BatchArgs<XInvParams<T>> a) {
  pair_xinv_body<C, true, false, T>(BatchSrc<XInvParams<T>>{a});
}

// LDS of a pair block: its lines, the stage B twiddles, and P1's column table.
template <typename T>
size_t pair_lds(const PairFFT<T>& P, int lines, int ints) {
  return pair_lds_bytes(P.ra, P.rb, P.ld, lines, sizeof(cx<T>)) + (size_t)ints * sizeof(int);
}

}  // namespace

// ------------------------------------------------------------------ launchers
template <typename T, int C>
void launch_pair_xfwd_c(const XFwdParams<T>& p, hipStream_t s) {
  const size_t lds = pair_lds(p.pair, p.pnl, p.NX);
  if (p.pml)
    launch_persistent(k_pxfwd<T, C, true>, p, p.pthreads, lds, p.ntiles, s);
  else
    launch_persistent(k_pxfwd<T, C, false>, p, p.pthreads, lds, p.ntiles, s);
}
template <typename T, int C>
void launch_pair_ypass_c(const YPassParams<T>& p, int inverse, hipStream_t s) {
  const size_t lds = pair_lds(p.pair, p.pnl, 0);
  if (inverse)
    launch_persistent(k_pypass<1, T, C>, p, p.pthreads, lds, p.ntiles, s);
  else
    launch_persistent(k_pypass<-1, T, C>, p, p.pthreads, lds, p.ntiles, s);
}
template <typename T, int C>
void launch_pair_zpush_c(const ZPushParams<T>& p, hipStream_t s) {
  const size_t lds = pair_lds(p.pair, (p.pml ? 12 : 11) * p.pnl, 0);
  if (p.pml)
    launch_persistent(k_pzpush<T, C, true>, p, p.pthreads, lds, p.ntiles, s);
  else
    launch_persistent(k_pzpush<T, C, false>, p, p.pthreads, lds, p.ntiles, s);
}
template <typename T, int C>
void launch_pair_xinv_c(const XInvParams<T>& p, hipStream_t s) {
  const size_t lds = pair_lds(p.pair, p.pnl, 0);
  if (p.pml)
    launch_persistent(k_pxinv<T, C, true>, p, p.pthreads, lds, p.ntiles, s);
  else
    launch_persistent(k_pxinv<T, C, false>, p, p.pthreads, lds, p.ntiles, s);
}
template <typename T, int C>
void launch_pair_xfwd_batch(const BatchArgs<XFwdParams<T>>& a, int threads, size_t lds, hipStream_t s) {
  launch_persistent(k_pxfwd_b<T, C>, a, threads, lds, a.total, s);
}
template <typename T, int C>
void launch_pair_ypass_batch(const BatchArgs<YPassParams<T>>& a, int inverse, int threads, size_t lds, hipStream_t s) {
  if (inverse)
    launch_persistent(k_pypass_b<1, T, C>, a, threads, lds, a.total, s);
  else
    launch_persistent(k_pypass_b<-1, T, C>, a, threads, lds, a.total, s);
}
template <typename T, int C>
void launch_pair_zpush_batch(const BatchArgs<ZPushParams<T>>& a, int threads, size_t lds, hipStream_t s) {
  launch_persistent(k_pzpush_b<T, C>, a, threads, lds, a.total, s);
}
template <typename T, int C>
void launch_pair_xinv_batch(const BatchArgs<XInvParams<T>>& a, int threads, size_t lds, hipStream_t s) {
  launch_persistent(k_pxinv_b<T, C>, a, threads, lds, a.total, s);
}

// Explicit instantiations, taken up by the units at the end of passes.hip.
#define PSATD_PAIR_1(T, C) template void launch_pair_xfwd_c<T, C>(const XFwdParams<T>&, hipStream_t);
#define PSATD_PAIR_2(T, C) template void launch_pair_ypass_c<T, C>(const YPassParams<T>&, int, hipStream_t);
#define PSATD_PAIR_3(T, C) template void launch_pair_zpush_c<T, C>(const ZPushParams<T>&, hipStream_t);
#define PSATD_PAIR_4(T, C) template void launch_pair_xinv_c<T, C>(const XInvParams<T>&, hipStream_t);
#define PSATD_PAIR_BATCH_1(T, C) \
  template void launch_pair_xfwd_batch<T, C>(const BatchArgs<XFwdParams<T>>&, int, size_t, hipStream_t);
#define PSATD_PAIR_BATCH_2(T, C) \
  template void launch_pair_ypass_batch<T, C>(const BatchArgs<YPassParams<T>>&, int, int, size_t, hipStream_t);
#define PSATD_PAIR_BATCH_3(T, C) \
  template void launch_pair_zpush_batch<T, C>(const BatchArgs<ZPushParams<T>>&, int, size_t, hipStream_t);
#define PSATD_PAIR_BATCH_4(T, C) \
  template void launch_pair_xinv_batch<T, C>(const BatchArgs<XInvParams<T>>&, int, size_t, hipStream_t);

}  // namespace psatd
