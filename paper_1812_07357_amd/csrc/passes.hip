// The five passes of one PSATD step on a box (gfx950).
//
//   P1 xfwd   G1 (periodic gather, guard fill fused) or box reals -> x R2C -> layout A
//   P2 ypass  layout A -> y C2C forward -> layout B
//   P3 zpush  layout B -> z C2C forward, analytic push, z C2C inverse -> layout B (E, B)
//   P4 ypass  layout B -> y C2C inverse -> layout A (E, B)
//   P5 xinv   layout A -> x C2R -> box reals or G1 interior (guard merge fused)
//
// Sec. 1.1 of arXiv:1812.07357 (Fourier transform, analytic k-space update,
// inverse transform) and Sec. 2.5.2 (fill G2 guards from G1, copy the interior
// back).  The real-to-complex and complex-to-real x transforms pack two
// neighbouring real y-lines into one complex line: with z = a + i b,
//   A(k) = (Z(k) + conj Z(-k)) / 2,   B(k) = (Z(k) - conj Z(-k)) / (2 i),
// and the inverse rebuilds Z = A + i B over the full line from the half
// spectra (imaginary parts of the self-conjugate bins dropped).
//
// Every kernel is persistent: a block loads a tile into LDS (through registers,
// in rounds of a few values per thread), transforms it, writes it out and takes
// the next tile.  Blocks are small enough in registers (FP32: at most 128, 96 for
// the z pass and 80 for the single-box y pass, whatever that costs in spills) that
// several share a CU and overlap one another's loads, transforms and barriers.
// All global accesses go through buffer resources with hardware range checks
// (gmem.hpp); an index that is out of range by construction (kOOB) reads zero
// and drops writes.
//
// Each pass body is written against a parameter source: a single box (the
// parameters are the kernel argument) or a batch of boxes of different sizes
// (per-box parameters in device memory, tiles of all boxes numbered one after
// the other).  A batched launch is one persistent grid over the tiles of every
// box (Fig. 1(a) of the paper: many sub-domains, each advanced on its own).

#include "internal.hpp"
#include "pass_common.hpp"
#include "pair_passes.hpp"

namespace psatd {

namespace {

// ------------------------------------------------------------------ P1
// Tiles are ty consecutive y rows of one (field, z) plane, packed as ty/2
// complex lines.  Loads go to LDS in rounds of load_round values per thread;
// overlap comes from several blocks per CU.
template <typename T, typename Src>
__device__ __forceinline__ void xfwd_body(const Src& S) {
  constexpr int kRound = load_round<T>::v;  // element pairs loaded per thread before they go to LDS
  cx<T>* lds = lds_base<T>();
  const int tid = threadIdx.x, nth = blockDim.x;

  for (int tile = blockIdx.x; tile < S.ntiles(); tile += gridDim.x) {
    int lt;
    const XFwdParams<T>& p = S.box(tile, lt);
    const int q = fdiv(lt, p.fd_ytiles);
    const int ybase = (lt - q * p.ytiles) * p.ty;
    const int f = fdiv(q, p.fd_NZ);
    const int z = q - f * p.NZ;
    const int NX = p.NX, NY = p.NY, NXH = p.NXH, ty = p.ty, nc = ty >> 1;
    const int ld = fft_slots(p.fft.sch.n);
    const int nld = nc * NX;
    {
      const rsrc_t src = make_rsrc(p.src[f], p.src_bytes);
      const int zrow = p.gather ? fmod_i(p.z0 + z, p.fd_GZ) * p.GY : z * NY;
      const int rowlen = p.gather ? p.GX : NX;
      // Gather table, after the tile's lines: the wrapped x of every column, then the G1
      // offset of every real row of the tile, so the loads below need no divisions.
      int* tab = reinterpret_cast<int*>(lds + nc * ld);
      if (p.xtab) {
        for (int i = tid; i < NX + ty; i += nth)
          tab[i] = i < NX ? fmod_i(p.x0 + i, p.fd_GX) : (zrow + fmod_i(p.y0 + ybase + (i - NX), p.fd_GY)) * rowlen;
        __syncthreads();
      }
      Walk w;
      w.row = fdiv(tid, p.fd_NX);
      w.col = tid - w.row * NX;
      for (int e0 = 0; e0 < nld; e0 += kRound * nth) {
        T re[kRound], im[kRound];
        Walk w0 = w;
#pragma unroll
        for (int u = 0; u < kRound; ++u) {
          uint32_t ia = kOOB, ib = kOOB;
          if (e0 + tid + u * nth < nld) {
            const int ya = ybase + 2 * w.row;
            int xs = w.col, ra = ya, rb = ya + 1;
            if (p.xtab) {
              const int xt = tab[w.col];
              if (ya < NY) ia = (uint32_t)(tab[NX + 2 * w.row] + xt);
              if (ya + 1 < NY) ib = (uint32_t)(tab[NX + 2 * w.row + 1] + xt);
            } else {
              if (p.gather) {
                xs = fmod_i(p.x0 + w.col, p.fd_GX);
                ra = fmod_i(p.y0 + ya, p.fd_GY);
                rb = fmod_i(p.y0 + ya + 1, p.fd_GY);
              }
              if (ya < NY) ia = (uint32_t)((zrow + ra) * rowlen + xs);
              if (ya + 1 < NY) ib = (uint32_t)((zrow + rb) * rowlen + xs);
            }
          }
          re[u] = gm<T>::ld(src, ia);
          im[u] = gm<T>::ld(src, ib);
          w.next(p.ld_drow, p.ld_dcol, NX);
        }
#pragma unroll
        for (int u = 0; u < kRound; ++u) {
          if (e0 + tid + u * nth < nld) lds[w0.row * ld + lpad(w0.col)] = {re[u], im[u]};
          w0.next(p.ld_drow, p.ld_dcol, NX);
        }
      }
    }
    __syncthreads();
    lds_line_fft<-1, T>(lds, ld, nc, p.fft);

    // Split each complex line c into the half spectra of its two real lines
    // (y = 2c and 2c + 1), written as one pair; y fastest.
    const rsrc_t dst = make_rsrc(p.dst + (i64)f * p.fsA, p.dst_bytes);
    const int ny_t = min(ty, NY - ybase);
    const int nwr = NXH * nc;
    Walk v;
    v.row = fdiv(tid, p.fd_nc);
    v.col = tid - v.row * nc;
#pragma unroll 2
    for (int e = tid; e < nwr; e += nth) {
      const int kx = v.row, c = v.col;
      const cx<T> za = lds[c * ld + lpad(kx)];
      const cx<T> zb = cconj(lds[c * ld + lpad(kx == 0 ? 0 : NX - kx)]);
      const cx<T> sum = cadd(za, zb), dif = csub(za, zb);
      const cx<T> va = cscale(sum, T(0.5));
      const cx<T> vb = {T(0.5) * dif.im, T(-0.5) * dif.re};
      const int t = 2 * c;
      const uint32_t o = (uint32_t)((z * NXH + kx) * NY + ybase + t);
      // streamed: layout A is read back by the y pass after all of it has been written
      if (t + 1 < ny_t)
        gm<T>::template stc2<kXStore<T>>(dst, o, va, vb);
      else if (t < ny_t)
        gm<T>::template stc<kXStore<T>>(dst, o, va);
      v.next(p.wr_drow, p.wr_dcol, nc);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ P2 / P4
// Tiles are y-lines (about 5k elements); loads go to LDS in rounds of
// load_round values per thread, and several blocks per CU overlap each other.
template <int S_, typename T, typename Src>
__device__ __forceinline__ void ypass_body(const Src& S) {
  constexpr int kRound = load_round<T>::v;
  cx<T>* lds = lds_base<T>();
  const int tid = threadIdx.x, nth = blockDim.x;

  struct Tile {
    int f, o, u0, nlt;
    FastDiv fnl;
  };
  auto decode = [&](const YPassParams<T>& p, int lt) {
    Tile t;
    const int q = fdiv(lt, p.fd_utiles);
    const int ut = lt - q * p.utiles;
    t.f = fdiv(q, p.fd_nouter);
    t.o = q - t.f * p.nouter;
    t.u0 = p.u_lo + ut * p.nl;
    const bool last = (ut == p.utiles - 1);
    t.nlt = last ? p.nl_last : p.nl;
    t.fnl = last ? p.fd_nl_last : p.fd_nl;
    return t;
  };
  // walk over a tile's input elements in the input's preferred order:
  // positions fastest when lines are contiguous, line index fastest otherwise
  auto start_in = [&](const YPassParams<T>& p, const Tile& t, Walk& w, int& dr, int& dc, int& ncol) {
    if (p.ps_in == 1) {
      w.row = fdiv(tid, p.fd_n);
      w.col = tid - w.row * p.n;
      dr = fdiv(nth, p.fd_n);
      dc = nth - dr * p.n;
      ncol = p.n;
    } else {
      w.row = fdiv(tid, t.fnl);
      w.col = tid - w.row * t.nlt;
      dr = fdiv(nth, t.fnl);
      dc = nth - dr * t.nlt;
      ncol = t.nlt;
    }
  };
  for (int tile = blockIdx.x; tile < S.ntiles(); tile += gridDim.x) {
    int lt;
    const YPassParams<T>& p = S.box(tile, lt);
    const Tile t = decode(p, lt);
    const int ld = fft_slots(p.fft.sch.n);
    {
      const rsrc_t in = make_rsrc(p.in + (i64)t.f * p.fs_in + (i64)t.o * p.ob_in, p.in_bytes);
      const int base = t.o * p.os_in + t.u0 * p.ls_in;
      const int tot = t.nlt * p.n;
      Walk w;
      int dr, dc, ncol;
      start_in(p, t, w, dr, dc, ncol);
      for (int e0 = 0; e0 < tot; e0 += kRound * nth) {
        cx<T> r[kRound];
        Walk w0 = w;
#pragma unroll
        for (int u = 0; u < kRound; ++u) {
          uint32_t idx = kOOB;
          if (e0 + tid + u * nth < tot) {
            const int li = (p.ps_in == 1) ? w.row : w.col;
            const int q = (p.ps_in == 1) ? w.col : w.row;
            idx = (uint32_t)(base + li * p.ls_in + q * p.ps_in);
          }
          r[u] = gm<T>::ldc(in, idx);
          w.next(dr, dc, ncol);
        }
#pragma unroll
        for (int u = 0; u < kRound; ++u) {
          if (e0 + tid + u * nth < tot) {
            const int li = (p.ps_in == 1) ? w0.row : w0.col;
            const int q = (p.ps_in == 1) ? w0.col : w0.row;
            lds[li * ld + lpad(q)] = r[u];
          }
          w0.next(dr, dc, ncol);
        }
      }
    }
    __syncthreads();
    lds_line_fft<S_, T>(lds, ld, t.nlt, p.fft);

    const rsrc_t out = make_rsrc(p.out + (i64)t.f * p.fs_out + (i64)t.o * p.ob_out, p.out_bytes);
    const int obase = t.o * p.os_out + t.u0 * p.ls_out;
    const int np = p.p_hi - p.p_lo;
    const int tot = t.nlt * np;
    Walk w;
    int dr, dc, ncol;
    if (p.ps_out == 1) {
      w.row = fdiv(tid, p.fd_np);
      w.col = tid - w.row * np;
      dr = fdiv(nth, p.fd_np);
      dc = nth - dr * np;
      ncol = np;
    } else {
      w.row = fdiv(tid, t.fnl);
      w.col = tid - w.row * t.nlt;
      dr = fdiv(nth, t.fnl);
      dc = nth - dr * t.nlt;
      ncol = t.nlt;
    }
#pragma unroll 4
    for (int e = tid; e < tot; e += nth) {
      const int li = (p.ps_out == 1) ? w.row : w.col;
      const int q = p.p_lo + ((p.ps_out == 1) ? w.col : w.row);
      gm<T>::stc(out, (uint32_t)(obase + li * p.ls_out + q * p.ps_out), lds[li * ld + lpad(q)]);
      w.next(dr, dc, ncol);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ P3
// Push (Sec. 1.1; J constant over the step, rho at both ends):
//   E' = C E + i c^2 S1 (K x B) - (S1/eps0) J + i (c^2/eps0) K (X3 rho_old - X2 rho_new)
//   B' = C B - i S1 (K x E) + i (X1/eps0) (K x J)
// A tile is ncol consecutive (kx, ky) columns (one for long lines, several for
// short ones): their 11 z-lines each are loaded into LDS, transformed, pushed
// point by point, and the 6 lines of E and B per column transformed back and
// stored over the interior z range.  LDS line f * ncol + c holds field f of
// the tile's column c, so the E and B lines of all columns come first and the
// inverse transform runs over one contiguous block of 6 ncol lines (the last
// tile of a box may have fewer columns: its missing lines hold zeros).  This pass
// does not hold the next tile in registers: the transforms leave no room for
// it, and small blocks with a 96-register cap (FP32, five per CU) let several
// tiles per CU overlap each other's loads and barriers instead.
// MULTI = false compiles the single-column case (ncol == 1) without the column bookkeeping.
// PML selects the split-field increments of push_point_pml instead of the ordinary push:
// twelve output lines per column (both split sets) instead of six.
template <typename T, bool MULTI, typename Src, bool PML = false>
__device__ __forceinline__ void zpush_body(const Src& S) {
  constexpr int kRound = 16;  // line chunks of 64 points loaded per thread before they go to LDS
  cx<T>* lds = lds_base<T>();
  const int tid = threadIdx.x, nth = blockDim.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int nwaves = nth >> 6;
  for (int tile = blockIdx.x; tile < S.ntiles(); tile += gridDim.x) {
    int lt;
    const ZPushParams<T>& p = S.box(tile, lt);
    const int NZ = p.NZ;
    const int ld = fft_slots(p.fft.sch.n);
    const int col0 = lt * p.ncol;
    const int ncol = MULTI ? p.ncol : 1;
    const int nct = MULTI ? min(ncol, p.NXH * p.NY - col0) : 1;  // columns present in this tile
    const int nlines = 11 * ncol;
    const int per_line = (NZ + 63) >> 6;
    const int items = ((nlines - wave + nwaves - 1) / nwaves) * per_line;  // (line, chunk) pairs of this wave
    for (int q0 = 0; q0 < items; q0 += kRound) {
      cx<T> r[kRound];
#pragma unroll
      for (int u = 0; u < kRound; ++u) {
        const int q = q0 + u;
        const int sl = q / per_line, i = q - sl * per_line;
        const int l = wave + sl * nwaves;  // LDS line: field l / ncol, column l % ncol
        const int f = MULTI ? fdiv(l, p.fd_ncol) : l, c = MULTI ? l - f * ncol : 0;
        const int z = lane + 64 * i;
        const bool ok = q < items && z < NZ && (!MULTI || c < nct);
        const rsrc_t rb = make_rsrc(p.b + (i64)(col0 + (ok ? c : 0)) * p.csB + (ok ? f : 0) * NZ,
                                    (uint32_t)NZ * (uint32_t)sizeof(cx<T>));
        r[u] = gm<T>::ldc(rb, ok ? (uint32_t)z : kOOB);
      }
#pragma unroll
      for (int u = 0; u < kRound; ++u) {
        const int q = q0 + u;
        const int sl = q / per_line, i = q - sl * per_line;
        const int z = lane + 64 * i;
        if (q < items && z < NZ) lds[(wave + sl * nwaves) * ld + lpad(z)] = r[u];
      }
    }
    __syncthreads();
    // lines are independent: transform them in groups that fit the block's butterfly budget
    if (p.zgroup >= nlines)
      lds_line_fft<-1, T>(lds, ld, nlines, p.fft);
    else
      for (int l0 = 0; l0 < nlines; l0 += p.zgroup)
        lds_line_fft<-1, T>(lds + l0 * ld, ld, min(p.zgroup, nlines - l0), p.fft);

    const int fs = ncol * ld;  // LDS distance between the lines of consecutive fields
    for (int e = tid; e < nct * NZ; e += nth) {
      const int c = MULTI ? fdiv(e, p.fd_NZ) : 0;
      const int at = c * ld + lpad(e - c * NZ);
      PushPoint<T> q;
      q.load(p, col0, e, nct * NZ);
      q.wavenumbers(p, col0 + c, e - c * NZ);
      if constexpr (PML)
        push_point_pml(p, lds, fs, at, q);
      else
        push_point_c(p, lds, fs, at, q);
    }
    __syncthreads();
    constexpr int kOut = PML ? 12 : 6;  // output lines per column
    if (p.zgroup >= kOut * ncol)
      lds_line_fft<1, T>(lds, ld, kOut * ncol, p.fft);
    else
      for (int l0 = 0; l0 < kOut * ncol; l0 += p.zgroup)
        lds_line_fft<1, T>(lds + l0 * ld, ld, min(p.zgroup, kOut * ncol - l0), p.fft);

    for (int l = wave; l < kOut * ncol; l += nwaves) {
      const int f = MULTI ? fdiv(l, p.fd_ncol) : l, c = MULTI ? l - f * ncol : 0;
      if (MULTI && c >= nct) continue;
      const rsrc_t rb = make_rsrc(p.b + (i64)(col0 + c) * p.csB + f * NZ, (uint32_t)NZ * (uint32_t)sizeof(cx<T>));
      for (int z = p.z_lo + lane; z < p.z_hi; z += 64) gm<T>::stc(rb, (uint32_t)z, lds[l * ld + lpad(z)]);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ P5
// Tiles are ty/2 complex x-lines rebuilt from the half spectra of ty real
// lines; loads go straight to LDS in rounds, several blocks per CU overlap.
template <typename T, typename Src>
__device__ __forceinline__ void xinv_body(const Src& S) {
  constexpr int kRound = load_round<T>::v / 2;  // two values per element
  cx<T>* lds = lds_base<T>();
  const int tid = threadIdx.x, nth = blockDim.x;

  for (int tile = blockIdx.x; tile < S.ntiles(); tile += gridDim.x) {
    int lt;
    const XInvParams<T>& p = S.box(tile, lt);
    const int q = fdiv(lt, p.fd_ytiles);
    const int ybase = p.y_lo + (lt - q * p.ytiles) * p.ty;
    const int f = fdiv(q, p.fd_nz);
    const int zs = q - f * p.nzs, z = p.zfirst + zs;  // plane of the interior, and of the box
    const int NX = p.NX, NY = p.NY, NXH = p.NXH, nc = p.ty >> 1;
    const int ld = fft_slots(p.fft.sch.n);
    {
      // Rebuild Z = A + i B over the full line from the half spectra of the two real lines.
      const int nld = nc * NXH;
      const rsrc_t src = make_rsrc(p.src + (i64)f * p.npts, p.src_bytes);
      const int sbase = zs * NXH * NY;
      Walk w;
      w.row = fdiv(tid, p.fd_nc);  // (kx, complex line)
      w.col = tid - w.row * nc;
      const int ldr = fdiv(nth, p.fd_nc), ldc = nth - ldr * nc;  // block stride over (kx, complex line)
      for (int e0 = 0; e0 < nld; e0 += kRound * nth) {
        cx<T> av[kRound], bv[kRound];
        Walk w0 = w;
#pragma unroll
        for (int u = 0; u < kRound; ++u) {
          uint32_t ia = kOOB, ib = kOOB;
          if (e0 + tid + u * nth < nld) {
            const int ya = ybase + 2 * w.col;
            if (ya < p.y_hi) ia = (uint32_t)(sbase + w.row * NY + ya);
            if (ya + 1 < p.y_hi) ib = (uint32_t)(sbase + w.row * NY + ya + 1);
          }
          av[u] = gm<T>::ldc(src, ia);
          bv[u] = gm<T>::ldc(src, ib);
          w.next(ldr, ldc, nc);
        }
#pragma unroll
        for (int u = 0; u < kRound; ++u) {
          if (e0 + tid + u * nth < nld) {
            const int kx = w0.row, c = w0.col;
            cx<T> x = av[u], y = bv[u];
            const bool selfconj = (kx == 0) || (2 * kx == NX);
            if (selfconj) {
              x.im = T(0);
              y.im = T(0);
            }
            lds[c * ld + lpad(kx)] = {x.re - y.im, x.im + y.re};
            if (!selfconj) lds[c * ld + lpad(NX - kx)] = {x.re + y.im, y.re - x.im};
          }
          w0.next(ldr, ldc, nc);
        }
      }
    }
    __syncthreads();
    lds_line_fft<1, T>(lds, ld, nc, p.fft);

    const rsrc_t dst = make_rsrc(p.dst[f], p.dst_bytes);
    const int zrow = p.scatter ? fmod_i(p.oz + z - p.gz, p.fd_GZ) * p.GY : z * NY;
    const int rowlen = p.scatter ? p.GX : NX;
    const int nwr = nc * NX;
    Walk v;
    v.row = fdiv(tid, p.fd_NX);  // (complex line, x)
    v.col = tid - v.row * NX;
    const int wdr = fdiv(nth, p.fd_NX), wdc = nth - wdr * NX;  // block stride over (complex line, x)
#pragma unroll 4
    for (int e = tid; e < nwr; e += nth) {
      const int c = v.row, n = v.col;
      const cx<T> val = lds[c * ld + lpad(n)];
      const int ya = ybase + 2 * c;
      uint32_t ia = kOOB, ib = kOOB;
      if (!p.scatter) {
        if (ya < p.y_hi) ia = (uint32_t)((zrow + ya) * rowlen + n);
        if (ya + 1 < p.y_hi) ib = (uint32_t)((zrow + ya + 1) * rowlen + n);
      } else if (n >= p.gx && n < p.gx + p.nx) {
        // the interior is no larger than the grid and its origin lies in it: one wrap at most
        const int xg = wrap_once(p.ox + n - p.gx, p.GX);
        const int ra = wrap_once(p.oy + ya - p.gy, p.GY);
        if (ya < p.y_hi) ia = (uint32_t)((zrow + ra) * rowlen + xg);
        if (ya + 1 < p.y_hi) ib = (uint32_t)((zrow + wrap_once(ra + 1, p.GY)) * rowlen + xg);
      }
      // streamed: G1 is read back by the next step's fill
      gm<T>::template st<kXStore<T>>(dst, ia, val.re);
      gm<T>::template st<kXStore<T>>(dst, ib, val.im);
      v.next(wdr, wdc, NX);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ kernels
// x forward: at most 128 registers in FP32 (two blocks per CU).
template <typename T>
__global__ void __launch_bounds__(kLineThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 1)))
k_xfwd(XFwdParams<T>) {
  xfwd_body<T>(SingleSrc<XFwdParams<T>>{});
}
template <typename T>
__global__ void __launch_bounds__(kLineThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 1)))
k_xfwd_b(BatchArgs<XFwdParams<T>> a) {
  xfwd_body<T>(BatchSrc<XFwdParams<T>>{a});
}
// y passes (single box): FP32 capped at 80 registers, three blocks per CU.  The
// spills this costs are cheaper than the lost latency hiding of two blocks.
template <int S, typename T>
__global__ void __launch_bounds__(kLineThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 6 : 1)))
k_ypass(YPassParams<T>) {
  ypass_body<S, T>(SingleSrc<YPassParams<T>>{});
}
template <int S, typename T>
__global__ void __launch_bounds__(kLineThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 1)))
k_ypass_b(BatchArgs<YPassParams<T>> a) {
  ypass_body<S, T>(BatchSrc<YPassParams<T>>{a});
}
// z pass: FP32 single-box tiles (one column: only lengths without a pair come here) fit 96
// registers (5 waves per SIMD), batched ones 128 (4); FP64 256 (2).
template <typename T, int NTH, bool PML = false>
__global__ void __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 5 : 2)))
k_zpush(ZPushParams<T>) {
  zpush_body<T, false, SingleSrc<ZPushParams<T>>, PML>(SingleSrc<ZPushParams<T>>{});
}
template <typename T, int NTH>
__global__ void __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
k_zpush_b(BatchArgs<ZPushParams<T>> a) {
  zpush_body<T, true>(BatchSrc<ZPushParams<T>>{a});
}
// x inverse: at most 128 registers in FP32; 256-thread blocks (four per CU) unless
// the lines need the larger block.
template <typename T, int NTH>
__global__ void __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 1)))
k_xinv(XInvParams<T>) {
  xinv_body<T>(SingleSrc<XInvParams<T>>{});
}
template <typename T, int NTH>
__global__ void __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 1)))
k_xinv_b(BatchArgs<XInvParams<T>> a) {
  xinv_body<T>(BatchSrc<XInvParams<T>>{a});
}

}  // namespace

// ------------------------------------------------------------------ launchers
template <typename T>
size_t xfwd_lds(const XFwdParams<T>& p) {
  const size_t lines = (size_t)(p.ty / 2) * fft_slots(p.fft.sch.n) * cx_bytes<T>();
  return lines + (p.xtab ? (size_t)(p.NX + p.ty) * sizeof(int) : 0);
}
template <typename T>
size_t ypass_lds(const YPassParams<T>& p) {
  return (size_t)p.nl * fft_slots(p.fft.sch.n) * cx_bytes<T>();
}
template <typename T>
size_t zpush_lds(const ZPushParams<T>& p) {
  return (size_t)(p.pml ? 12 : 11) * p.ncol * fft_slots(p.fft.sch.n) * cx_bytes<T>();
}
template <typename T>
size_t xinv_lds(const XInvParams<T>& p) {
  return (size_t)(p.ty / 2) * fft_slots(p.fft.sch.n) * cx_bytes<T>();
}

template <typename T>
void launch_xfwd(const XFwdParams<T>& p, hipStream_t s) {
  launch_persistent(k_xfwd<T>, p, kLineThreads, xfwd_lds(p), p.ntiles, s);
}
template <typename T>
void launch_ypass(const YPassParams<T>& p, int inverse, hipStream_t s) {
  if (inverse)
    launch_persistent(k_ypass<1, T>, p, kLineThreads, ypass_lds(p), p.ntiles, s);
  else
    launch_persistent(k_ypass<-1, T>, p, kLineThreads, ypass_lds(p), p.ntiles, s);
}
template <typename T, bool PML>
void launch_zpush_line(const ZPushParams<T>& p, int nthreads, hipStream_t s) {
  if (nthreads == kZThreads[0])
    launch_persistent(k_zpush<T, kZThreads[0], PML>, p, nthreads, zpush_lds(p), p.ntiles, s);
  else
    launch_persistent(k_zpush<T, kZThreads[1], PML>, p, nthreads, zpush_lds(p), p.ntiles, s);
}
// The ordinary and the PML kernels build as two units, in parallel.
#if defined(PSATD_UNIT) && PSATD_UNIT != 6
extern template void launch_zpush_line<float, true>(const ZPushParams<float>&, int, hipStream_t);
extern template void launch_zpush_line<double, true>(const ZPushParams<double>&, int, hipStream_t);
#endif
template <typename T>
void launch_zpush(const ZPushParams<T>& p, int nthreads, hipStream_t s) {
  if (p.pml)  // split-field increments
    launch_zpush_line<T, true>(p, nthreads, s);
  else
    launch_zpush_line<T, false>(p, nthreads, s);
}
template <typename T>
void launch_xinv(const XInvParams<T>& p, hipStream_t s) {
  if (p.nthreads == kXInvThreads)
    launch_persistent(k_xinv<T, kXInvThreads>, p, kXInvThreads, xinv_lds(p), p.ntiles, s);
  else
    launch_persistent(k_xinv<T, kLineThreads>, p, kLineThreads, xinv_lds(p), p.ntiles, s);
}

template <typename T>
void launch_xfwd_batch(const BatchArgs<XFwdParams<T>>& a, size_t lds, hipStream_t s) {
  launch_persistent(k_xfwd_b<T>, a, kLineThreads, lds, a.total, s);
}
template <typename T>
void launch_ypass_batch(const BatchArgs<YPassParams<T>>& a, int inverse, size_t lds, hipStream_t s) {
  if (inverse)
    launch_persistent(k_ypass_b<1, T>, a, kLineThreads, lds, a.total, s);
  else
    launch_persistent(k_ypass_b<-1, T>, a, kLineThreads, lds, a.total, s);
}
template <typename T>
void launch_zpush_batch(const BatchArgs<ZPushParams<T>>& a, int nthreads, size_t lds, hipStream_t s) {
  if (nthreads == kZThreads[0])
    launch_persistent(k_zpush_b<T, kZThreads[0]>, a, nthreads, lds, a.total, s);
  else
    launch_persistent(k_zpush_b<T, kZThreads[1]>, a, nthreads, lds, a.total, s);
}
template <typename T>
void launch_xinv_batch(const BatchArgs<XInvParams<T>>& a, int nthreads, size_t lds, hipStream_t s) {
  if (nthreads == kXInvThreads)
    launch_persistent(k_xinv_b<T, kXInvThreads>, a, kXInvThreads, lds, a.total, s);
  else
    launch_persistent(k_xinv_b<T, kLineThreads>, a, kLineThreads, lds, a.total, s);
}


// Explicit instantiations.  The build compiles this file once per unit and precision
// (-DPSATD_UNIT=1..9 -DPSATD_REAL=float|double) so that the units compile in parallel:
// 1..6 the Stockham kernels of one pass, 7 the direct and 8 the chirp-z pair kernels, 9 those
// of batches; -DPSATD_PART=1..4 takes one pass (x forward, y, z, x inverse) of a unit 7..9 and
// -DPSATD_CLASS=0|2 one class of unit 9.
#define PSATD_INST_1(T)                                                                     \
  template void launch_xfwd<T>(const XFwdParams<T>&, hipStream_t);                          \
  template void launch_xfwd_batch<T>(const BatchArgs<XFwdParams<T>>&, size_t, hipStream_t); \
  template size_t xfwd_lds<T>(const XFwdParams<T>&);
#define PSATD_INST_2(T)                                                                               \
  template void launch_ypass<T>(const YPassParams<T>&, int, hipStream_t);                             \
  template void launch_ypass_batch<T>(const BatchArgs<YPassParams<T>>&, int, size_t, hipStream_t); \
  template size_t ypass_lds<T>(const YPassParams<T>&);
#define PSATD_INST_3(T)                                                   \
  template void launch_zpush<T>(const ZPushParams<T>&, int, hipStream_t); \
  template size_t zpush_lds<T>(const ZPushParams<T>&);
#define PSATD_INST_6(T) template void launch_zpush_line<T, true>(const ZPushParams<T>&, int, hipStream_t);
#define PSATD_INST_4(T) \
  template void launch_zpush_batch<T>(const BatchArgs<ZPushParams<T>>&, int, size_t, hipStream_t);
#define PSATD_INST_5(T)                                                                     \
  template void launch_xinv<T>(const XInvParams<T>&, hipStream_t);                          \
  template void launch_xinv_batch<T>(const BatchArgs<XInvParams<T>>&, int, size_t, hipStream_t); \
  template size_t xinv_lds<T>(const XInvParams<T>&);

#define PSATD_CAT2(a, b) a##b
#define PSATD_CAT(a, b) PSATD_CAT2(a, b)
#if PSATD_UNIT <= 6
PSATD_CAT(PSATD_INST_, PSATD_UNIT)(PSATD_REAL)
#else
// units 7 and 8: direct and chirp-z pairs (both classes), 9: batches (classes 0 and 2)
#if PSATD_UNIT == 9 && defined(PSATD_CLASS)
#define PSATD_PAIR(part) PSATD_CAT(PSATD_PAIR_BATCH_, part)(PSATD_REAL, PSATD_CLASS)
#elif PSATD_UNIT == 9
#define PSATD_PAIR(part) \
  PSATD_CAT(PSATD_PAIR_BATCH_, part)(PSATD_REAL, 0) PSATD_CAT(PSATD_PAIR_BATCH_, part)(PSATD_REAL, 2)
#elif PSATD_UNIT == 8
#define PSATD_PAIR(part) PSATD_CAT(PSATD_PAIR_, part)(PSATD_REAL, 2) PSATD_CAT(PSATD_PAIR_, part)(PSATD_REAL, 3)
#else
#define PSATD_PAIR(part) PSATD_CAT(PSATD_PAIR_, part)(PSATD_REAL, 0) PSATD_CAT(PSATD_PAIR_, part)(PSATD_REAL, 1)
#endif
#if defined(PSATD_PART)
PSATD_PAIR(PSATD_PART)
#else
PSATD_PAIR(1) PSATD_PAIR(2) PSATD_PAIR(3) PSATD_PAIR(4)
#endif
#endif

}  // namespace psatd
