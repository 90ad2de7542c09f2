// Guard-width surrogate network on the GPU: forward, backward and Adam (gfx950).
//
// The paper calls a model of the number of guard cells n_g required by a local
// solver, as a function of its order, time step and cell size, crucial (Sec.
// 1.4; n_g drives memory and cost, Sec. 2.2) and leaves it open.  This file
// evaluates and trains a 6 -> 64 -> 64 -> 1 network that predicts log10 of the
// local-vs-global truncation error of a run from six features of it:
//
//   x  = (features - in_mean) * in_scale        (per-feature standardisation)
//   h1 = silu(W1 x + b1),  h2 = silu(W2 h1 + b2),  u = W3 h2 + b3
//   prediction = out_mean + out_scale * u
//   loss over a batch of B samples = (1/B) sum (u - (target - out_mean) / out_scale)^2
//
// Weights live twice: an FP32 master copy that Adam updates and a bfloat16
// copy (round to nearest, ties to even) that the forward and backward kernels
// read.  Activations, products and sums are FP32: the products are FP32 matrix
// instructions (16x16x4) on tiles of 16 samples.  Calls are small, so each
// kernel is a chain of latencies and not of rates.  Weights go from memory into the
// operand registers of their wave, without LDS, and only what crosses waves
// (inputs, h1, dz2) passes through LDS.  With FMAs on LDS tiles of 32 samples 12
// predictions took 8.6 us of kernel time (now 3.4) and a gradient over 512 samples 18.3 + 5.1
// for its two kernels (now 7.2 + 2.7).
//
// Parameter vector (a documented format): W1 (64 x 6, row-major out x in), b1,
// W2 (64 x 64), b2, W3 (64), b3 -- 4673 values.
//
// Gradients are deterministic: each block writes the partial gradient of its
// sample tile, and a second kernel sums the partials in block order.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/psatd.h"
#include "internal.hpp"

namespace {

constexpr int NIN = 6, NH = 64;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NIN, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH, NPARAM = OFF_B3 + 1;
static_assert(NPARAM == PSATD_MLP_NPARAM, "parameter count");
constexpr int TS = 16;       // samples per tile
constexpr int NT = 256;      // threads per block: four waves, 16 units of a layer each
constexpr int LD = NH + 4;   // padded row length of the LDS tiles: operand reads without bank conflicts
constexpr int XP = 8;        // padded row length of the inputs
// A block walks every gridDim-th tile with its weights in registers.  One partial gradient
// per block bounds what the second kernel reads; 256 CUs hold two blocks of the gradient each.
constexpr int kGradBlocks = 512, kForwardBlocks = 2048;

struct Norm {
  float in_mean[NIN];
  float in_scale[NIN];
  float out_mean, out_scale;
};

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// float -> bfloat16, round to nearest with ties to even; NaN stays a quiet NaN
__host__ __device__ inline uint16_t f32_to_bf16(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// silu(z) and its derivative
__device__ __forceinline__ float silu(float z, float& d) {
  const float q = 1.0f + expf(-z), s = 1.0f / q;
  d = s * (1.0f + z * (1.0f - s));
  return z / q;
}

typedef float f4 __attribute__((ext_vector_type(4)));

// D = A B + C with A 16x4 (lane l: row l % 16, column l / 16), B 4x16 (lane l: row l / 16, column
// l % 16), C and D 16x16 (lane l: rows 4 (l / 16) + 0..3, column l % 16).  The four columns of A and
// rows of B of one instruction are any four of the inner index, as long as both agree.
__device__ __forceinline__ f4 mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct Tile {
  float x[TS * XP];  // standardised inputs, column 6 one and column 7 zero
  float t[TS], valid[TS];
  float u[4 * TS];   // the output's sums over the units of each wave
  alignas(16) float h1[TS * LD];
  alignas(16) float dz[TS * LD];
};

// Lane l of wave w holds unit n = 16 w + l % 16 and the inner range of group g = l / 16.
struct Weights {
  float w1[2];   // W1[n][2 g + 0..1], zero for g = 3
  float w2[16];  // W2[n][16 g + 0..15]
  float b1, b2, w3, b3;
};
__device__ __forceinline__ void load_weights(Weights& q, const uint16_t* __restrict__ w, int n, int g) {
  const uint32_t p = g < 3 ? *reinterpret_cast<const uint32_t*>(w + OFF_W1 + n * NIN + 2 * g) : 0u;
  const uint4 a = *reinterpret_cast<const uint4*>(w + OFF_W2 + n * NH + 16 * g),
              b = *reinterpret_cast<const uint4*>(w + OFF_W2 + n * NH + 16 * g + 8);
  q.w1[0] = __uint_as_float(p << 16);
  q.w1[1] = __uint_as_float(p & 0xffff0000u);
  const uint32_t v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    q.w2[2 * k] = __uint_as_float(v[k] << 16);
    q.w2[2 * k + 1] = __uint_as_float(v[k] & 0xffff0000u);
  }
  q.b1 = bf16_to_f32(w[OFF_B1 + n]);
  q.b2 = bf16_to_f32(w[OFF_B2 + n]);
  q.w3 = bf16_to_f32(w[OFF_W3 + n]);
  q.b3 = bf16_to_f32(w[OFF_B3]);
}
static_assert(OFF_W1 % 2 == 0 && NIN % 2 == 0 && OFF_W2 % 8 == 0 && NH % 8 == 0, "alignment of the vector loads");

// The tile's standardised inputs; samples past the batch or with an out-of-range index are masked
// out (valid = 0, inputs 0).
__device__ __forceinline__ void load_tile(Tile& L, const float* __restrict__ X, const float* __restrict__ tgt, int n,
                                          const int* __restrict__ idx, int first, int count, const Norm& nm) {
  const int tid = threadIdx.x;
  if (tid < TS * XP) {
    const int m = tid / XP, k = tid % XP, b = first + m;  // b: position in the batch
    int s = -1;
    if (b < count) s = idx ? idx[b] : b;
    const bool ok = s >= 0 && s < n;
    float mean = nm.in_mean[0], scale = nm.in_scale[0];
#pragma unroll
    for (int c = 1; c < NIN; ++c)
      if (k == c) {
        mean = nm.in_mean[c];
        scale = nm.in_scale[c];
      }
    float v = k == NIN ? 1.0f : 0.0f;
    if (k < NIN) v = ok ? (X[(size_t)s * NIN + k] - mean) * scale : 0.0f;
    L.x[tid] = v;
    if (k == XP - 1) {
      L.valid[m] = ok ? 1.0f : 0.0f;
      L.t[m] = (ok && tgt) ? (tgt[s] - nm.out_mean) / nm.out_scale : 0.0f;
    }
  }
}

// Sum over the 16 lanes of a group, in every lane.
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) v += __shfl_xor(v, d);
  return v;
}
// Sum over the four groups, in every lane.
__device__ __forceinline__ float across_groups(float v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

// 16 floats of an LDS row from 16 g on, the A operands of the 16 products over 64 inner indices
__device__ __forceinline__ void load_row(float* a, const float* row) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const f4 v = *reinterpret_cast<const f4*>(row + 4 * k);
#pragma unroll
    for (int c = 0; c < 4; ++c) a[4 * k + c] = v[c];
  }
}

// Samples 4 g + 0..3 of unit n: h1, h2 and the derivatives of their silu; u (of the same samples) and
// h1 also through LDS.  Starts once the tile's inputs are written (barrier inside).
__device__ __forceinline__ void forward_tile(Tile& L, const Weights& q, int wave, int c, int g, f4& h1, f4& d1, f4& h2,
                                             f4& d2, f4& u) {
  __syncthreads();
  f4 z = {q.b1, q.b1, q.b1, q.b1};
#pragma unroll
  for (int j = 0; j < 2; ++j) z = mfma(L.x[c * XP + 2 * g + j], q.w1[j], z);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float d;
    h1[i] = silu(z[i], d);
    d1[i] = d;
    L.h1[(4 * g + i) * LD + 16 * wave + c] = h1[i];
  }
  __syncthreads();
  float a[16];
  load_row(a, L.h1 + c * LD + 16 * g);
  // two sums, so that each product waits for the one before the last
  f4 za = {q.b2, q.b2, q.b2, q.b2}, zb = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 16; j += 2) {
    za = mfma(a[j], q.w2[j], za);
    zb = mfma(a[j + 1], q.w2[j + 1], zb);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float d;
    h2[i] = silu(za[i] + zb[i], d);
    d2[i] = d;
    const float p = group_sum(q.w3 * h2[i]);
    if (c == 0) L.u[wave * TS + 4 * g + i] = p;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = 4 * g + i;
    u[i] = q.b3 + ((L.u[m] + L.u[TS + m]) + (L.u[2 * TS + m] + L.u[3 * TS + m]));
  }
}

__global__ void __launch_bounds__(NT) k_mlp_forward(const uint16_t* __restrict__ w, const float* __restrict__ X,
                                                     int n, float* __restrict__ y, Norm nm) {
  __shared__ Tile L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  Weights q;
  load_weights(q, w, 16 * wave + c, g);
  for (int tile = blockIdx.x; tile <= (n - 1) / TS; tile += gridDim.x) {
    const int first = tile * TS;
    load_tile(L, X, nullptr, n, nullptr, first, n, nm);
    f4 h1, d1, h2, d2, u;
    forward_tile(L, q, wave, c, g, h1, d1, h2, d2, u);
    // (the inputs of the next tile are written after the last barrier that follows their last read)
    if (wave == 0 && c == 0)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (first + 4 * g + i < n) y[first + 4 * g + i] = nm.out_mean + nm.out_scale * u[i];
  }
}

// Partial MSE gradient of a block's tiles of the batch.
__global__ void __launch_bounds__(NT) k_mlp_grad(const uint16_t* __restrict__ w, const float* __restrict__ X,
                                                  const float* __restrict__ tgt, int n, const int* __restrict__ idx,
                                                  int count, float* __restrict__ part, float* __restrict__ lossp,
                                                  Norm nm) {
  __shared__ Tile L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  const int unit = 16 * wave + c;
  Weights q;
  load_weights(q, w, unit, g);
  float w2t[16];  // W2[16 g + 0..15][n]
#pragma unroll
  for (int j = 0; j < 16; ++j) w2t[j] = bf16_to_f32(w[OFF_W2 + (16 * g + j) * NH + unit]);
  const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f4 gw2[4] = {zero, zero, zero, zero};  // dW2 of rows 16 wave + 4 g + 0..3, columns c + 16 k
  f4 gw1 = zero;                         // dW1 of the same rows, column c; column 6 is db1
  float gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, loss = 0.0f;
  for (int tile = blockIdx.x; tile <= (count - 1) / TS; tile += gridDim.x) {
    const int first = tile * TS;
    load_tile(L, X, tgt, n, idx, first, count, nm);
    f4 h1, d1, h2, d2, u, dz2;
    forward_tile(L, q, wave, c, g, h1, d1, h2, d2, u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = 4 * g + i;
      const float r = (u[i] - L.t[m]) * L.valid[m];
      const float dy = 2.0f * r / (float)count;
      loss += r * r;
      gb3 += dy;
      gw3 = fmaf(dy, h2[i], gw3);
      dz2[i] = dy * q.w3 * d2[i];
      gb2 += dz2[i];
      L.dz[m * LD + unit] = dz2[i];
    }
    // dW2[j][i] += sum over samples of dz2[s][j] h1[s][i]
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) gw2[k] = mfma(dz2[i], L.h1[(4 * g + i) * LD + 16 * k + c], gw2[k]);
    __syncthreads();
    // dz1[s][i] = silu'(z1[s][i]) sum over j of W2[j][i] dz2[s][j]
    float a[16];
    load_row(a, L.dz + c * LD + 16 * g);
    f4 sa = zero, sb = zero;
#pragma unroll
    for (int j = 0; j < 16; j += 2) {
      sa = mfma(a[j], w2t[j], sa);
      sb = mfma(a[j + 1], w2t[j + 1], sb);
    }
    // dW1[j][k] += sum over samples of dz1[s][j] x[s][k]
#pragma unroll
    for (int i = 0; i < 4; ++i)
      gw1 = mfma(d1[i] * (sa[i] + sb[i]), c < XP ? L.x[(4 * g + i) * XP + c] : 0.0f, gw1);
    __syncthreads();  // the next tile's inputs overwrite these
  }
  float* out = part + (size_t)blockIdx.x * NPARAM;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = 16 * wave + 4 * g + i;
#pragma unroll
    for (int k = 0; k < 4; ++k) out[OFF_W2 + j * NH + 16 * k + c] = gw2[k][i];
    if (c < NIN) out[OFF_W1 + j * NIN + c] = gw1[i];
    if (c == NIN) out[OFF_B1 + j] = gw1[i];
  }
  gb2 = across_groups(gb2);
  gw3 = across_groups(gw3);
  gb3 = across_groups(gb3);
  loss = across_groups(loss);
  if (g == 0) {
    out[OFF_B2 + unit] = gb2;
    out[OFF_W3 + unit] = gw3;
  }
  if (threadIdx.x == 0) {
    out[OFF_B3] = gb3;
    lossp[blockIdx.x] = loss;
  }
}

// grad[p] = sum over blocks of the partials, a quarter of them per wave and the quarters in order; loss =
// sum of loss partials / count.  Both also to the caller's arrays where it gave any (two copies
// of their own took as long as this kernel).
constexpr int kReduceParams = 64;
__global__ void __launch_bounds__(256) k_mlp_reduce(const float* __restrict__ part, const float* __restrict__ lossp,
                                                    int nblk, int count, float* __restrict__ grad,
                                                    float* __restrict__ loss, float* __restrict__ grad_out,
                                                    float* __restrict__ loss_out) {
  __shared__ float sum[4][kReduceParams];
  const int k = threadIdx.x % kReduceParams, wave = threadIdx.x / kReduceParams;
  const int p = blockIdx.x * kReduceParams + k;
  const int per = (nblk + 3) / 4, lo = min(nblk, wave * per), hi = min(nblk, lo + per);
  float a = 0.0f;
  if (p < NPARAM) {
#pragma unroll 8
    for (int b = lo; b < hi; ++b) a += part[(size_t)b * NPARAM + p];
  } else if (p == NPARAM) {
    for (int b = lo; b < hi; ++b) a += lossp[b];
  }
  sum[wave][k] = a;
  __syncthreads();
  if (wave != 0 || p > NPARAM) return;
  a = ((sum[0][k] + sum[1][k]) + sum[2][k]) + sum[3][k];
  if (p < NPARAM) {
    grad[p] = a;
    if (grad_out) grad_out[p] = a;
  } else {
    a /= (float)count;
    *loss = a;
    if (loss_out) *loss_out = a;
  }
}

// One Adam step on the FP32 master weights; refreshes the bfloat16 copy.
__global__ void k_mlp_adam(float* __restrict__ master, uint16_t* __restrict__ wbf, float* __restrict__ m,
                           float* __restrict__ v, const float* __restrict__ grad, float lr, float beta1, float beta2,
                           float eps, float bc1, float bc2) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= NPARAM) return;
  const float g = grad[p];
  const float mm = beta1 * m[p] + (1.0f - beta1) * g;
  const float vv = beta2 * v[p] + (1.0f - beta2) * g * g;
  m[p] = mm;
  v[p] = vv;
  const float w = master[p] - lr * (mm / bc1) / (sqrtf(vv / bc2) + eps);
  master[p] = w;
  wbf[p] = f32_to_bf16(w);
}

__global__ void k_mlp_round(const float* __restrict__ master, uint16_t* __restrict__ wbf) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NPARAM) wbf[p] = f32_to_bf16(master[p]);
}

__global__ void k_mlp_zero(float* __restrict__ a, int n) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n) a[p] = 0.0f;
}

}  // namespace

struct psatd_mlp {
  float* master = nullptr;
  uint16_t* wbf = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  float* grad = nullptr;
  float* loss = nullptr;
  float* part = nullptr;
  float* lossp = nullptr;
  int max_batch = 0;
  long long step = 0;
  Norm nm{};
};

namespace {

using psatd::report_error;

int hip_fail(const char* where) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return report_error(PSATD_EHIP, "%s: %s", where, hipGetErrorString(e));
  return PSATD_OK;
}

void free_mlp(psatd_mlp* p) {
  if (!p) return;
  for (void* q : {(void*)p->master, (void*)p->wbf, (void*)p->m, (void*)p->v, (void*)p->grad, (void*)p->loss,
                  (void*)p->part, (void*)p->lossp})
    if (q) (void)hipFree(q);
  delete p;
}

int nblocks(int n, int per) { return (n + per - 1) / per; }

void enqueue_grad(psatd_mlp* p, const float* X, const float* t, int n, const int* idx, int count, float* grad,
                  float* loss, hipStream_t s) {
  const int nb = std::min(nblocks(count, TS), kGradBlocks);
  k_mlp_grad<<<nb, NT, 0, s>>>(p->wbf, X, t, n, idx, count, p->part, p->lossp, p->nm);
  k_mlp_reduce<<<nblocks(NPARAM + 1, kReduceParams), 256, 0, s>>>(p->part, p->lossp, nb, count, p->grad, p->loss, grad,
                                                                  loss);
}

void enqueue_adam(psatd_mlp* p, float lr, float beta1, float beta2, float eps, hipStream_t s) {
  ++p->step;
  const float bc1 = (float)(1.0 - std::pow((double)beta1, (double)p->step));
  const float bc2 = (float)(1.0 - std::pow((double)beta2, (double)p->step));
  k_mlp_adam<<<nblocks(NPARAM, 256), 256, 0, s>>>(p->master, p->wbf, p->m, p->v, p->grad, lr, beta1, beta2, eps,
                                                   bc1, bc2);
}

bool adam_args_ok(float lr, float beta1, float beta2, float eps) {
  return std::isfinite(lr) && lr > 0.f && beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f &&
         std::isfinite(eps) && eps >= 0.f;
}

}  // namespace

extern "C" {

int psatd_mlp_create(const float* init, const float* in_mean, const float* in_scale, float out_mean,
                     float out_scale, int max_batch, psatd_mlp** out) {
  if (!out) return report_error(PSATD_EINVAL, "psatd_mlp_create: out is NULL");
  *out = nullptr;
  if (!init || !in_mean || !in_scale)
    return report_error(PSATD_EINVAL, "psatd_mlp_create: init, in_mean and in_scale are required");
  if (max_batch < 1 || max_batch > (1 << 24))
    return report_error(PSATD_EINVAL, "psatd_mlp_create: max_batch %d outside [1, 2^24]", max_batch);
  if (!(std::isfinite(out_scale) && out_scale != 0.f) || !std::isfinite(out_mean))
    return report_error(PSATD_EINVAL, "psatd_mlp_create: out_scale must be finite and nonzero");
  psatd_mlp* p = new psatd_mlp;
  p->max_batch = max_batch;
  for (int k = 0; k < NIN; ++k) {
    p->nm.in_mean[k] = in_mean[k];
    p->nm.in_scale[k] = in_scale[k];
  }
  p->nm.out_mean = out_mean;
  p->nm.out_scale = out_scale;
  const size_t pb = sizeof(float) * NPARAM;
  const int nb = std::min(nblocks(max_batch, TS), kGradBlocks);
  if (hipMalloc(&p->master, pb) != hipSuccess || hipMalloc(&p->wbf, sizeof(uint16_t) * NPARAM) != hipSuccess ||
      hipMalloc(&p->m, pb) != hipSuccess || hipMalloc(&p->v, pb) != hipSuccess ||
      hipMalloc(&p->grad, pb) != hipSuccess || hipMalloc(&p->loss, sizeof(float)) != hipSuccess ||
      hipMalloc(&p->part, pb * (size_t)nb) != hipSuccess || hipMalloc(&p->lossp, sizeof(float) * nb) != hipSuccess) {
    (void)hipGetLastError();
    free_mlp(p);
    return report_error(PSATD_ENOMEM, "psatd_mlp_create: device allocation failed");
  }
  const int rc = psatd_mlp_set(p, init);
  if (rc) {
    free_mlp(p);
    return rc;
  }
  *out = p;
  return PSATD_OK;
}

int psatd_mlp_set(psatd_mlp* p, const float* master) {
  if (!p || !master) return report_error(PSATD_EINVAL, "psatd_mlp_set: NULL argument");
  if (hipMemcpy(p->master, master, sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess)
    return hip_fail("psatd_mlp_set copy");
  k_mlp_round<<<nblocks(NPARAM, 256), 256>>>(p->master, p->wbf);
  k_mlp_zero<<<nblocks(NPARAM, 256), 256>>>(p->m, NPARAM);
  k_mlp_zero<<<nblocks(NPARAM, 256), 256>>>(p->v, NPARAM);
  p->step = 0;
  if (hipDeviceSynchronize() != hipSuccess) return hip_fail("psatd_mlp_set");
  return hip_fail("psatd_mlp_set");
}

int psatd_mlp_get(const psatd_mlp* p, float* master, unsigned short* bf16) {
  if (!p) return report_error(PSATD_EINVAL, "psatd_mlp_get: NULL plan");
  if (hipDeviceSynchronize() != hipSuccess) return hip_fail("psatd_mlp_get");
  if (master && hipMemcpy(master, p->master, sizeof(float) * NPARAM, hipMemcpyDeviceToHost) != hipSuccess)
    return hip_fail("psatd_mlp_get master");
  if (bf16 && hipMemcpy(bf16, p->wbf, sizeof(uint16_t) * NPARAM, hipMemcpyDeviceToHost) != hipSuccess)
    return hip_fail("psatd_mlp_get bf16");
  return PSATD_OK;
}

int psatd_mlp_predict(const psatd_mlp* p, const float* X, int n, float* y, void* stream) {
  if (!p || (n > 0 && (!X || !y))) return report_error(PSATD_EINVAL, "psatd_mlp_predict: NULL argument");
  if (n < 0) return report_error(PSATD_EINVAL, "psatd_mlp_predict: n = %d", n);
  if (n == 0) return PSATD_OK;
  k_mlp_forward<<<std::min(nblocks(n, TS), kForwardBlocks), NT, 0, (hipStream_t)stream>>>(p->wbf, X, n, y, p->nm);
  return hip_fail("psatd_mlp_predict");
}

int psatd_mlp_grad(psatd_mlp* p, const float* X, const float* t, int n, const int* idx, int batch, float* grad,
                   float* loss, void* stream) {
  if (!p || !X || !t) return report_error(PSATD_EINVAL, "psatd_mlp_grad: NULL argument");
  if (n < 1 || batch < 1 || batch > p->max_batch || (!idx && batch > n))
    return report_error(PSATD_EINVAL, "psatd_mlp_grad: n = %d, batch = %d (max %d)", n, batch, p->max_batch);
  hipStream_t s = (hipStream_t)stream;
  enqueue_grad(p, X, t, n, idx, batch, grad, loss, s);
  return hip_fail("psatd_mlp_grad");
}

int psatd_mlp_adam(psatd_mlp* p, float lr, float beta1, float beta2, float eps, void* stream) {
  if (!p) return report_error(PSATD_EINVAL, "psatd_mlp_adam: NULL plan");
  if (!adam_args_ok(lr, beta1, beta2, eps)) return report_error(PSATD_EINVAL, "psatd_mlp_adam: bad hyperparameters");
  enqueue_adam(p, lr, beta1, beta2, eps, (hipStream_t)stream);
  return hip_fail("psatd_mlp_adam");
}

int psatd_mlp_train(psatd_mlp* p, const float* X, const float* t, int n, const int* idx, int nsteps, int batch,
                    float lr, float beta1, float beta2, float eps, float* loss_hist, void* stream) {
  if (!p || !X || !t) return report_error(PSATD_EINVAL, "psatd_mlp_train: NULL argument");
  if (n < 1 || nsteps < 0 || batch < 1 || batch > p->max_batch || (!idx && batch > n))
    return report_error(PSATD_EINVAL, "psatd_mlp_train: n = %d, nsteps = %d, batch = %d (max %d)", n, nsteps, batch,
                        p->max_batch);
  if (!adam_args_ok(lr, beta1, beta2, eps)) return report_error(PSATD_EINVAL, "psatd_mlp_train: bad hyperparameters");
  hipStream_t s = (hipStream_t)stream;
  for (int k = 0; k < nsteps; ++k) {
    enqueue_grad(p, X, t, n, idx ? idx + (size_t)k * batch : nullptr, batch, nullptr,
                 loss_hist ? loss_hist + k : nullptr, s);
    enqueue_adam(p, lr, beta1, beta2, eps, s);
  }
  return hip_fail("psatd_mlp_train");
}

void psatd_mlp_destroy(psatd_mlp* p) { free_mlp(p); }

}  // extern "C"
