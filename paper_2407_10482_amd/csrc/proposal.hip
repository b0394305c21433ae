// Learned per-ray sample-interval proposal (an extension beyond the paper).
//
// Network: r = [o; d] -> Fourier features sin/cos(2^k pi r_j), k = 0..3 (48)
// -> 64 -> 64 -> 4 (ReLU hidden), outputs t_near, t_far, t_term and a
// confidence logit.  Parameters (float32 master, caller-owned, 7556 values):
// W1[64][48], b1[64], W2[64][64], b2[64], W3[4][64], b3[4].
//
// Every product is a 16x16 tile of v_mfma_f32_16x16x16_bf16 (bfloat16
// operands, float32 accumulation).  Training: a workgroup owns 64 rays, each of
// its four waves runs 16 of them through the network and back with the
// activations and gradients chained in registers (as proposal_net.h), then the
// waves share the weight gradients, products with K = the workgroup's rays of
// operands left in LDS.  Per-workgroup gradient partials are summed in a fixed
// order; the last kernel also applies Adam to the float32 master copy.
#include <hip/hip_runtime.h>

#include <cmath>

#include "device.h"
#include "internal.h"
#include "proposal_net.h"
#include "reduce.h"

namespace ngprt {

constexpr int kPIn = 48, kPH = 64, kPOut = 4;
constexpr int kPW1 = 0, kPB1 = 3072, kPW2 = 3136, kPB2 = 7232, kPW3 = 7296, kPB3 = 7552;
constexpr int kPParams = 7556;
constexpr int kPPartial = kPParams + 1;          // + loss

// Operand tiles of the backward products beside the kPropTiles of the forward:
// W3^T (m) at kPropTiles + m, W2^T (m, kc) at kPropTiles + 4 + 4 m + kc; tile t,
// lane l: W3[4 (l / 16) + e][16 m + l % 16] (rows past the 4 outputs zero) and
// W2[16 kc + 4 (l / 16) + e][16 m + l % 16], e = 0..3.
constexpr int kPropTrainTiles = kPropTiles + 4 + 16;

// Float32 master weights -> the A-operand tiles and biases of
// prop_infer_wave (proposal_net.h): 32 tiles x 64 lanes of four bfloat16,
// then b1, b2, b3 as float32 (NULL: not wanted).  n_tiles = kPropTrainTiles: the
// backward's tiles too.
__global__ void prop_arrange_kernel(const float* __restrict__ P, uint2* __restrict__ tiles, int n_tiles,
                                    float* __restrict__ bias) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= kPropTiles * 64 && t < n_tiles * 64) {
    const int tile = (t >> 6) - kPropTiles, lane = t & 63;
    const int i = lane & 15, k0 = 4 * (lane >> 4);
    uint16_t h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (tile < 4) {
        h[e] = k0 + e < kPOut ? bf16_rne(P[kPW3 + (k0 + e) * kPH + 16 * tile + i]) : (uint16_t)0;
      } else {
        const int m = (tile - 4) >> 2, kc = (tile - 4) & 3;
        h[e] = bf16_rne(P[kPW2 + (16 * kc + k0 + e) * kPH + 16 * m + i]);
      }
    }
    tiles[t] = make_uint2(uint32_t(h[0]) | (uint32_t(h[1]) << 16), uint32_t(h[2]) | (uint32_t(h[3]) << 16));
  }
  if (t < kPropTiles * 64) {
    const int tile = t >> 6, lane = t & 63;
    const int i = lane & 15, k0 = 4 * (lane >> 4);
    int base, row, col, ld;
    bool zero = false;
    if (tile < 12) {             // layer 1: W1[64][48]
      base = kPW1; ld = kPIn; row = 16 * (tile / 3) + i; col = 16 * (tile % 3) + k0;
    } else if (tile < 28) {      // layer 2: W2[64][64]
      const int q = tile - 12;
      base = kPW2; ld = kPH; row = 16 * (q / 4) + i; col = 16 * (q % 4) + k0;
    } else {                     // layer 3: W3[4][64], rows 4..15 zero
      base = kPW3; ld = kPH; row = i; col = 16 * (tile - 28) + k0;
      zero = i >= kPOut;
    }
    uint16_t h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = zero ? (uint16_t)0 : bf16_rne(P[base + (zero ? 0 : row) * ld + col + e]);
    tiles[t] = make_uint2(uint32_t(h[0]) | (uint32_t(h[1]) << 16), uint32_t(h[2]) | (uint32_t(h[3]) << 16));
  }
  if (bias && t < kPropBias) bias[t] = t < 64 ? P[kPB1 + t] : (t < 128 ? P[kPB2 + t - 64] : P[kPB3 + t - 128]);
}

// Stand-alone inference: four waves per workgroup, one wave per 64 rays.
__global__ void __launch_bounds__(256) prop_infer_kernel(int64_t n, const float* __restrict__ O,
                                                         const float* __restrict__ D,
                                                         const uint2* __restrict__ tiles,
                                                         const float* __restrict__ bias,
                                                         float* __restrict__ out) {
  __shared__ float out4_all[4][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t ray_base = (int64_t(blockIdx.x) * 4 + wave) * 64;
  prop_infer_wave(tiles, bias, O, D, ray_base, n, lane, out4_all[wave]);
  __syncthreads();
  const int64_t ray = ray_base + lane;
  if (ray < n) {
#pragma unroll
    for (int c = 0; c < 4; ++c) out[ray * 4 + c] = out4_all[wave][4 * lane + c];
  }
}

// LDS of a workgroup in training, feature-major ([feature][ray], bfloat16), so
// that the weight gradients' operands are four consecutive rays; the row pitch
// spreads the four lane groups of a store over the banks.
constexpr int kRP = 68;
struct PropLds {
  uint16_t enc[kPIn * kRP];
  uint16_t h1[kPH * kRP];
  uint16_t h2[kPH * kRP];
  uint16_t gz2[kPH * kRP];
  uint16_t gz1[kPH * kRP];
  uint16_t gout[16 * kRP];     // rows 4..15 zero
  float sums[4][2 * kPH + 5];  // per wave: db2, db1, db3, loss
};

// sum over the 16 lanes that share (lane >> 4)
__device__ __forceinline__ float sum16(float v) {
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// bfloat16 v[e] of rows row0 + e to column `ray`
__device__ __forceinline__ void put_rows(uint16_t* a, int row0, int ray, pn_bf16x4 v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) a[(row0 + e) * kRP + ray] = (uint16_t)v[e];
}

// four consecutive rays of one row, an operand of the weight gradients
__device__ __forceinline__ pn_bf16x4 rays4(const uint16_t* a, int row, int ray) {
  return *reinterpret_cast<const pn_bf16x4*>(a + row * kRP + ray);
}

// D = sum over the 64 rays of A[i][ray] B[j][ray], rows ra + i of A, rb + j of B
__device__ __forceinline__ pn_f32x4 outer_rays(const uint16_t* A, int ra, const uint16_t* B, int rb, int lane) {
  const int i = lane & 15, s = lane >> 4;
  pn_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < 4; ++kc)
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(rays4(A, ra + i, 16 * kc + 4 * s),
                                                    rays4(B, rb + i, 16 * kc + 4 * s), acc, 0, 0, 0);
  return acc;
}

// Labels [n][4]: t_near, t_far, t_term, valid (1/0).  phase 1: pinball
// losses on t_near (quantile 0.05) and t_far (0.95), squared error on t_term;
// phase >= 2: + confidence cross-entropy with target = valid and
// [out0 - margin, out1 + margin] contains [t_near, t_far].  Loss terms are
// divided by n (the batch).
// Bound by the latency of its chain of small products (2^14 rays are 256
// workgroups, one a CU): a wave of 64 rays with every operand gathered from LDS
// by 2-byte reads took 36.8 us, four waves of 16 rays with the products chained
// in registers 16.7 us.
__global__ void __launch_bounds__(256) prop_train_kernel(int64_t n, const float* __restrict__ O,
                                                         const float* __restrict__ D,
                                                         const float* __restrict__ labels, int phase, float margin,
                                                         const float* __restrict__ P,
                                                         const uint2* __restrict__ tiles,
                                                         float* __restrict__ partial) {
  __shared__ __align__(16) PropLds L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, s = lane >> 4;
  const int col = 16 * wave + j;                            // this lane's ray in the workgroup
  const int64_t ray = int64_t(blockIdx.x) * 64 + col;
  const bool in_range = ray < n;
  float* part = partial + int64_t(blockIdx.x) * kPPartial;
  // forward (the operand layout is prop_infer_wave's)
  pn_bf16x4 enc[3], h1[4], h2[4];
#pragma unroll
  for (int kc = 0; kc < 3; ++kc) {
    const int comp = 2 * kc + (s >> 1);
    const float* src = comp < 3 ? O : D;
    const float r = in_range ? src[3 * (in_range ? ray : 0) + (comp < 3 ? comp : comp - 3)] : 0.0f;
    const int k0 = 2 * (s & 1);
    const float a0 = float(1 << k0) * r, a1 = float(2 << k0) * r;
    enc[kc] = pn_pack(sinpif(a0), cospif(a0), sinpif(a1), cospif(a1));
    put_rows(L.enc, 16 * kc + 4 * s, col, enc[kc]);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    pn_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 3; ++kc)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pn_tile(tiles, m * 3 + kc, lane), enc[kc], acc, 0, 0, 0);
    const float* b = P + kPB1 + 16 * m + 4 * s;
    h1[m] = pn_pack(fmaxf(acc[0] + b[0], 0.0f), fmaxf(acc[1] + b[1], 0.0f), fmaxf(acc[2] + b[2], 0.0f),
                    fmaxf(acc[3] + b[3], 0.0f));
    put_rows(L.h1, 16 * m + 4 * s, col, h1[m]);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    pn_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pn_tile(tiles, 12 + m * 4 + kc, lane), h1[kc], acc, 0, 0, 0);
    const float* b = P + kPB2 + 16 * m + 4 * s;
    h2[m] = pn_pack(fmaxf(acc[0] + b[0], 0.0f), fmaxf(acc[1] + b[1], 0.0f), fmaxf(acc[2] + b[2], 0.0f),
                    fmaxf(acc[3] + b[3], 0.0f));
    put_rows(L.h2, 16 * m + 4 * s, col, h2[m]);
  }
  pn_f32x4 out = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < 4; ++kc)
    out = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pn_tile(tiles, 28 + kc, lane), h2[kc], out, 0, 0, 0);

  // loss and dL/dout: the four outputs of a ray are in lane j of the first 16
  const float inv_n = 1.0f / float(n);
  float go[4] = {0.f, 0.f, 0.f, 0.f};
  float loss = 0.0f;
  if (s == 0 && in_range) {
    const float* y = labels + ray * 4;
    const bool valid = y[3] != 0.0f;
    float ov[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) ov[c] = out[c] + P[kPB3 + c];
    if (valid) {
      // t_near: pinball loss at quantile 0.05; t_far: at 0.95; t_term: squared error
      const float r0 = y[0] - ov[0], r1 = y[1] - ov[1], df = ov[2] - y[2];
      loss += (r0 >= 0.0f ? 0.05f * r0 : -0.95f * r0) + (r1 >= 0.0f ? 0.95f * r1 : -0.05f * r1) + df * df;
      go[0] = (ov[0] > y[0] ? 0.95f : -0.05f) * inv_n;
      go[1] = (ov[1] > y[1] ? 0.05f : -0.95f) * inv_n;
      go[2] = 2.0f * df * inv_n;
    }
    if (phase >= 2) {
      const float tgt = (valid && ov[0] - margin <= y[0] && ov[1] + margin >= y[1]) ? 1.0f : 0.0f;
      const float sg = 1.0f / (1.0f + __expf(-ov[3]));
      loss += -(tgt * __logf(sg + 1e-12f) + (1.0f - tgt) * __logf(1.0f - sg + 1e-12f));
      go[3] = (sg - tgt) * inv_n;
    }
  }
  float* sums = L.sums[wave];
  {
    const float ls = sum16(loss * inv_n);
    float b3[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) b3[c] = sum16(go[c]);
    if (lane == 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c) sums[2 * kPH + c] = b3[c];
      sums[2 * kPH + 4] = ls;
    }
  }
  // B operand of the first backward product: rows 4 s + e, of which 0..3 hold
  // dL/dout (zero on the lanes of s > 0, as go is)
  const pn_bf16x4 gout = pn_pack(go[0], go[1], go[2], go[3]);
  put_rows(L.gout, 4 * s, col, gout);
  // gz2 = (W3^T gout) * [h2 > 0], gz1 = (W2^T gz2) * [h1 > 0]
  pn_bf16x4 gz2[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    pn_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pn_tile(tiles, kPropTiles + m, lane), gout, acc, 0, 0, 0);
    float g[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      g[q] = bf16_to_f32((uint16_t)h2[m][q]) > 0.0f ? acc[q] : 0.0f;
      const float t = sum16(g[q]);
      if (j == 0) sums[16 * m + 4 * s + q] = t;
    }
    gz2[m] = pn_pack(g[0], g[1], g[2], g[3]);
    put_rows(L.gz2, 16 * m + 4 * s, col, gz2[m]);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    pn_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pn_tile(tiles, kPropTiles + 4 + 4 * m + kc, lane), gz2[kc], acc,
                                                      0, 0, 0);
    float g[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      g[q] = bf16_to_f32((uint16_t)h1[m][q]) > 0.0f ? acc[q] : 0.0f;
      const float t = sum16(g[q]);
      if (j == 0) sums[kPH + 16 * m + 4 * s + q] = t;
    }
    put_rows(L.gz1, 16 * m + 4 * s, col, pn_pack(g[0], g[1], g[2], g[3]));
  }
  __syncthreads();
  // weight gradients: wave w takes row block w of dW2 and dW1, column block w of dW3
  {
    const pn_f32x4 r = outer_rays(L.gout, 0, L.h2, 16 * wave, lane);
    if (s == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) part[kPW3 + q * kPH + 16 * wave + j] = r[q];
    }
  }
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const pn_f32x4 r = outer_rays(L.gz2, 16 * wave, L.h1, 16 * nt, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) part[kPW2 + (16 * wave + 4 * s + q) * kPH + 16 * nt + j] = r[q];
  }
#pragma unroll
  for (int nt = 0; nt < 3; ++nt) {
    const pn_f32x4 r = outer_rays(L.gz1, 16 * wave, L.enc, 16 * nt, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) part[kPW1 + (16 * wave + 4 * s + q) * kPIn + 16 * nt + j] = r[q];
  }
  // the biases' and the loss's sums over the four waves
  const int t = int(threadIdx.x);
  if (t < 2 * kPH + 5) {
    const float a = (L.sums[0][t] + L.sums[1][t]) + (L.sums[2][t] + L.sums[3][t]);
    part[t < kPH ? kPB2 + t : (t < 2 * kPH ? kPB1 + t - kPH : (t < 2 * kPH + 4 ? kPB3 + t - 2 * kPH : kPParams))] = a;
  }
}

// The groups' sums in order, the loss, and Adam on the float32 weights when m
// and v are given (the update of adam_kernel).
__global__ void prop_finish_kernel(const float* __restrict__ tmp, float* __restrict__ grad, float* __restrict__ loss,
                                   float* __restrict__ p, float* __restrict__ m, float* __restrict__ v, float lr,
                                   float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kPPartial) return;
  float a = 0.0f;
#pragma unroll 16
  for (int g = 0; g < kSumGroups; ++g) a += tmp[int64_t(g) * kPPartial + i];
  if (i == kPParams) {
    if (loss) loss[0] += a;
    return;
  }
  if (grad) grad[i] = a;
  if (m) {
    const float mi = b1 * m[i] + (1.0f - b1) * a;
    const float vi = b2 * v[i] + (1.0f - b2) * a * a;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
  }
}

static int ensure_prop_buffers(ngprt_ctx* ctx, int64_t n_parts, hipStream_t st) {
  if (!ctx->prop_wb &&
      dev_malloc_async((void**)&ctx->prop_wb, size_t(kPropTrainTiles) * 64 * sizeof(uint2), st) != hipSuccess) {
    (void)hipGetLastError();
    return fail(ctx, NGPRT_E_ALLOC, "proposal buffers");
  }
  const size_t need = size_t(n_parts + kSumGroups) * kPPartial * sizeof(float);
  if (need > ctx->ws_bytes) {
    if (ctx->ws) (void)hipFreeAsync(ctx->ws, st);
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
    if (dev_malloc_async((void**)&ctx->ws, need, st) != hipSuccess) {
      (void)hipGetLastError();
      return fail(ctx, NGPRT_E_ALLOC, "proposal workspace");
    }
    ctx->ws_bytes = need;
  }
  return NGPRT_OK;
}

constexpr size_t kPropNetBytes = size_t(kPropTiles) * 64 * sizeof(uint2) + kPropBias * sizeof(float);

// dst: kPropNetBytes of device memory (tiles, then biases)
int launch_prop_arrange(ngprt_ctx* ctx, const float* P, void* dst, hipStream_t st) {
  uint2* tiles = reinterpret_cast<uint2*>(dst);
  float* bias = reinterpret_cast<float*>(reinterpret_cast<char*>(dst) + size_t(kPropTiles) * 64 * sizeof(uint2));
  hipLaunchKernelGGL(prop_arrange_kernel, dim3((kPropTiles * 64 + 255) / 256), dim3(256), 0, st, P, tiles,
                     kPropTiles, bias);
  return check_launch(ctx, "prop_arrange_kernel");
}

int launch_prop_infer(ngprt_ctx* ctx, int64_t n, const float* o, const float* d, const float* P, float* out,
                      hipStream_t st) {
  if (!ctx->prop_tmp && dev_malloc((void**)&ctx->prop_tmp, kPropNetBytes) != hipSuccess) {
    (void)hipGetLastError();
    ctx->prop_tmp = nullptr;
    return fail(ctx, NGPRT_E_ALLOC, "proposal inference weights");
  }
  int rc = launch_prop_arrange(ctx, P, ctx->prop_tmp, st);
  if (rc) return rc;
  const int64_t blocks = (n + 255) / 256;
  if (blocks > 0x7FFFFFFF) return fail(ctx, NGPRT_E_SHAPE, "too many rays");
  const uint2* tiles = reinterpret_cast<const uint2*>(ctx->prop_tmp);
  const float* bias = reinterpret_cast<const float*>(reinterpret_cast<const char*>(ctx->prop_tmp) +
                                                     size_t(kPropTiles) * 64 * sizeof(uint2));
  hipLaunchKernelGGL(prop_infer_kernel, dim3(unsigned(blocks)), dim3(256), 0, st, n, o, d, tiles, bias, out);
  return check_launch(ctx, "prop_infer_kernel");
}

int load_proposal(ngprt_ctx* ctx, const float* P, hipStream_t st) {
  if (!ctx->prop_net && dev_malloc((void**)&ctx->prop_net, kPropNetBytes) != hipSuccess) {
    (void)hipGetLastError();
    ctx->prop_net = nullptr;
    return fail(ctx, NGPRT_E_ALLOC, "proposal network");
  }
  int rc = launch_prop_arrange(ctx, P, ctx->prop_net, st);
  if (rc) return rc;
  ctx->prop_loaded = true;
  return NGPRT_OK;
}

int launch_prop_train(ngprt_ctx* ctx, int64_t n, const float* o, const float* d, const float* labels,
                      int phase, float margin, float* P, float* m, float* v, int32_t step, float lr,
                      float* loss, float* grad_out, hipStream_t st) {
  const int64_t blocks = (n + 63) / 64;
  if (blocks > (int64_t(1) << 24)) return fail(ctx, NGPRT_E_SHAPE, "batch too large");
  int rc = ensure_prop_buffers(ctx, blocks, st);
  if (rc) return rc;
  uint2* tiles = reinterpret_cast<uint2*>(ctx->prop_wb);
  hipLaunchKernelGGL(prop_arrange_kernel, dim3((kPropTrainTiles * 64 + 255) / 256), dim3(256), 0, st, P, tiles,
                     kPropTrainTiles, nullptr);
  if ((rc = check_launch(ctx, "prop_arrange_kernel"))) return rc;
  float* partial = reinterpret_cast<float*>(ctx->ws);
  hipLaunchKernelGGL(prop_train_kernel, dim3(unsigned(blocks)), dim3(256), 0, st, n, o, d, labels, phase, margin, P,
                     tiles, partial);
  if ((rc = check_launch(ctx, "prop_train_kernel"))) return rc;
  // one thread a parameter over all partials took 59 us at 2^14 rays; 64 groups
  // of partials, then the groups, 8 us with Adam
  float* tmp = partial + size_t(blocks) * kPPartial;
  hipLaunchKernelGGL(partial_group_sums_kernel, dim3((kPPartial + 255) / 256, kSumGroups), dim3(256), 0, st, partial,
                     blocks, kPPartial, tmp);
  if ((rc = check_launch(ctx, "partial_group_sums_kernel"))) return rc;
  const bool adam = m && v;
  const double c1 = adam ? 1.0 / (1.0 - std::pow(double(0.9f), double(step))) : 1.0;
  const double c2 = adam ? 1.0 / (1.0 - std::pow(double(0.99f), double(step))) : 1.0;
  hipLaunchKernelGGL(prop_finish_kernel, dim3((kPPartial + 255) / 256), dim3(256), 0, st, tmp, grad_out, loss, P,
                     adam ? m : nullptr, adam ? v : nullptr, lr, 0.9f, 0.99f, 1e-8f, float(c1), float(c2));
  return check_launch(ctx, "prop_finish_kernel");
}

}  // namespace ngprt
