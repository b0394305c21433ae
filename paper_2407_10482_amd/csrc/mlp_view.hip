// View-dependent deferred MLP (Eq. 5; supplement "Network Design"):
// C = sigmoid(C_d + MLP_psi(C_d, F, SH(d))), MLP_psi 23 -> 64 -> 64 -> 3 with
// ReLU hidden layers, SH(d) the 16 real spherical harmonics of degrees 0..3
// of the normalised view direction.
//
// A separate pass after the march: the render kernel leaves C_d and F in the
// caller's output buffers, and this kernel runs the MLP over all rays.  One
// workgroup = 16 waves sharing one copy of the weights, pre-arranged at load
// time in the order the MFMA sequence consumes them (one 64-float record per
// instruction, lane l reading element l), staged once per workgroup in LDS
// (35 KB); the grid holds only as many workgroups as stay resident together,
// each wave taking groups of 16 rays in turn.  Every layer is a chain of
// v_mfma_f32_16x16x4f32 with the hidden units as rows and the 16 rays as
// columns: four lanes share a ray, lane (ray i, slot s) giving input 4 c + s of
// chunk c from its registers; the hidden index handed to the next layer is
// permuted (k-slot s of chunk (m, r) = unit 16 m + 4 s + r) so each layer
// consumes the previous accumulators in place.
// What bounds it: the matrix pipe, 104 instructions of 32 cycles per 16 rays,
// once every SIMD has waves; 16 rays a wave rather than 64 let 66,105 rays reach
// all 256 CUs instead of 65 of them.  Measured, 64 rays a wave
// against this: 66,105 rays 32.4 -> 20.1 us; 2.07 M rays 266 -> 265 us (176 us of
// matrix instructions).
#include <hip/hip_runtime.h>

#include "internal.h"
#include "reduce.h"

namespace ngprt {

typedef float f32x4v __attribute__((ext_vector_type(4)));

// MFMA operand records: layer 1 (4 output blocks x 6 K-chunks), layer 2
// (4 output blocks x 16 chunks), layer 3 (16 chunks), then the biases laid
// out per lane: b0 [4 blocks][64 lanes][4], b1 likewise, b2 [64 lanes][4].
// The backward's transposed products follow: W2^T (4 output blocks, one chunk),
// W1^T (4 output blocks x 16 chunks), W0^T (16 chunks, its 7 rows of C_d and F).
constexpr int kL1Rec = 4 * 6, kL2Rec = 4 * 16, kL3Rec = 16;
constexpr int kViewFwdFloats = (kL1Rec + kL2Rec + kL3Rec) * 64 + (4 + 4 + 1) * 64 * 4;   // 8960
constexpr int kT2Rec = 4, kT1Rec = 4 * 16, kT0Rec = 16;
constexpr int kViewRecFloats = kViewFwdFloats + (kT2Rec + kT1Rec + kT0Rec) * 64;         // 14336
static_assert(kViewRecFloats == kMlpViewRec, "record size");

// Rearrange the flattened parameters W0[64][23], b0[64], W1[64][64], b1[64],
// W2[3][64], b2[3] into the MFMA records (one thread per record float).
__global__ void view_mlp_arrange_kernel(const float* __restrict__ P, float* __restrict__ rec) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= kViewRecFloats) return;
  const float* W0 = P;
  const float* b0 = W0 + 64 * 23;
  const float* W1 = b0 + 64;
  const float* b1 = W1 + 64 * 64;
  const float* W2 = b1 + 64;
  const float* b2 = W2 + 3 * 64;
  const int lane = t & 63, i = lane & 15, s = lane >> 4;
  int rix = t >> 6;
  float v = 0.0f;
  if (rix < kL1Rec) {                                    // layer 1: (mo, c)
    const int mo = rix / 6, c = rix % 6, k = 4 * c + s;
    v = k < 23 ? W0[(mo * 16 + i) * 23 + k] : 0.0f;
  } else if ((rix -= kL1Rec) < kL2Rec) {                 // layer 2: (mo, m, r)
    const int mo = rix / 16, m = (rix / 4) % 4, r = rix % 4;
    v = W1[(mo * 16 + i) * 64 + m * 16 + 4 * s + r];
  } else if ((rix -= kL2Rec) < kL3Rec) {                 // layer 3: (m, r)
    const int m = rix / 4, r = rix % 4;
    v = i < 3 ? W2[i * 64 + m * 16 + 4 * s + r] : 0.0f;
  } else if (t >= kViewFwdFloats) {                      // transposed products
    rix = (t - kViewFwdFloats) >> 6;
    if (rix < kT2Rec) {                                  // W2^T: (mo)
      v = s < 3 ? W2[s * 64 + rix * 16 + i] : 0.0f;
    } else if ((rix -= kT2Rec) < kT1Rec) {               // W1^T: (mo, m, r)
      const int mo = rix / 16, m = (rix / 4) % 4, r = rix % 4;
      v = W1[(m * 16 + 4 * s + r) * 64 + mo * 16 + i];
    } else {                                             // W0^T: (m, r)
      rix -= kT1Rec;
      const int m = rix / 4, r = rix % 4;
      v = i < 7 ? W0[(m * 16 + 4 * s + r) * 23 + i] : 0.0f;
    }
  } else {                                               // biases per lane
    const int b = t - (kL1Rec + kL2Rec + kL3Rec) * 64;   // [9][64][4]
    const int blk = b / 256, ln = (b / 4) % 64, r = b % 4, unit = 4 * (ln >> 4) + r;
    if (blk < 4) v = b0[blk * 16 + unit];
    else if (blk < 8) v = b1[(blk - 4) * 16 + unit];
    else v = unit < 3 ? b2[unit] : 0.0f;
  }
  rec[t] = v;
}

__device__ __forceinline__ void sh16(float x, float y, float z, float* Y) {
  // real spherical harmonics, degrees 0..3 (orthonormal, no Condon-Shortley phase)
  const float c0 = 0.28209479177387814f;                 // 1/2 sqrt(1/pi)
  const float c1 = 0.4886025119029199f;                  // sqrt(3/(4 pi))
  const float c2a = 1.0925484305920792f;                 // 1/2 sqrt(15/pi)
  const float c2b = 0.31539156525252005f;                // 1/4 sqrt(5/pi)
  const float c2c = 0.5462742152960396f;                 // 1/4 sqrt(15/pi)
  const float c3a = 0.5900435899266435f;                 // 1/4 sqrt(35/(2 pi))
  const float c3b = 2.890611442640554f;                  // 1/2 sqrt(105/pi)
  const float c3c = 0.4570457994644658f;                 // 1/4 sqrt(21/(2 pi))
  const float c3d = 0.3731763325901154f;                 // 1/4 sqrt(7/pi)
  const float c3e = 1.445305721320277f;                  // 1/4 sqrt(105/pi)
  const float xx = x * x, yy = y * y, zz = z * z;
  Y[0] = c0;
  Y[1] = c1 * y; Y[2] = c1 * z; Y[3] = c1 * x;
  Y[4] = c2a * x * y; Y[5] = c2a * y * z; Y[6] = c2b * (3.0f * zz - 1.0f);
  Y[7] = c2a * x * z; Y[8] = c2c * (xx - yy);
  Y[9] = c3a * y * (3.0f * xx - yy); Y[10] = c3b * x * y * z; Y[11] = c3c * y * (5.0f * zz - 1.0f);
  Y[12] = c3d * z * (5.0f * zz - 3.0f); Y[13] = c3c * x * (5.0f * zz - 1.0f);
  Y[14] = c3e * z * (xx - yy); Y[15] = c3a * x * (xx - 3.0f * yy);
}

// orders a wave's LDS accesses; also keeps a loop's loads in the loop
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

constexpr int kViewWaves = 16;                    // waves per workgroup of view_mlp_kernel

// Inputs of a ray at its slot s: x[c] = input 4 c + s of (C_d, F, SH, 0); c_d
// and f the ray's own.  Zero for rays out of range and directions without one.
__device__ __forceinline__ void view_inputs(bool ok, int64_t ray, int s, const float* __restrict__ D,
                                            const float* __restrict__ c_d, const float* __restrict__ feat,
                                            float cd[3], float x[6]) {
  float v[24];
#pragma unroll
  for (int j = 0; j < 24; ++j) v[j] = 0.0f;
  if (ok) {
#pragma unroll
    for (int j = 0; j < 3; ++j) v[j] = c_d[ray * 3 + j];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[3 + j] = feat[ray * 4 + j];
    const float d0 = D[ray * 3], d1 = D[ray * 3 + 1], d2 = D[ray * 3 + 2];
    const float nn = sqrtf((d0 * d0 + d1 * d1) + d2 * d2);
    if (nn > 0.0f && isfinite(nn)) sh16(d0 / nn, d1 / nn, d2 / nn, v + 7);
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) cd[j] = v[j];
  // by masks: a choice of array elements would become an indexed load
  const uint32_t odd = uint32_t(-(s & 1)), high = uint32_t(-(s >> 1));
  auto pick = [](uint32_t m, float a, float b) {
    return __uint_as_float((__float_as_uint(a) & ~m) | (__float_as_uint(b) & m));
  };
#pragma unroll
  for (int c = 0; c < 6; ++c)
    x[c] = pick(high, pick(odd, v[4 * c], v[4 * c + 1]), pick(odd, v[4 * c + 2], v[4 * c + 3]));
}

// The forward of 16 rays: activations h1, h2 (unit 16 m + 4 s + r of lane
// (i, s) at [m][r]) and, at the lanes of slot 0, the outputs before the
// addition of C_d in o[0..2].  W: the forward's records in LDS.
__device__ __forceinline__ void view_forward(const float* W, const float x[6], int lane, float h1[4][4],
                                             float h2[4][4], float o[3]) {
  const float* R1 = W;
  const float* R2 = W + kL1Rec * 64;
  const float* R3 = R2 + kL2Rec * 64;
  const float* B = R3 + kL3Rec * 64;
#pragma unroll
  for (int mo = 0; mo < 4; ++mo) {
    f32x4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 6; ++c)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(R1[(mo * 6 + c) * 64 + lane], x[c], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) h1[mo][r] = fmaxf(acc[r] + B[(mo * 64 + lane) * 4 + r], 0.0f);
  }
#pragma unroll
  for (int mo = 0; mo < 4; ++mo) {
    f32x4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(R2[((mo * 4 + m) * 4 + r) * 64 + lane], h1[m][r], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) h2[mo][r] = fmaxf(acc[r] + B[((4 + mo) * 64 + lane) * 4 + r], 0.0f);
  }
  f32x4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(R3[(m * 4 + r) * 64 + lane], h2[m][r], acc, 0, 0, 0);
#pragma unroll
  for (int j = 0; j < 3; ++j) o[j] = acc[j] + B[(8 * 64 + lane) * 4 + j];
}

__global__ void __launch_bounds__(64 * kViewWaves) view_mlp_kernel(int64_t n, const float* __restrict__ D,
                                                       const float* __restrict__ c_d,
                                                       const float* __restrict__ feat,
                                                       const float* __restrict__ rec,
                                                       float* __restrict__ rgb) {
  __shared__ float W[kViewFwdFloats];
  for (int t = threadIdx.x; t < kViewFwdFloats; t += 64 * kViewWaves) W[t] = rec[t];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, s = lane >> 4;
  const int64_t groups = (n + 15) / 16;
  for (int64_t g = int64_t(blockIdx.x) * kViewWaves + wave; g < groups; g += int64_t(gridDim.x) * kViewWaves) {
    const int64_t ray = g * 16 + i;
    wave_lds_fence();                             // the weights do not fit the registers
    float cd[3], x[6], h1[4][4], h2[4][4], o[3];
    view_inputs(ray < n, ray, s, D, c_d, feat, cd, x);
    view_forward(W, x, lane, h1, h2, o);
    if (s == 0 && ray < n) {
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const float z = cd[j] + o[j];
        rgb[ray * 3 + j] = 1.0f / (1.0f + __expf(-z));
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Backward of the view-dependent MLP (a training extension).  A wave takes 16
// rays at a time like the forward, whose pass it repeats: gz = dL/drgb * rgb (1 -
// rgb), g2 = (W2^T gz) masked, g1 = (W1^T g2) masked, dL/dC_d = gz + (W0^T
// g1)[0..2], dL/dF = (W0^T g1)[3..6], each product on v_mfma_f32_16x16x4f32
// with the units as rows and the rays as columns, in registers throughout.  The
// weight gradients are sums over rays of outer products, with the rays as K:
// their operands hold a unit a lane where the products above leave a ray a
// lane, so each is transposed through 5 KB of LDS a wave (rows of 20 floats:
// both the stores and the 16-byte loads spread over all banks; slot s takes rays
// 4 s .. 4 s + 3, in both operands).  The sums stay in 117 accumulators a lane over
// all rays of a wave, then a workgroup's eight waves are added in a fixed order
// and written as one 5891-float partial; the partials are added in a fixed
// order too (reduce.h).  A constant input of 1 (weight 0) gives db0.
// What bounds it: the matrix pipe, 300 instructions of 32 cycles per 16 rays; the
// 57 KB of weights a workgroup stages are read once a workgroup, as many as
// stay resident together.  Measured, a lane a ray with its dot
// products on the vector unit, a workgroup and a partial each 64 rays, against
// this: 66,105 rays 154 -> 48 us.
constexpr int kViewBwdWaves = 8;                         // waves per workgroup of the backward
constexpr int kVP = 20;                                  // LDS row pitch of the transposes
constexpr int kW0 = 0, kB0 = 64 * 23, kW1 = kB0 + 64, kB1 = kW1 + 64 * 64, kW2 = kB1 + 64,
              kB2 = kW2 + 3 * 64;
static_assert(kB2 + 3 == kMlpViewParams, "parameter layout");
// the weights and the waves' transposes; at the end four copies of the sums
constexpr int kViewBwdFloats = kViewRecFloats + kViewBwdWaves * 64 * kVP;
static_assert(4 * kMlpViewParams <= kViewBwdFloats && kViewBwdWaves == 8, "four copies, two waves each");

// out[a][c] = v of unit 16 a + i at ray 4 s + c, for v[m][r] the value of unit
// 16 m + 4 s + r at ray i
__device__ __forceinline__ void view_transpose(float* T, const float v[4][4], int i, int s, float out[4][4]) {
  wave_lds_fence();
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) T[(16 * m + 4 * s + r) * kVP + i] = v[m][r];
  wave_lds_fence();
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const float4 q = *reinterpret_cast<const float4*>(T + (16 * a + i) * kVP + 4 * s);
    out[a][0] = q.x; out[a][1] = q.y; out[a][2] = q.z; out[a][3] = q.w;
  }
}

__global__ void __launch_bounds__(64 * kViewBwdWaves) view_mlp_backward_kernel(
    int64_t n, const float* __restrict__ D, const float* __restrict__ c_d, const float* __restrict__ feat,
    const float* __restrict__ grad_rgb, const float* __restrict__ rec, float* __restrict__ grad_cf,
    float* __restrict__ partial) {
  __shared__ __align__(16) float L[kViewBwdFloats];
  for (int t = threadIdx.x; t < kViewRecFloats; t += 64 * kViewBwdWaves) L[t] = rec[t];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, s = lane >> 4;
  float* T = L + kViewRecFloats + wave * 64 * kVP;
  const float* T2 = L + kViewFwdFloats;
  const float* T1 = T2 + kT2Rec * 64;
  const float* T0 = T1 + kT1Rec * 64;
  const f32x4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4v dW1[4][4], dW0[4][2], dW2[4];
  float db1[4], db2 = 0.0f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int b = 0; b < 4; ++b) dW1[a][b] = zero;
    dW0[a][0] = dW0[a][1] = dW2[a] = zero;
    db1[a] = 0.0f;
  }
  const int64_t groups = (n + 15) / 16;
  for (int64_t grp = int64_t(blockIdx.x) * kViewBwdWaves + wave; grp < groups;
       grp += int64_t(gridDim.x) * kViewBwdWaves) {
    const int64_t ray = grp * 16 + i;
    const bool ok = ray < n;
    float cd[3], x[6], h1[4][4], h2[4][4], o[3], g[3] = {0.0f, 0.0f, 0.0f};
    view_inputs(ok, ray, s, D, c_d, feat, cd, x);
    if (ok) {
#pragma unroll
      for (int j = 0; j < 3; ++j) g[j] = grad_rgb[ray * 3 + j];
    }
    view_forward(L, x, lane, h1, h2, o);
    // gz at the lanes of slot 0, then component s at slot s
    float gz[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float C = 1.0f / (1.0f + __expf(-(cd[c] + o[c])));
      gz[c] = __shfl(g[c] * C * (1.0f - C), i, 64);
    }
    const float gs = s == 0 ? gz[0] : (s == 1 ? gz[1] : (s == 2 ? gz[2] : 0.0f));
    // dW2 [3][64] = sum gz (x) a2 (rows: units, columns: components); db2
    float A[4][4], B[4][4];
    view_transpose(T, h2, i, s, A);
    wave_lds_fence();
    if (s < 3) T[s * kVP + i] = gs;
    wave_lds_fence();
    {
      const float4 q = *reinterpret_cast<const float4*>(T + i * kVP + 4 * s);   // rows 3 and on: columns not used
      const float Z[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int a = 0; a < 4; ++a) dW2[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[a][c], Z[c], dW2[a], 0, 0, 0);
        db2 += Z[c];
      }
    }
    // g2, over h2
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const f32x4v r4 = __builtin_amdgcn_mfma_f32_16x16x4f32(T2[m * 64 + lane], gs, zero, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[m][r] = h2[m][r] > 0.0f ? r4[r] : 0.0f;
    }
    // dW1 [64][64] = sum g2 (x) a1; db1
    view_transpose(T, h2, i, s, A);
    view_transpose(T, h1, i, s, B);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          dW1[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[a][c], B[b][c], dW1[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < 4; ++a) db1[a] += A[a][c];
    }
    // g1, over h1
    {
      f32x4v acc[4] = {zero, zero, zero, zero};
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int mo = 0; mo < 4; ++mo)
            acc[mo] = __builtin_amdgcn_mfma_f32_16x16x4f32(T1[((mo * 4 + m) * 4 + r) * 64 + lane], h2[m][r], acc[mo],
                                                           0, 0, 0);
#pragma unroll
      for (int mo = 0; mo < 4; ++mo)
#pragma unroll
        for (int r = 0; r < 4; ++r) h1[mo][r] = h1[mo][r] > 0.0f ? acc[mo][r] : 0.0f;
    }
    // input gradients: rows 0..3 at slot 0, 4..6 at slot 1
    f32x4v gx = zero;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        gx = __builtin_amdgcn_mfma_f32_16x16x4f32(T0[(m * 4 + r) * 64 + lane], h1[m][r], gx, 0, 0, 0);
    if (ok && s == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) grad_cf[ray * 7 + c] = gz[c] + gx[c];
      grad_cf[ray * 7 + 3] = gx[3];
    }
    if (ok && s == 1) {
#pragma unroll
      for (int c = 0; c < 3; ++c) grad_cf[ray * 7 + 4 + c] = gx[c];
    }
    // dW0 [64][23] = sum g1 (x) x; input 23 is 1: db0
    if (s == 3) x[5] = 1.0f;
    view_transpose(T, h1, i, s, A);
    wave_lds_fence();
#pragma unroll
    for (int c = 0; c < 6; ++c) T[(4 * c + s) * kVP + i] = x[c];
    wave_lds_fence();
#pragma unroll
    for (int b = 0; b < 2; ++b) {                        // rows 24 and on: columns not used
      const float4 q = *reinterpret_cast<const float4*>(T + (16 * b + i) * kVP + 4 * s);
      B[b][0] = q.x; B[b][1] = q.y; B[b][2] = q.z; B[b][3] = q.w;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          dW0[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[a][c], B[b][c], dW0[a][b], 0, 0, 0);
  }
  // slots' parts of the bias sums
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    db1[a] += __shfl_xor(db1[a], 16, 64);
    db1[a] += __shfl_xor(db1[a], 32, 64);
  }
  db2 += __shfl_xor(db2, 16, 64);
  db2 += __shfl_xor(db2, 32, 64);
  // waves 0..3 store their sums over the weights, waves 4..7 add theirs, the
  // workgroup adds the four copies
  float* copy = L + (wave & 3) * kMlpViewParams;
  for (int half = 0; half < 2; ++half) {
    __syncthreads();
    if ((wave >> 2) == half) {
      auto put = [&](int idx, float v) { copy[idx] = half ? copy[idx] + v : v; };
#pragma unroll
      for (int a = 0; a < 4; ++a) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int u = 16 * a + 4 * s + q;
#pragma unroll
          for (int b = 0; b < 4; ++b) put(kW1 + u * 64 + 16 * b + i, dW1[a][b][q]);
          put(kW0 + u * 23 + i, dW0[a][0][q]);
          if (i < 7) put(kW0 + u * 23 + 16 + i, dW0[a][1][q]);
          if (i == 7) put(kB0 + u, dW0[a][1][q]);
          if (i < 3) put(kW2 + i * 64 + u, dW2[a][q]);
        }
        if (s == 0) put(kB1 + 16 * a + i, db1[a]);
      }
      if (s == 0 && i < 3) put(kB2 + i, db2);
    }
  }
  __syncthreads();
  float* part = partial + int64_t(blockIdx.x) * kMlpViewParams;
  for (int t = threadIdx.x; t < kMlpViewParams; t += 64 * kViewBwdWaves)
    part[t] = ((L[t] + L[kMlpViewParams + t]) + L[2 * kMlpViewParams + t]) + L[3 * kMlpViewParams + t];
}

// workgroups of a kernel that stay resident together on the context's device
template <class Kernel>
static int resident_groups(ngprt_ctx* ctx, Kernel kernel, int threads, int* out) {
  if (*out > 0) return NGPRT_OK;
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess ||
      per_cu <= 0 || cus <= 0) {
    (void)hipGetLastError();
    return fail(ctx, NGPRT_E_HIP, "view MLP occupancy query failed");
  }
  *out = per_cu * cus;
  return NGPRT_OK;
}

int launch_view_mlp_backward(ngprt_ctx* ctx, int64_t n, const float* d, const float* c_d, const float* feat,
                             const float* grad_rgb, float* grad_cf, float* gmlp, hipStream_t st) {
  if ((n + 63) / 64 > 0x7FFFFFFF) return fail(ctx, NGPRT_E_SHAPE, "too many rays for one launch");
  int rc = resident_groups(ctx, view_mlp_backward_kernel, 64 * kViewBwdWaves, &ctx->vmlp_bwd_resident);
  if (rc) return rc;
  const int64_t groups = (n + 16 * kViewBwdWaves - 1) / (16 * kViewBwdWaves);
  const int64_t blocks = groups < ctx->vmlp_bwd_resident ? groups : ctx->vmlp_bwd_resident;
  const size_t need = (size_t(blocks) + kSumGroups) * kMlpViewParams * sizeof(float);
  if (need > ctx->ws_bytes) {
    if (ctx->ws) (void)hipFreeAsync(ctx->ws, st);
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
    if (dev_malloc_async((void**)&ctx->ws, need, st) != hipSuccess) {
      (void)hipGetLastError();
      return fail(ctx, NGPRT_E_ALLOC, "view MLP backward workspace allocation failed");
    }
    ctx->ws_bytes = need;
  }
  float* partial = reinterpret_cast<float*>(ctx->ws);
  hipLaunchKernelGGL(view_mlp_backward_kernel, dim3(unsigned(blocks)), dim3(64 * kViewBwdWaves), 0, st, n, d, c_d, feat,
                     grad_rgb, ctx->mlp_rec, grad_cf, partial);
  rc = check_launch(ctx, "view_mlp_backward_kernel");
  if (rc) return rc;
  return launch_partial_sums(ctx, partial, blocks, kMlpViewParams, partial + size_t(blocks) * kMlpViewParams, gmlp,
                             st);
}

int launch_view_mlp_arrange(ngprt_ctx* ctx, const float* params, hipStream_t st) {
  hipLaunchKernelGGL(view_mlp_arrange_kernel, dim3((kViewRecFloats + 255) / 256), dim3(256), 0, st, params,
                     ctx->mlp_rec);
  return check_launch(ctx, "view_mlp_arrange_kernel");
}

int launch_view_mlp(ngprt_ctx* ctx, int64_t n, const float* d, const float* c_d, const float* feat,
                    float* rgb, hipStream_t st) {
  if (n <= 0) return NGPRT_OK;
  int rc = resident_groups(ctx, view_mlp_kernel, 64 * kViewWaves, &ctx->vmlp_resident);
  if (rc) return rc;
  const int64_t groups = (n + 16 * kViewWaves - 1) / (16 * kViewWaves);
  const int64_t blocks = groups < ctx->vmlp_resident ? groups : ctx->vmlp_resident;
  hipLaunchKernelGGL(view_mlp_kernel, dim3(unsigned(blocks)), dim3(64 * kViewWaves), 0, st, n, d, c_d, feat,
                     ctx->mlp_rec, rgb);
  return check_launch(ctx, "view_mlp_kernel");
}

}  // namespace ngprt
