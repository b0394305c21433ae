// Render kernels: occupancy-distance march, hashed lookup + attention,
// front-to-back compositing, and the deferred MLP on MFMA.
//
// One lane owns one ray; a wave owns 64 rays (an 8x8 pixel tile when the
// caller orders rays tile-major, which keeps the coarse-level gathers of a
// wave on shared cache lines; neighbouring rays also march alike, so the
// wave's lanes finish within a sample or two of each other).  Each iteration
// the wave marches until every live lane has a sample at hand (one 2-byte
// grid read per marching point, none inside a known-empty region; lanes that
// have one run ahead meanwhile, SampleRing), then all lanes take the first of
// theirs and evaluate it together (the gather-heavy part runs with the wave
// converged).  After the last ray of the wave finishes, the wave runs
// the deferred MLP for its 64 rays with v_mfma_f32_16x16x4_f32.
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"
#include "internal.h"
#include "march.h"
#include "proposal_net.h"

namespace ngprt {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// MODE_RENDER: plain render.  MODE_RENDER_EXT: render that also writes the
// label outputs (t_first / t_far / t_half) and honours a proposal.
// MODE_MARCH: sample lists for parity checks (no MLP).
enum { MODE_RENDER = 0, MODE_MARCH = 1, MODE_RENDER_EXT = 2 };

// Optional per-ray sample-interval proposal [t_near, t_far, t_term,
// confidence], given per ray (prop) or computed by the loaded network in the
// kernel's prologue (net_w): a ray whose confidence reaches conf_thr marches
// only the lattice points with t in [t_near - margin, t_far + margin] (box:
// from lattice index max(0, floor((t_near - margin - t0) / step)); contracted
// domain: points before t_near - margin are visited without a read; without
// use_near from its start).  With far_guard > 0 the far end ends a ray only
// once its transmittance is below far_guard; otherwise it marches on.  A
// proposed ray that takes no sample in its interval marches again from its
// start as the plain march (its samples are then the plain render's; its
// read count includes both marches).
struct ProposalArgs {
  const float* prop;     // [n][4] (NULL: no per-ray proposal given)
  const uint2* net_w;    // loaded network: A-operand tiles (NULL: none)
  const float* net_b;    // its biases
  float* prop_out;       // [n][4] the network's outputs (NULL-able)
  float conf_thr;
  float margin;
  int use_near;
  float far_guard;
  int32_t* fallback;     // [n] 1 where the plain march ran after a proposal (NULL-able)
};

struct MarchRecord {
  int32_t* sample_k;
  int32_t* n_samples;
  int32_t* n_reads;
  int cap;
};

// Deferred MLP of the 64 rays of this wave (Eq. 5), 7 -> 16 -> 16 -> 3 on
// v_mfma_f32_16x16x4_f32.  xin: this wave's LDS slab [8][64] holding
// (C_d, F, 0) of every lane's ray.  Layout of the 16x16x4 product D = A B:
// lane l supplies A[l%16][l/16] and B[l/16][l%16] and receives
// D[4*(l/16) + r][l%16], r = 0..3.  The hidden index handed from one layer
// to the next is permuted (k-slot s of chunk c = unit 4s + c) so every layer
// consumes the previous layer's accumulators in place.
__device__ __forceinline__ void wave_mlp(const float* __restrict__ P, const float* xin, int lane,
                                         int64_t ray_base, int64_t n, float* __restrict__ rgb) {
  const int i = lane & 15, s = lane >> 4;
  float a1[2], a2[4], a3[4];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    int k = 4 * c + s;
    a1[c] = (k < 7) ? P[i * 7 + k] : 0.0f;
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    a2[c] = P[128 + i * 16 + 4 * s + c];
    a3[c] = (i < 3) ? P[400 + i * 16 + 4 * s + c] : 0.0f;
  }
  float b0[4], b1[4], b2[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    b0[r] = P[112 + 4 * s + r];
    b1[r] = P[384 + 4 * s + r];
    b2[r] = (4 * s + r < 3) ? P[448 + 4 * s + r] : 0.0f;
  }
#pragma unroll
  for (int blk = 0; blk < 4; ++blk) {
    const int ray = blk * 16 + i;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 2; ++c)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[c], xin[(4 * c + s) * 64 + ray], acc, 0, 0, 0);
    float h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = fmaxf(acc[r] + b0[r], 0.0f);
    acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[c], h[c], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = fmaxf(acc[r] + b1[r], 0.0f);
    acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a3[c], h[c], acc, 0, 0, 0);
    if (s == 0) {
      const int64_t gr = ray_base + ray;
      if (gr < n) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          float z = xin[j * 64 + ray] + (acc[j] + b2[j]);
          rgb[gr * 3 + j] = 1.0f / (1.0f + __expf(-z));
        }
      }
    }
  }
}

// Occupancy floor of the render kernel (waves per SIMD; the 16-level kernels
// fit 4 with ~126 VGPRs).  Giving each XCD one contiguous eighth of the rays
// measured slower on the 8-view 1080p workload (54.2 -> 61.9 ms): the XCDs
// then work on different views at once and share no Infinity Cache lines.
#ifndef NGPRT_RENDER_WAVES_PER_EU
#define NGPRT_RENDER_WAVES_PER_EU 4
#endif

// One wave a workgroup: a wave's time varies with its rays (0.65 ms in the
// median, 2 ms at most on 1920x1080 views), and a workgroup of four held its
// slots until the slowest was done (256 against 64 threads: eight 1920x1080
// views 49.0 against 44.8 ms, one 1200x800 view 4.67 against 4.37, 2^18
// training rays on 16 x 2^19 tables 2.93 against 2.45).
constexpr int block_threads(int slots) { return slots == 1 ? 64 : 256; }

// MODEL: bit 0 = baked feature model, bit 1 = occupancy pyramid march,
// bit 2 = the baked model's ablation aggregations
// SLOTS: lanes a ray (march_slots); above 1 for small launches, without a
// proposal: a workgroup then holds 256 / SLOTS rays
template <int DOM, int DT, int LMAX, int MODE, int MODEL, int SLOTS>
__global__ void __launch_bounds__(block_threads(SLOTS)) __attribute__((amdgpu_waves_per_eu(NGPRT_RENDER_WAVES_PER_EU)))
render_kernel(SceneArgs S, int64_t n, const float* __restrict__ O,
                                                     const float* __restrict__ D, RayOut out,
                                                     MarchRecord rec, const float* __restrict__ mlp,
                                                     int naive, ProposalArgs pa) {
  constexpr bool EXT = MODE == MODE_RENDER_EXT;
  constexpr bool KEEP_K = EXT || MODE == MODE_MARCH;    // the samples' lattice indices are used
  constexpr bool RING = SLOTS == 1;
  constexpr int kWaves = block_threads(SLOTS) / 64;
  __shared__ float xin_all[RING ? kWaves : 1][8 * 64];
  __shared__ float ring_t[RING ? kWaves : 1][RING ? kRingWords : 1];
  __shared__ int32_t ring_reads[RING ? kWaves : 1][RING ? kRingWords : 1];
  __shared__ int32_t ring_k[RING && KEEP_K ? kWaves : 1][RING && KEEP_K ? kRingWords : 1];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const unsigned block = blockIdx.x;
  // first ray of the wave (SLOTS > 1: of the workgroup)
  const int64_t ray_base = RING ? (int64_t(block) * kWaves + wave) * 64 : int64_t(block) * (256 / SLOTS);
  const int ray_index = RING ? lane : int(threadIdx.x) / SLOTS;
  const int64_t ray = ray_base + ray_index;
  const bool in_range = ray < n;

  MarchState m;
  const float* oray = O + 3 * (in_range ? ray : 0);
  const float* dray = D + 3 * (in_range ? ray : 0);
  march_init<DOM>(S, oray, dray, in_range, m);
  bool proposed = false, fell_back = false;
  if (RING && EXT && (pa.prop || pa.net_w)) {
    float q[4];
    if (pa.net_w) {
      // the loaded network, run by the wave for its 64 rays (uniform branch:
      // every wave of the grid takes it)
      float* out4 = xin_all[wave];
      prop_infer_wave(pa.net_w, pa.net_b, O, D, ray_base, n, lane, out4);
      __syncthreads();
#pragma unroll
      for (int c = 0; c < 4; ++c) q[c] = out4[4 * lane + c];
      __syncthreads();
      if (pa.prop_out && in_range) {
#pragma unroll
        for (int c = 0; c < 4; ++c) pa.prop_out[4 * ray + c] = q[c];
      }
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) q[c] = in_range ? pa.prop[4 * ray + c] : 0.0f;
    }
    if (in_range && !m.done && q[3] >= pa.conf_thr) {
      m.t_hi = q[1] + pa.margin;
      if (pa.use_near) {
        const float lo = q[0] - pa.margin;
        if (DOM == DOM_BOX) {
          const float kf = floorf((lo - m.t0) / S.step);
          m.k = kf > 0.0f ? (kf < (float)kMaxLattice ? (int)kf : kMaxLattice) : 0;
        } else {
          m.t_lo = lo;
        }
      }
      proposed = true;
    }
  }
  float T = 1.0f, cd[3] = {0.f, 0.f, 0.f}, fv[4] = {0.f, 0.f, 0.f, 0.f}, depth = 0.0f;
  // labels: t of the first sample, of the sample after which T < 0.5, and of
  // the sample after which T < 1e-3 (the proposal's far end)
  float t_first = 0.0f, t_last = 0.0f, t_half = 0.0f, t_far = 0.0f;
  bool half_set = false, far_set = false;
  // distortion regulariser: running sums of w, w m and w (m W_< - S_<), and w^2
  float dW = 0.0f, dS = 0.0f, dP = 0.0f, dQ = 0.0f;
  int ns = 0, reads = 0;        // reads: of the march, which may be ahead of the samples
  int reads_at = 0;             // up to the last evaluated sample
  bool ended = false;           // by transmittance or the sample cap
  constexpr bool PYR = (MODEL & 2) != 0;
  if constexpr (RING) {
  SampleRing ring{ring_t[wave], ring_reads[wave], KEEP_K ? ring_k[KEEP_K ? wave : 0] : nullptr, 0, 0};

  for (;;) {
    march_ahead<DOM, PYR, EXT, KEEP_K>(S, m, naive != 0, reads, ring, lane);
    if constexpr (EXT) {
      // a proposed ray at the end of its interval with every sample evaluated
      bool resumed = false;
      if (ring.count == 0 && proposed && !fell_back && !ended) {
        if (ns == 0) {
          // the proposed interval holds no occupied lattice point: march again
          // from the start as the plain march
          march_init<DOM>(S, oray, dray, in_range, m);
          fell_back = true;
          resumed = true;
        } else if (m.stopped_at_hi && pa.far_guard > 0.0f && !(T < pa.far_guard)) {
          // at the proposed far end with too much transmittance left: march on
          m.t_hi = __int_as_float(0x7F800000);
          m.done = false;
          m.stopped_at_hi = false;
          resumed = true;
        }
      }
      if (__ballot(resumed) != 0) march_ahead<DOM, PYR, EXT, KEEP_K>(S, m, naive != 0, reads, ring, lane);
    }
    const bool have = ring.count > 0;
    if (__ballot(have) == 0) break;
    float u[3] = {0.f, 0.f, 0.f}, ts = 0.0f;
    int ks = 0;
    if (have) {
      const int at = ring.head * 64 + lane;
      ts = ring.t[at];
      reads_at = ring.reads[at];
      if (KEEP_K) ks = ring.k[at];
      ring.head = (ring.head + 1) & (kAhead - 1);
      --ring.count;
      lattice_coord<DOM>(S, m, ts, u);
    }
    if (have) {
      float f[8];
      NoSink sink;
      eval_sample<MODEL & 5, DT, LMAX>(S, u, f, sink);
      const float sigma = exp32(f[0]);
      const float e = exp32(-(sigma * S.step));
      const float alpha = 1.0f - e;
      const float w = T * alpha;
#pragma unroll
      for (int j = 0; j < 3; ++j) cd[j] = __builtin_fmaf(w, f[1 + j], cd[j]);
#pragma unroll
      for (int j = 0; j < 4; ++j) fv[j] = __builtin_fmaf(w, f[4 + j], fv[j]);
      depth = __builtin_fmaf(w, ts, depth);
      if (MODE == MODE_MARCH && ns < rec.cap) rec.sample_k[ray * rec.cap + ns] = ks;
      T = T * e;
      if (EXT) {
        const float mid = ((float)ks + 0.5f) * S.step;
        dP = __builtin_fmaf(w, mid * dW - dS, dP);
        dQ = __builtin_fmaf(w, w, dQ);
        dW = dW + w;
        dS = __builtin_fmaf(w, mid, dS);
        if (ns == 0) t_first = ts;
        t_last = ts;
        if (!half_set && T < 0.5f) { t_half = ts; half_set = true; }
        if (!far_set && T < 1e-3f) { t_far = ts; far_set = true; }
      }
      ++ns;
      if (T < S.thr || ns >= S.max_samples) {
        m.done = true;
        ended = true;
        ring.count = 0;
      }
    }
  }
  } else {
  // the same, SLOTS lanes a ray: each takes one of the ray's next samples, and
  // the sums run over them in order on every lane of the ray, so they are the
  // one-lane kernel's bit for bit
  const int slot = lane & (SLOTS - 1);
  for (;;) {
    float u[3] = {0.f, 0.f, 0.f}, ts = 0.0f;
    int ks = 0, my_reads = 0;
    const bool have = march_slots<DOM, PYR, SLOTS>(S, m, slot, reads, u, ts, ks, my_reads);
    const uint32_t bits = slot_bits<SLOTS>(have, lane);
    if (__ballot(have) == 0) break;
    float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, e = 1.0f;
    if (have) {
      NoSink sink;
      eval_sample<MODEL & 5, DT, LMAX>(S, u, f, sink);
      e = exp32(-(exp32(f[0]) * S.step));
    }
    each_slot<SLOTS>([&](auto J) {
      const float ej = slot_value<SLOTS, J>(e), tj = slot_value<SLOTS, J>(ts);
      const int rj = slot_value<SLOTS, J>(my_reads), kj = EXT ? slot_value<SLOTS, J>(ks) : 0;
      float fj[7];
#pragma unroll
      for (int c = 0; c < 7; ++c) fj[c] = slot_value<SLOTS, J>(f[1 + c]);
      if (((bits >> J) & 1u) && !ended) {
        const float w = T * (1.0f - ej);
#pragma unroll
        for (int j = 0; j < 3; ++j) cd[j] = __builtin_fmaf(w, fj[j], cd[j]);
#pragma unroll
        for (int j = 0; j < 4; ++j) fv[j] = __builtin_fmaf(w, fj[3 + j], fv[j]);
        depth = __builtin_fmaf(w, tj, depth);
        T = T * ej;
        reads_at = rj;
        if (EXT) {
          const float mid = ((float)kj + 0.5f) * S.step;
          dP = __builtin_fmaf(w, mid * dW - dS, dP);
          dQ = __builtin_fmaf(w, w, dQ);
          dW = dW + w;
          dS = __builtin_fmaf(w, mid, dS);
          if (ns == 0) t_first = tj;
          t_last = tj;
          if (!half_set && T < 0.5f) { t_half = tj; half_set = true; }
          if (!far_set && T < 1e-3f) { t_far = tj; far_set = true; }
        }
        ++ns;
        ended = T < S.thr || ns >= S.max_samples;
      }
    });
    if (ended) m.done = true;
  }
  }
  if (ended) reads = reads_at;
  if (!half_set) t_half = t_last;
  if (!far_set) t_far = t_last;

  if (MODE == MODE_MARCH) {
    if (in_range) {
      for (int j = ns; j < rec.cap; ++j) rec.sample_k[ray * rec.cap + j] = -1;
      if (rec.n_samples) rec.n_samples[ray] = ns;
      if (rec.n_reads) rec.n_reads[ray] = reads;
    }
    return;
  }
  if (in_range && (RING || (lane & (SLOTS - 1)) == 0)) {
    if (out.c_d) { for (int j = 0; j < 3; ++j) out.c_d[ray * 3 + j] = cd[j]; }
    if (out.feat) { for (int j = 0; j < 4; ++j) out.feat[ray * 4 + j] = fv[j]; }
    if (out.t_final) out.t_final[ray] = T;
    if (out.depth) out.depth[ray] = depth;
    if (out.n_samples) out.n_samples[ray] = ns;
    if (out.n_reads) out.n_reads[ray] = reads;
    if (EXT) {
      if (out.t_first) out.t_first[ray] = t_first;
      if (out.t_far) out.t_far[ray] = t_far;
      if (out.t_half) out.t_half[ray] = t_half;
      if (out.dist_loss) out.dist_loss[ray] = 2.0f * dP + dQ * (S.step * (1.0f / 3.0f));
      if (pa.fallback) pa.fallback[ray] = fell_back ? 1 : 0;
    }
  }
  float* xin = xin_all[RING ? wave : 0];
  if (RING || (lane & (SLOTS - 1)) == 0) {
    const int at = RING ? lane : ray_index;
    xin[0 * 64 + at] = cd[0];
    xin[1 * 64 + at] = cd[1];
    xin[2 * 64 + at] = cd[2];
    xin[3 * 64 + at] = fv[0];
    xin[4 * 64 + at] = fv[1];
    xin[5 * 64 + at] = fv[2];
    xin[6 * 64 + at] = fv[3];
    xin[7 * 64 + at] = 0.0f;
  }
  __syncthreads();
  // SLOTS > 1: the workgroup's rays (at most 64) on its first wave; a column of
  // the products is a ray, so columns past them touch nothing
  if (!S.view_mlp && (RING || wave == 0)) {
    const int64_t end = RING ? n : (ray_base + 256 / SLOTS < n ? ray_base + 256 / SLOTS : n);
    wave_mlp(mlp, xin, lane, ray_base, end, out.rgb);
  }
}

// ---------------------------------------------------------------------------
// dispatch

template <int MODE, int DOM, int DT, int SLOTS>
static inline void dispatch_l(const SceneArgs& S, hipStream_t st, int64_t n, const float* o, const float* d,
                       const RayOut& out, const MarchRecord& rec, const float* mlp, int naive,
                       const ProposalArgs& pa) {
  const int64_t rays = block_threads(SLOTS) / SLOTS;      // per workgroup
  const dim3 g(unsigned((n + rays - 1) / rays));
#define NGPRT_RENDER(LM, MD)                                                                                 \
  hipLaunchKernelGGL((render_kernel<DOM, DT, LM, MODE, MD, SLOTS>), g, dim3(block_threads(SLOTS)), 0, st, S, n, o, \
                     d, out, rec, mlp, naive, pa)
  if (S.model == 1 && S.gen) {
    // the ablation aggregations: float32 tables only (checked at create)
    if constexpr (DT == DT_F32) {
      if (S.pyr_n > 0) NGPRT_RENDER(4, 7);
      else NGPRT_RENDER(4, 5);
    }
  } else if (S.model == 1 && S.L <= 2) {
    // at most two fine levels: coarse rows of at most 12 channels
    if (S.pyr_n > 0) NGPRT_RENDER(2, 3);
    else NGPRT_RENDER(2, 1);
  } else if (S.model == 1) {
    if (S.pyr_n > 0) NGPRT_RENDER(4, 3);
    else NGPRT_RENDER(4, 1);
  } else if (S.pyr_n > 0) {
    NGPRT_RENDER(16, 2);
  } else if (S.L <= 8) {
    NGPRT_RENDER(8, 0);
  } else {
    NGPRT_RENDER(16, 0);
  }
#undef NGPRT_RENDER
}

template <int MODE, int SLOTS>
static inline void dispatch(const SceneArgs& S, int dom, int dt, hipStream_t st, int64_t n, const float* o,
                     const float* d, const RayOut& out, const MarchRecord& rec, const float* mlp, int naive,
                     const ProposalArgs& pa) {
#define NGPRT_CASE(DOMV, DTV)                                                       \
  if (dom == DOMV && dt == DTV) {                                                   \
    dispatch_l<MODE, DOMV, DTV, SLOTS>(S, st, n, o, d, out, rec, mlp, naive, pa);   \
    return;                                                                         \
  }
  NGPRT_CASE(DOM_BOX, DT_F32)
  NGPRT_CASE(DOM_BOX, DT_BF16)
  NGPRT_CASE(DOM_BOX, DT_FP8)
  NGPRT_CASE(DOM_CONTRACT, DT_F32)
  NGPRT_CASE(DOM_CONTRACT, DT_BF16)
  NGPRT_CASE(DOM_CONTRACT, DT_FP8)
#undef NGPRT_CASE
}

// One function per kernel family, each compiled in a file of its own (a family
// is some 45 kernels: domains x table types x feature models and marches).
#define NGPRT_DISPATCH_ARGS                                                                          \
  const SceneArgs &S, int dom, int dt, hipStream_t st, int64_t n, const float *o, const float *d,     \
      const RayOut &out, const MarchRecord &rec, const float *mlp, int naive, const ProposalArgs &pa
void render_plain(NGPRT_DISPATCH_ARGS);     // MODE_RENDER
void render_ext(NGPRT_DISPATCH_ARGS);       // MODE_RENDER_EXT
void render_march(NGPRT_DISPATCH_ARGS);     // MODE_MARCH
// several lanes a ray, with or without the label outputs
void render_small(NGPRT_DISPATCH_ARGS);     // kSmallSlots
void render_mid(NGPRT_DISPATCH_ARGS);       // kMidSlots

constexpr int kSmallSlots = 16, kMidSlots = 8;

}  // namespace ngprt
