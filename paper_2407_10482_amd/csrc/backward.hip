// Backward of the render path (a training extension; the paper trains its
// model but states no gradient code).  FP32 tables only.
//
// Forward state is recomputed per ray instead of stored per sample:
//  pass 1  re-march the ray: composited C_d and F (Eq. 2, Eq. 5), or take
//          the forward's per-ray C_d and F when the caller hands them over
//          (the same float32 values; not with the regulariser, whose sums
//          this pass also forms); then, per
//          lane, the deferred MLP forward and backward give dL/dC_d, dL/dF,
//          and per-ray outer products whose sum over the workgroup's 16 or 64
//          rays is taken on v_mfma_f32_16x16x4_f32 (K = rays) and written as
//          one 451-float partial per workgroup (with the view-dependent MLP,
//          dL/dC_d and dL/dF come per ray from its own backward, `ups`);
//  pass 2  re-march again with the same decisions; at each sample
//          dL/dsigma_i = delta (T_{i+1} s_i - (S - P_i)) with
//          s_i = dL/dC_d . c_i + dL/dF . v_i, S = dL/dC_d . C_d + dL/dF . F and
//          P_i the running sum of w_j s_j; then the softmax adjoint
//          dL/da_l = w_l (dL/df . v_l - dL/df . f) and the trilinear scatter of
//          every level's 9-channel gradient into its 8 corner entries with
//          hardware float atomics (order-nondeterministic sums).  The dot
//          products dL/df . v_l come from two sums a level that the sample's
//          one lookup leaves behind (GradSink), not from a second gather.
//          The wave first merges the samples of equal cells, whose eight
//          corner rows then leave as one row each (scatter_cells).
//          The baked model scatters into its fine levels and coarse atlas
//          rows instead (baked_scatter).  In the deterministic mode each
//          contribution goes to a record of its own instead (det.hip).
// The workgroups' MLP partials are then added in a fixed order (reduce.h).
#include <hip/hip_runtime.h>

#include <cmath>

#include "device.h"
#include "internal.h"
#include "march.h"
#include "reduce.h"

namespace ngprt {

typedef float bf32x4 __attribute__((ext_vector_type(4)));

constexpr int kPad = 17;   // LDS row pitch of the per-wave staging (bank spread)

// value of lane (lane ^ J) for every lane of a full wave; J = 1, 2, 4, 8 by
// DPP lane moves (quad_perm, row_half_mirror, row_mirror), 16 by ds_swizzle,
// 32 by ds_bpermute
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane) {
  const int x = int(v);
  if constexpr (J == 1) return uint32_t(__builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));
  if constexpr (J == 2) return uint32_t(__builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));
  if constexpr (J == 4) {
    const int h = __builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false);   // i ^ 7 within 8
    return uint32_t(__builtin_amdgcn_update_dpp(h, h, 0x1B, 0xF, 0xF, false)); // then ^ 3
  }
  if constexpr (J == 8) {
    const int m = __builtin_amdgcn_update_dpp(x, x, 0x140, 0xF, 0xF, false);   // i ^ 15 within 16
    return uint32_t(__builtin_amdgcn_update_dpp(m, m, 0x141, 0xF, 0xF, false)); // then ^ 7
  }
  if constexpr (J == 16) return uint32_t(__builtin_amdgcn_ds_swizzle(x, 0x401F));
  return uint32_t(__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, x));
}

// one compare-exchange stage of a bitonic sort over the wave's 64 lanes
template <int K, int J>
__device__ __forceinline__ uint32_t bitonic_stage(uint32_t v, int lane) {
  const uint32_t o = lane_xor<J>(v, lane);
  const bool keep_min = ((lane & J) == 0) == ((lane & K) == 0);
  const uint32_t lo = v < o ? v : o, hi = v < o ? o : v;
  return keep_min ? lo : hi;
}

// Ascending sort of one word per lane over the wave's 64 lanes.
__device__ __forceinline__ uint32_t wave_sort(uint32_t w, int lane) {
  w = bitonic_stage<2, 1>(w, lane);
  w = bitonic_stage<4, 2>(w, lane);   w = bitonic_stage<4, 1>(w, lane);
  w = bitonic_stage<8, 4>(w, lane);   w = bitonic_stage<8, 2>(w, lane);   w = bitonic_stage<8, 1>(w, lane);
  w = bitonic_stage<16, 8>(w, lane);  w = bitonic_stage<16, 4>(w, lane);  w = bitonic_stage<16, 2>(w, lane);
  w = bitonic_stage<16, 1>(w, lane);
  w = bitonic_stage<32, 16>(w, lane); w = bitonic_stage<32, 8>(w, lane);  w = bitonic_stage<32, 4>(w, lane);
  w = bitonic_stage<32, 2>(w, lane);  w = bitonic_stage<32, 1>(w, lane);
  w = bitonic_stage<64, 32>(w, lane); w = bitonic_stage<64, 16>(w, lane); w = bitonic_stage<64, 8>(w, lane);
  w = bitonic_stage<64, 4>(w, lane);  w = bitonic_stage<64, 2>(w, lane);  w = bitonic_stage<64, 1>(w, lane);
  return w;
}

// LDS of one wave for scatter_cells, in floats: the samples' corner weights
// [64][8], row indices [64][8] and gradients [64][16] (the last sized for the
// widest row), in sorted order.  Shared with the MLP's staging (2 x 64 x kPad),
// which is done before the first scatter.
constexpr int kStageW = 0, kStageI = 64 * 8, kStageG = 2 * 64 * 8, kStageFloats = 2 * 64 * kPad;
static_assert(kStageG + 64 * 16 <= kStageFloats, "staging slab");

constexpr uint32_t kNoRow = 0xFFFFFFFFu;

// Adds w[k] * g[j] to gbase[idx[k] * stride + j] (k < 8 corners, j < nv <= NV
// channels; idx kNoRow: no such row) for every lane with have set, summing the
// lanes of equal cells (key0, key1) first.  Every lane of the wave calls it.
//
// What bounds it: the memory side takes float atomics as requests of 64 bytes
// at 21 G a second whatever their address, order, scope or working set (a
// probe over 0.15 to 302 MB), so the rows that leave the wave are what a
// scatter costs; next to that, the instructions of merging them.  A cell's
// samples share all eight corner rows, so the wave sorts its 64 samples by
// cell once a level (not once a corner), and the sum over a cell's samples of
// the outer product w (8) x g (9) is a matrix product with the samples as K:
// v_mfma_f32_16x16x4_f32 takes two cells at a time (rows: their 2 x 8 corners;
// columns: up to 16 channels; the sorted samples of a cell are contiguous, so
// two cells take one or two instructions when nothing repeats and 16 when the
// wave shares one).  Its result rows go from the accumulators straight to the
// atomics, each row's channels on neighbouring lanes so that a row is one or
// two requests; x-adjacent corners (neighbouring rows for even x) share an
// instruction, which the memory side merges when they share a line.
// Measured (training step of 2^18 rays, tables 8 x 2^14 / 16 x 2^19): a sort and
// scan a corner, with a second gather of the level's rows, 7.49 / 21.7 ms; this
// 3.70 / 17.9 ms (before lanes a ray and padded rows, below).
// A wave that holds a non-finite gradient adds its contributions lane by lane
// instead: in a matrix product it would reach the other cell's rows too.
template <int NV>
__device__ __forceinline__ void scatter_cells(float* __restrict__ gbase, int stride, int nv, bool have,
                                              uint32_t key0, uint32_t key1, const uint32_t idx[8],
                                              const float w[8], const float g[NV], int lane, float* stage) {
  const uint64_t active = __ballot(have);
  if (active == 0) return;
  const int na = __popcll(active);
  float mag = 0.0f;
#pragma unroll
  for (int j = 0; j < NV; ++j) mag += fabsf(g[j]);
  if (__ballot(have && !(mag < __int_as_float(0x7F800000))) != 0) {
    if (have) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (idx[k] != kNoRow) {
          float* dst = gbase + size_t(idx[k]) * size_t(stride);
          for (int j = 0; j < NV; ++j)
            if (j < nv) unsafeAtomicAdd(dst + j, w[k] * g[j]);
        }
    }
    return;
  }
  // sort by a 25-bit hash of the cell; lanes without a sample go last.  Cells
  // whose hashes collide only split each other's runs: a run is of equal keys.
  uint32_t h = (key0 * 0x9E3779B1u) ^ (key1 * 0x85EBCA77u);
  h ^= h >> 15;
  const uint32_t word = wave_sort(have ? (((h >> 1) & ~63u) | uint32_t(lane)) : (0xFFFFFFC0u | uint32_t(lane)), lane);
  const int src = int(word & 63u);
  const uint32_t k0 = uint32_t(__builtin_amdgcn_ds_bpermute(src << 2, int(key0)));
  const uint32_t k1 = uint32_t(__builtin_amdgcn_ds_bpermute(src << 2, int(key1)));
  const uint32_t p0 = __shfl_up(k0, 1, 64), p1 = __shfl_up(k1, 1, 64);
  uint64_t heads = __ballot(lane < na && (lane == 0 || k0 != p0 || k1 != p1));
  // the sample's place in the sorted order, at its own lane
  const int row = __builtin_amdgcn_ds_permute(src << 2, lane);
  float* sW = stage + kStageW;
  uint32_t* sI = reinterpret_cast<uint32_t*>(stage + kStageI);
  float* sG = stage + kStageG;
  constexpr int GP = NV <= 12 ? 12 : 16;
  if (have) {
    float4* dw = reinterpret_cast<float4*>(sW + row * 8);
    dw[0] = make_float4(w[0], w[1], w[2], w[3]);
    dw[1] = make_float4(w[4], w[5], w[6], w[7]);
    // corners by the accumulator layout: even ones, then odd ones
    uint4* di = reinterpret_cast<uint4*>(sI + row * 8);
    di[0] = make_uint4(idx[0], idx[2], idx[4], idx[6]);
    di[1] = make_uint4(idx[1], idx[3], idx[5], idx[7]);
    float4* dg = reinterpret_cast<float4*>(sG + row * GP);
#pragma unroll
    for (int q = 0; q < GP / 4; ++q) {
      float4 t;
      t.x = 4 * q < NV ? g[4 * q < NV ? 4 * q : 0] : 0.0f;
      t.y = 4 * q + 1 < NV ? g[4 * q + 1 < NV ? 4 * q + 1 : 0] : 0.0f;
      t.z = 4 * q + 2 < NV ? g[4 * q + 2 < NV ? 4 * q + 2 : 0] : 0.0f;
      t.w = 4 * q + 3 < NV ? g[4 * q + 3 < NV ? 4 * q + 3 : 0] : 0.0f;
      dg[q] = t;
    }
  }
  // the other lanes' rows are read below: a wave-scope fence orders the LDS
  // stores before the loads (and the next call's stores after them)
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const int i = lane & 15, s = lane >> 4;
  const int corner = 2 * (i & 3) + ((i >> 2) & 1);      // of accumulator row i
  while (heads) {
    const int a0 = __ffsll((unsigned long long)heads) - 1;
    heads &= heads - 1;
    const int b0 = heads ? __ffsll((unsigned long long)heads) - 1 : na;
    heads &= heads - 1;
    const int end = heads ? __ffsll((unsigned long long)heads) - 1 : na;
    const int lo = i < 8 ? a0 : b0, hi = i < 8 ? b0 : end;
    bf32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int c = a0 >> 2; 4 * c < end; ++c) {
      const int r = 4 * c + s;
      const float A = (r >= lo && r < hi) ? sW[r * 8 + corner] : 0.0f;
      const float B = (r >= a0 && r < end && i < GP) ? sG[r * GP + i] : 0.0f;
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(A, B, acc, 0, 0, 0);
    }
    const int head = s < 2 ? a0 : b0;
    if (head < na && i < nv) {
      const uint4 id = *reinterpret_cast<const uint4*>(sI + head * 8 + 4 * (s & 1));
      if (id.x != kNoRow) unsafeAtomicAdd(gbase + size_t(id.x) * size_t(stride) + i, acc[0]);
      if (id.y != kNoRow) unsafeAtomicAdd(gbase + size_t(id.y) * size_t(stride) + i, acc[1]);
      if (id.z != kNoRow) unsafeAtomicAdd(gbase + size_t(id.z) * size_t(stride) + i, acc[2]);
      if (id.w != kNoRow) unsafeAtomicAdd(gbase + size_t(id.w) * size_t(stride) + i, acc[3]);
    }
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// What the backward keeps of a sample's lookup, per level: the interpolated
// logit, density channel A_l = v_l[0] and colour sum
// B_l = dL/dC_d . v_l[1..3] + dL/dF . v_l[4..7], so that dL/df . v_l =
// dL/df_0 A_l + w B_l once the sample's weight w is known (dL/df_j = w times
// the ray's dL/dC_d or dL/dF).  Vectors, so that the rolled level loops index
// them by a wave-uniform register offset.
template <int LMAX>
struct GradSink {
  typedef float vec __attribute__((ext_vector_type(LMAX)));
  vec a, A, B;
  float run_max, esum;
  const float* gcd;
  const float* gfv;
  __device__ __forceinline__ void level(int l, const float* acc, const Corners&) {
    a[l] = acc[8];
    A[l] = acc[0];
    float b = 0.0f;
#pragma unroll
    for (int j = 0; j < 3; ++j) b = __builtin_fmaf(gcd[j], acc[1 + j], b);
#pragma unroll
    for (int j = 0; j < 4; ++j) b = __builtin_fmaf(gfv[j], acc[4 + j], b);
    B[l] = b;
  }
  __device__ __forceinline__ void done(float m, float e) { run_max = m; esum = e; }
  // baked model: the level's gates in a and g
  vec g;
  __device__ __forceinline__ void gates(int l, float gw, float gb, const float* acc, const Corners&) {
    float b = 0.0f;
#pragma unroll
    for (int j = 0; j < 3; ++j) b = __builtin_fmaf(gcd[j], acc[1 + j], b);
#pragma unroll
    for (int j = 0; j < 4; ++j) b = __builtin_fmaf(gfv[j], acc[4 + j], b);
#pragma unroll
    for (int q = 0; q < LMAX; ++q)
      if (q == l) {
        a[q] = gw;
        g[q] = gb;
        A[q] = acc[0];
        B[q] = b;
      }
  }
};

// D[i][j] = sum over the wave's 64 rays r of A_r[i] * B_r[j] (i, j < 16).
// sA, sB: [64][kPad].  Lane l returns D[4*(l/16) + q][l%16], q = 0..3.
__device__ __forceinline__ bf32x4 wave_outer_sum(const float* sA, const float* sB, int lane) {
  const int i = lane & 15, s = lane >> 4;
  bf32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const int r = 4 * c + s;
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sA[r * kPad + i], sB[r * kPad + i], acc, 0, 0, 0);
  }
  return acc;
}

// Adjoint of the baked feature construction at one sample (Sec. 4.2 Eq. 7-8):
// with f_0 = f~_0 + sum_l g(omega_l) s_l and f_j = f~_j + sum_l g(beta_l) v_lj
// (j >= 1), dL/df (gf) gives
//   fine level l:  dL/dv_l0 = gf_0 g(omega_l),  dL/dv_lj = gf_j g(beta_l),
//   coarse row:    dL/df~_j = gf_j,
//                  dL/domega_l = gf_0 s_l g'(omega_l),
//                  dL/dbeta_l = sum_{j>=1} gf_j v_lj g'(beta_l),
// each spread trilinearly over its 8 corners; g' = g (1 - g).  The gates, s_l
// and sum_j gf_j v_lj come from the lookup (q; w: the sample's weight).
// Vertices of empty blocks take the default vector and receive no gradient.
// Every lane of the wave takes part (have = false: no contribution).
// gtab: [L][T][tstride] (channel 8, the hash model's logit, untouched); gatlas:
// [n_blocks][8][8][8][C], C = 8 + 2 L.
template <int LMAX>
__device__ __forceinline__ void baked_scatter(const SceneArgs& S, const float u[3], bool have, const float gf[8],
                                              float w, const GradSink<LMAX>& q, float* __restrict__ gtab,
                                              int tstride, float* __restrict__ gatlas, int lane,
                                              float* stage) {
  static_assert(LMAX <= 4, "the coarse row holds at most 16 channels");
  constexpr int CMAX = 8 + 2 * LMAX;
  const int C = 8 + 2 * S.L;
  float gco[CMAX];
#pragma unroll
  for (int j = 0; j < 8; ++j) gco[j] = have ? gf[j] : 0.0f;
#pragma unroll
  for (int j = 8; j < CMAX; ++j) gco[j] = 0.0f;
  const size_t T_entries = size_t(1) << S.log2T;
#pragma unroll
  for (int l = 0; l < LMAX; ++l) {
    if (l >= S.L) break;
    Corners c;
    level_corners(u, S.N[l], S.Nf[l], S.mask, c);
    float gv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) gv[j] = 0.0f;
    if (have) {
      const float gw = q.a[l], gb = q.g[l];
      gco[8 + 2 * l] = gf[0] * q.A[l] * (gw * (1.0f - gw));
      gco[9 + 2 * l] = (w * q.B[l]) * (gb * (1.0f - gb));
      gv[0] = gf[0] * gw;
#pragma unroll
      for (int j = 1; j < 8; ++j) gv[j] = gf[j] * gb;
    }
    scatter_cells<8>(gtab + (size_t(l) * T_entries) * size_t(tstride), tstride, 8, have, c.key0, c.key1, c.idx, c.w,
                     gv, lane, stage);
  }
  // coarse rows: one vertex = (atlas row, local offset)
  int i0[3];
  float fr[3], gr[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float p = u[a] * S.LCf;
    int i = (int)floorf(p);
    i = i < 0 ? 0 : (i > S.LC - 1 ? S.LC - 1 : i);
    i0[a] = i;
    fr[a] = __builtin_fmaf(u[a], S.LCf, -(float)i);
    gr[a] = 1.0f - fr[a];
  }
  uint32_t idx[8];
  float wk[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int bx = k & 1, by = (k >> 1) & 1, bz = (k >> 2) & 1;
    const int vx = i0[0] + bx, vy = i0[1] + by, vz = i0[2] + bz;
    const int bid = have ? S.cidx[((vz >> 3) * S.nb + (vy >> 3)) * S.nb + (vx >> 3)] : -1;
    // n_blocks * 512 <= 2^31, so a vertex index never reads as kNoRow
    idx[k] = bid >= 0 ? uint32_t(bid) * 512u + uint32_t(((vz & 7) * 8 + (vy & 7)) * 8 + (vx & 7)) : kNoRow;
    wk[k] = ((bx ? fr[0] : gr[0]) * (by ? fr[1] : gr[1])) * (bz ? fr[2] : gr[2]);
  }
  // the cell's coordinates, below 2^11 each
  const uint32_t key = uint32_t(i0[0]) | (uint32_t(i0[1]) << 11);
  scatter_cells<CMAX>(gatlas, C, C, have, key, uint32_t(i0[2]), idx, wk, gco, lane, stage);
}

// SLOTS: lanes a ray (see march_slots); a workgroup holds 256 / SLOTS rays and
// writes one partial of the MLP gradient.
template <int DOM, int LMAX, bool PYR, int MODEL, int SLOTS>
__global__ void __launch_bounds__(256) backward_kernel(SceneArgs S, int64_t n, const float* __restrict__ O,
                                                       const float* __restrict__ D,
                                                       const float* __restrict__ grad_rgb,
                                                       const float* __restrict__ grad_dist,
                                                       const float* __restrict__ ups,
                                                       const float* __restrict__ fcd,
                                                       const float* __restrict__ ffv,
                                                       float* __restrict__ gtab, int tstride,
                                                       float* __restrict__ gatlas,
                                                       float* __restrict__ partial,
                                                       const float* __restrict__ P, DetRecords det) {
  __shared__ __align__(16) float stage_all[4][kStageFloats];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int slot = lane & (SLOTS - 1);
  constexpr int kRays = 256 / SLOTS;                     // of the workgroup, at most 64
  const int ray_in_block = int(threadIdx.x) / SLOTS;
  const int64_t ray = int64_t(blockIdx.x) * kRays + ray_in_block;
  const bool in_range = ray < n;
  const float* o = O + 3 * (in_range ? ray : 0);
  const float* d = D + 3 * (in_range ? ray : 0);

  // distortion regulariser (dL/d dist_loss of this ray, 0 if none): running
  // sums of w, w m, w (m W_< - S_<) and w^2 over the samples
  const float gdist = (grad_dist && in_range) ? grad_dist[ray] : 0.0f;
  float dW = 0.0f, dS = 0.0f, dP = 0.0f, dQ = 0.0f;

  // ---------------- pass 1: forward (or the forward's C_d and F, given:
  // the same float32 values, so pass 1 is skipped; not with the regulariser,
  // whose sums pass 1 also takes)
  MarchState m;
  float T = 1.0f, cd[3] = {0.f, 0.f, 0.f}, fv[4] = {0.f, 0.f, 0.f, 0.f};
  int ns = 0, reads = 0;
  // the wave's next samples; false when none of its rays goes on
  auto next_samples = [&](bool& have, float u[3], int& ks) -> bool {
    float t;
    int reads_at;
    have = march_slots<DOM, PYR, SLOTS>(S, m, slot, reads, u, t, ks, reads_at);
    return __ballot(have) != 0;
  };
  // the transmittance chain over the ray's new samples, in order (e: this
  // lane's exp(-sigma step)): before = T in front of this lane's sample, used =
  // the ray had not ended before it; T, ns and the ray's end move on
  auto advance = [&](bool have, float e, float& before, bool& used, int& my_ns) {
    const uint32_t bits = slot_bits<SLOTS>(have, lane);
    bool ended = false;
    before = T;
    used = false;
    each_slot<SLOTS>([&](auto J) {
      const float ej = slot_value<SLOTS, J>(e);
      if (((bits >> J) & 1u) && !ended) {
        if (slot == J) {
          before = T;
          used = true;
          my_ns = ns;
        }
        T = T * ej;
        ++ns;
        ended = T < S.thr || ns >= S.max_samples;
      }
    });
    if (ended) m.done = true;
  };
  if (fcd) {
    if (in_range) {
#pragma unroll
      for (int j = 0; j < 3; ++j) cd[j] = fcd[ray * 3 + j];
#pragma unroll
      for (int j = 0; j < 4; ++j) fv[j] = ffv[ray * 4 + j];
    }
  } else {
    march_init<DOM>(S, o, d, in_range, m);
    for (;;) {
      float u[3] = {0.f, 0.f, 0.f};
      int ks = 0;
      bool have;
      if (!next_samples(have, u, ks)) break;
      float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, e = 1.0f;
      if (have) {
        NoSink sink;
        eval_sample<MODEL, DT_F32, LMAX>(S, u, f, sink);
        e = exp32(-(exp32(f[0]) * S.step));
      }
      float before;
      bool used;
      int my_ns = 0;
      advance(have, e, before, used, my_ns);
      const float w = before * (1.0f - e);
      const float mid = ((float)ks + 0.5f) * S.step;
      const uint32_t bits = slot_bits<SLOTS>(used, lane);
      // the forward's sums, sample after sample, on every lane of the ray
      each_slot<SLOTS>([&](auto J) {
        const float wj = slot_value<SLOTS, J>(w), mj = slot_value<SLOTS, J>(mid);
        float fj[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) fj[c] = slot_value<SLOTS, J>(f[1 + c]);
        if ((bits >> J) & 1u) {
#pragma unroll
          for (int c = 0; c < 3; ++c) cd[c] = __builtin_fmaf(wj, fj[c], cd[c]);
#pragma unroll
          for (int c = 0; c < 4; ++c) fv[c] = __builtin_fmaf(wj, fj[3 + c], fv[c]);
          if (gdist != 0.0f) {
            dP = __builtin_fmaf(wj, mj * dW - dS, dP);
            dQ = __builtin_fmaf(wj, wj, dQ);
            dW = dW + wj;
            dS = __builtin_fmaf(wj, mj, dS);
          }
        }
      });
    }
  }

  float gcd[3], gfv[4];
  if (ups) {
    // dL/dC_d and dL/dF given per ray (the view-dependent MLP's adjoint):
    // no MLP here, no MLP partials
#pragma unroll
    for (int j = 0; j < 3; ++j) gcd[j] = in_range ? ups[ray * 7 + j] : 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) gfv[j] = in_range ? ups[ray * 7 + 3 + j] : 0.0f;
  } else {
    // ---------------- deferred MLP forward + backward (per lane)
    float x[8] = {cd[0], cd[1], cd[2], fv[0], fv[1], fv[2], fv[3], 1.0f};
    float z1[16], h1[16], z2[16], h2[16], oo[3];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float a = P[112 + i];
#pragma unroll
      for (int k = 0; k < 7; ++k) a = __builtin_fmaf(P[i * 7 + k], x[k], a);
      z1[i] = a;
      h1[i] = fmaxf(a, 0.0f);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float a = P[384 + i];
#pragma unroll
      for (int k = 0; k < 16; ++k) a = __builtin_fmaf(P[128 + i * 16 + k], h1[k], a);
      z2[i] = a;
      h2[i] = fmaxf(a, 0.0f);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      float a = P[448 + i];
#pragma unroll
      for (int k = 0; k < 16; ++k) a = __builtin_fmaf(P[400 + i * 16 + k], h2[k], a);
      oo[i] = a;
    }
    float gz[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const float C = 1.0f / (1.0f + __expf(-(cd[j] + oo[j])));
      const float g = in_range ? grad_rgb[ray * 3 + j] : 0.0f;
      gz[j] = g * C * (1.0f - C);
    }
    float gz2[16], gz1[16], gx[7];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      float a = 0.0f;
#pragma unroll
      for (int i = 0; i < 3; ++i) a = __builtin_fmaf(P[400 + i * 16 + k], gz[i], a);
      gz2[k] = z2[k] > 0.0f ? a : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      float a = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) a = __builtin_fmaf(P[128 + i * 16 + k], gz2[i], a);
      gz1[k] = z1[k] > 0.0f ? a : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      float a = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) a = __builtin_fmaf(P[i * 7 + k], gz1[i], a);
      gx[k] = a;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) gcd[j] = gz[j] + gx[j];
#pragma unroll
    for (int j = 0; j < 4; ++j) gfv[j] = gx[3 + j];

    // ---------------- MLP weight gradients: sums over the workgroup's rays on
    // MFMA by its first wave (a ray's first lane stages its row; rows beyond
    // kRays, if any, are zero)
    float* sA = stage_all[0];
    float* sB = stage_all[0] + 64 * kPad;
    const bool first = slot == 0;
    float* part = partial + int64_t(blockIdx.x) * kMlpParams;
    const int qi = lane >> 4, col = lane & 15;
    if (kRays < 64 && int(threadIdx.x) >= kRays && int(threadIdx.x) < 64) {
#pragma unroll
      for (int i = 0; i < 16; ++i) sA[threadIdx.x * kPad + i] = sB[threadIdx.x * kPad + i] = 0.0f;
    }
    float* rowA = sA + ray_in_block * kPad;
    float* rowB = sB + ray_in_block * kPad;
    // W0 (16 x 7) and b0 (column 7 of x is 1)
    if (first) {
#pragma unroll
      for (int i = 0; i < 16; ++i) rowA[i] = gz1[i];
#pragma unroll
      for (int j = 0; j < 16; ++j) rowB[j] = j < 8 ? x[j < 8 ? j : 0] : 0.0f;
    }
    __syncthreads();
    if (wave == 0) {
      bf32x4 r = wave_outer_sum(sA, sB, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 4 * qi + q;
        if (col < 7) part[i * 7 + col] = r[q];
        else if (col == 7) part[112 + i] = r[q];
      }
    }
    __syncthreads();
    // W1 (16 x 16) and b1
    if (first) {
#pragma unroll
      for (int i = 0; i < 16; ++i) rowA[i] = gz2[i];
#pragma unroll
      for (int j = 0; j < 16; ++j) rowB[j] = h1[j];
    }
    __syncthreads();
    if (wave == 0) {
      bf32x4 r = wave_outer_sum(sA, sB, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) part[128 + (4 * qi + q) * 16 + col] = r[q];
      if (lane < 16) {
        float a = 0.0f;
        for (int rr = 0; rr < kRays; ++rr) a += sA[rr * kPad + lane];
        part[384 + lane] = a;
      }
    }
    __syncthreads();
    // W2 (3 x 16) and b2
    if (first) {
#pragma unroll
      for (int i = 0; i < 16; ++i) rowA[i] = i < 3 ? gz[i < 3 ? i : 0] : 0.0f;
#pragma unroll
      for (int j = 0; j < 16; ++j) rowB[j] = h2[j];
    }
    __syncthreads();
    if (wave == 0) {
      bf32x4 r = wave_outer_sum(sA, sB, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 4 * qi + q;
        if (i < 3) part[400 + i * 16 + col] = r[q];
      }
      if (lane < 3) {
        float a = 0.0f;
        for (int rr = 0; rr < kRays; ++rr) a += sA[rr * kPad + lane];
        part[448 + lane] = a;
      }
    }
  }
  const float Ldist = 2.0f * dP + dQ * (S.step * (1.0f / 3.0f));
  const float Stot = gdist * (2.0f * Ldist) + (gcd[0] * cd[0] + gcd[1] * cd[1] + gcd[2] * cd[2]) +
                     (gfv[0] * fv[0] + gfv[1] * fv[1] + gfv[2] * fv[2] + gfv[3] * fv[3]);

  // ---------------- pass 2: re-march and scatter
  // Every lane takes part in each iteration (lanes without a sample carry no
  // gradient) so that the wave can merge the samples of equal cells.
  __syncthreads();
  march_init<DOM>(S, o, d, in_range, m);
  T = 1.0f;
  ns = 0;
  float Pc = 0.0f, rW = 0.0f, rS = 0.0f;
  const size_t T_entries = size_t(1) << S.log2T;
  float* stage = stage_all[wave];
  for (;;) {
    float u[3] = {0.f, 0.f, 0.f};
    int ks = 0;
    bool have;
    if (!next_samples(have, u, ks)) break;
    GradSink<LMAX> q;
    q.gcd = gcd;
    q.gfv = gfv;
    float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, sigma = 0.0f, e = 1.0f;
    if (have) {
      eval_sample<MODEL, DT_F32, LMAX>(S, u, f, q);
      sigma = exp32(f[0]);
      e = exp32(-(sigma * S.step));
    }
    float before;
    bool used;
    int my_ns = 0;
    advance(have, e, before, used, my_ns);
    have = used;
    const float w = before * (1.0f - e);
    const float scol = (gcd[0] * f[1] + gcd[1] * f[2] + gcd[2] * f[3]) +
                       (gfv[0] * f[4] + gfv[1] * f[5] + gfv[2] * f[6] + gfv[3] * f[7]);
    float s = scol;
    const uint32_t bits = slot_bits<SLOTS>(used, lane);
    if (gdist != 0.0f) {
      // dL_dist/dw_i = 2 sum_j w_j |m_i - m_j| + 2/3 step w_i (prefix sums over j < i)
      const float mid = ((float)ks + 0.5f) * S.step;
      float myW = rW, myS = rS;
      each_slot<SLOTS>([&](auto J) {
        const float wj = slot_value<SLOTS, J>(w), mj = slot_value<SLOTS, J>(mid);
        if (slot == J) {
          myW = rW;
          myS = rS;
        }
        if ((bits >> J) & 1u) {
          rW = rW + wj;
          rS = __builtin_fmaf(wj, mj, rS);
        }
      });
      const float pair = (mid * myW - myS) + ((dS - myS - w * mid) - mid * (dW - myW - w));
      s = __builtin_fmaf(gdist, 2.0f * pair + (2.0f / 3.0f) * S.step * w, s);
    }
    float myP = Pc;
    each_slot<SLOTS>([&](auto J) {
      const float wj = slot_value<SLOTS, J>(w), sj = slot_value<SLOTS, J>(s);
      if ((bits >> J) & 1u) Pc = __builtin_fmaf(wj, sj, Pc);
      if (slot == J) myP = Pc;
    });
    float gf[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (have) {
      const float gsig = S.step * (before * e * s - (Stot - myP));
      gf[0] = sigma * gsig;
#pragma unroll
      for (int j = 0; j < 3; ++j) gf[1 + j] = w * gcd[j];
#pragma unroll
      for (int j = 0; j < 4; ++j) gf[4 + j] = w * gfv[j];
    }
    if constexpr (MODEL == 1) {
      baked_scatter<LMAX>(S, u, have, gf, w, q, gtab, tstride, gatlas, lane, stage);
      continue;
    }
#pragma unroll 1
    for (int l = 0; l < S.L; ++l) {
      Corners c;
      level_corners(u, S.N[l], S.Nf[l], S.mask, c);
      float gv[9];
#pragma unroll
      for (int j = 0; j < 9; ++j) gv[j] = 0.0f;
      if (have) {
        const float wl = exp32(q.a[l] - q.run_max) / q.esum;
        // dL/df . (v_l - f), the differences first: they are exact or nearly so
        // where the products would cancel
        const float dot = __builtin_fmaf(gf[0], q.A[l] - f[0], w * (q.B[l] - scol));
#pragma unroll
        for (int j = 0; j < 8; ++j) gv[j] = wl * gf[j];
        gv[8] = wl * dot;
      }
      if (det.off) {
        // deterministic mode: every contribution to its own record
        if (have) {
          const int64_t base = ((det.off[ray] + my_ns) * S.L + l) * 8;
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int64_t rec = base + k;
            if (rec >= det.n) break;
            det.keys[rec] = uint32_t(l) * uint32_t(T_entries) + c.idx[k];
            det.order[rec] = uint32_t(rec);
#pragma unroll
            for (int j = 0; j < 9; ++j) det.vals[rec * 9 + j] = c.w[k] * gv[j];
          }
        }
      } else {
        scatter_cells<9>(gtab + (size_t(l) * T_entries) * size_t(tstride), tstride, 9, have, c.key0, c.key1, c.idx,
                         c.w, gv, lane, stage);
      }
    }
  }
}

__global__ void adam_kernel(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                            float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// Lanes a ray of the backward.  A ray's samples are a serial chain, and at
// four lanes a ray the chain is a quarter as long and four times the waves
// share the chip, for a few evaluations past a ray's end; small batches do not
// fill the chip even so and take sixteen.  Measured (training step, tables
// 8 x 2^14): 2^18 rays at 1 / 2 / 4 / 8 / 16 lanes a ray 3.70 / 3.15 / 3.17 /
// 3.83 / 5.41 ms, 2^15 rays 2.14 / 1.25 / 0.97 / 0.95 / 1.25, 2^14 rays 1.93 /
// 1.27 / 0.90 / 0.82 / 0.86 (0.89 at 4 and 0.76 at 16 with the fill rule of
// march_slots), 2^10 rays 2.29 / 1.24 / 0.83 / 0.67 / 0.64 ms.
// Lanes past a ray's last sample look up for nothing, so rays of about one
// sample lose by it (16 x 2^19 tables, 16,384 rays of 1.2 samples .38 ms with one
// lane a ray, .48 so; 2^18 rays 1.20 against 1.82, .25 of it padded rows); from
// 2.5 samples on they gain.
static int backward_slots(int64_t n) { return n <= 16384 ? 16 : 4; }

// workgroups of m rays of a batch of n
static int64_t backward_blocks(int64_t m, int64_t n) {
  const int64_t rays = 256 / backward_slots(n);          // per workgroup
  return (m + rays - 1) / rays;
}
static int64_t backward_blocks(int64_t n) { return backward_blocks(n, n); }

// Rays of one launch, a multiple of a workgroup's: a launch holds fewer than
// 2^32 threads, and these are 2^31 at four lanes a ray.
constexpr int64_t kLaunchRays = int64_t(1) << 29;

size_t backward_workspace_bytes(int64_t n) {
  return (size_t(backward_blocks(n)) + kSumGroups) * kMlpParams * sizeof(float);
}

static bool is_baked_model(const ngprt_ctx* ctx) { return ctx->desc.feature_model == NGPRT_MODEL_BAKED; }

// Padded gradient rows of the tables.  The memory side takes float atomics by
// 64-byte requests: a 36-byte row on its 36-byte stride costs 1.5 of them on
// average, a row on a 64-byte line of its own costs one (13.9 and 20.9 G rows a
// second).  So the scatter goes to rows of 16 floats of the context's, which are
// then added to the caller's.  (The baked model's atlas rows of 10 to 16 floats
// gain nothing by it: 2^18 rays on 124,416 to 1.6 M atlas rows, 1.74 to 1.81 ms
// without, 1.78 to 1.84 with.)
constexpr int kPadRow = 16;
constexpr size_t kPadMaxBytes = size_t(1) << 30;

// Whether n rays' scatter into tables of T rows a level pays for them: they cost
// 200 bytes a row to clear, read and add, and save a part of each row sent.
// Measured, ms of a backward padded / not, rays of 15 to 17 samples:
//   rays =          T/16         T/8          T/4          T/2
//   8 x 2^14, box   .196 / .186  .213 / .203  .208 / .221  .252 / .268
//   16 x 2^17, box  .944 / .956  1.57 / 1.64  2.50 / 2.80  4.25 / 4.68
//   16 x 2^19, box  3.14 / 3.16  4.70 / 4.80  5.16 / 5.34  11.3 / 11.9
//   same, contr.    3.27 / 3.13  4.72 / 4.54  8.03 / 7.90  14.5 / 14.7
//   16 x 2^20, box  5.05 / 5.03  5.63 / 5.39  12.5 / 12.8  21.2 / 22.5
// so from T/5 on; rays of three samples break even at T/2 to T (16 x 2^19: T/16
// .870 / .591, T/4 1.24 / .99, T 4.03 / 4.03).  The baked model's rows, of 8
// channels and on few levels, break even at T/2 (2 x 2^14: T/4 .162 / .157, T/2
// .208 / .209, T .319 / .322, 16 T 1.78 / 1.89).
static bool pad_pays(int64_t n, int64_t T, int64_t levels, bool baked) {
  return n >= (baked ? T / 2 : T / 5) && size_t(levels * T) * kPadRow * sizeof(float) <= kPadMaxBytes;
}

__global__ void clear_rows_kernel(float4* __restrict__ p, int64_t n) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// dst[9 r + c] += src[r * kPadRow + c] for the first nv of a row's 9 channels, by
// atomics like every other addition to a caller's rows: contexts on other
// streams may be adding to the same gradient.  n = 9 rows < 2^32 (kPadMaxBytes
// holds 2^24 rows).
__global__ void add_rows_kernel(const float* __restrict__ src, float* __restrict__ dst, uint32_t n, uint32_t nv) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t r = i / 9, c = i - r * 9;
  if (c >= nv) return;
  const float v = src[size_t(r) * kPadRow + c];
  if (v != 0.0f) unsafeAtomicAdd(dst + i, v);
}

static int launch_add_rows(ngprt_ctx* ctx, const float* src, float* dst, int64_t rows, int nv, hipStream_t st) {
  const uint32_t n = uint32_t(rows) * 9u;
  hipLaunchKernelGGL(add_rows_kernel, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, n, uint32_t(nv));
  return check_launch(ctx, "add_rows_kernel");
}

// The context's padded rows, grown to `bytes`; NULL when they cannot be had.
// They are kept apart from the workspace: a backward needs the workspace, the
// padded rows only make its scatter faster, so a device too full for them still
// trains (on the caller's rows).  Nor are they taken while the stream is being
// captured: that memory would be the graph's, and the context keeps it.
// The rows begin kPadShift into their buffer: large buffers, the tables' too,
// start on 2 MiB boundaries, and rows aligned alike cost the steps more (a
// step's time with the rows at 0 / 6,464 / 2^20 / 2^20 + 6,464 bytes: 8 x 2^14
// tables 2.64 / 2.56 / 2.62 / 2.50 ms, 16 x 2^19 13.83 / 13.74 / 13.93 / 13.77).
constexpr size_t kPadShift = (size_t(1) << 20) + 101 * 64;
static float* padded_rows(ngprt_ctx* ctx, size_t bytes, hipStream_t st) {
  bytes += kPadShift;
  if (bytes > ctx->pad_bytes) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      return nullptr;
    }
    if (ctx->pad_rows) (void)hipFreeAsync(ctx->pad_rows, st);
    ctx->pad_rows = nullptr;
    ctx->pad_bytes = 0;
    if (dev_malloc_async((void**)&ctx->pad_rows, bytes, st) != hipSuccess) {
      (void)hipGetLastError();
      ctx->pad_rows = nullptr;
      return nullptr;
    }
    ctx->pad_bytes = bytes;
  }
  return reinterpret_cast<float*>(reinterpret_cast<char*>(ctx->pad_rows) + kPadShift);
}

int launch_backward(ngprt_ctx* ctx, int64_t n, const float* o, const float* d, const float* grad_rgb,
                    const float* grad_dist, const float* ups, const float* fcd, const float* ffv,
                    float* gtab, float* gatlas, float* gmlp, hipStream_t st) {
  if (backward_blocks(n) > 0x7FFFFFFF) return fail(ctx, NGPRT_E_SHAPE, "too many rays");
  const bool baked = is_baked_model(ctx);
  const size_t need = backward_workspace_bytes(n);
  if (need > ctx->ws_bytes) {
    if (ctx->ws) (void)hipFreeAsync(ctx->ws, st);
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
    if (dev_malloc_async((void**)&ctx->ws, need, st) != hipSuccess) {
      (void)hipGetLastError();
      return fail(ctx, NGPRT_E_ALLOC, "backward workspace allocation failed");
    }
    ctx->ws_bytes = need;
  }
  float* partial = reinterpret_cast<float*>(ctx->ws);
  if (ctx->det_grad) {
    if (baked) return fail(ctx, NGPRT_E_UNSUPPORTED, "deterministic gradients are built for the hash model");
    return launch_backward_det(ctx, n, o, d, grad_rgb, grad_dist, ups, fcd, ffv, gtab, gmlp, partial, st);
  }
  const int64_t trows = int64_t(ctx->desc.n_levels) * ctx->T;
  const size_t floats = size_t(trows) * kPadRow;
  float* rows = pad_pays(n, ctx->T, ctx->desc.n_levels, baked) ? padded_rows(ctx, floats * sizeof(float), st) : nullptr;
  if (rows) {
    const int64_t n4 = int64_t(floats / 4);
    hipLaunchKernelGGL(clear_rows_kernel, dim3(unsigned((n4 + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<float4*>(rows), n4);
    int rc = check_launch(ctx, "clear_rows_kernel");
    if (rc) return rc;
  }
  int rc = launch_backward_ws(ctx, n, o, d, grad_rgb, grad_dist, ups, fcd, ffv, rows ? rows : gtab, rows ? kPadRow : 9,
                              gatlas, gmlp, partial, st);
  if (rc == NGPRT_OK && rows) rc = launch_add_rows(ctx, rows, gtab, trows, baked ? 8 : 9, st);
  return rc;
}

int launch_backward_ws(ngprt_ctx* ctx, int64_t n, const float* o, const float* d, const float* grad_rgb,
                       const float* grad_dist, const float* ups, const float* fcd, const float* ffv,
                       float* gtab, int tstride, float* gatlas, float* gmlp, float* partial,
                       hipStream_t st, const DetRecords& det) {
  SceneArgs S = scene_args(ctx);
  const int64_t blocks = backward_blocks(n);
  if (blocks > 0x7FFFFFFF) return fail(ctx, NGPRT_E_SHAPE, "too many rays");
  const bool box = ctx->desc.domain == DOM_BOX;
  const bool wide = backward_slots(n) == 16;
#define NGPRT_BW_S(DOMV, LM, PY, MD, SL)                                                               \
  hipLaunchKernelGGL((backward_kernel<DOMV, LM, PY, MD, SL>), g, dim3(256), 0, st, S, m, o + 3 * at, d + 3 * at, \
                     from(grad_rgb, 3), from(grad_dist, 1), from(ups, 7), from(fcd, 3), from(ffv, 4), gtab,    \
                     tstride, gatlas, part, ctx->mlp, rec)
#define NGPRT_BW(DOMV, LM, PY, MD)          \
  if (wide) NGPRT_BW_S(DOMV, LM, PY, MD, 16); \
  else NGPRT_BW_S(DOMV, LM, PY, MD, 4)
#define NGPRT_BW_DOM(LM, PY, MD)         \
  if (box) {                             \
    NGPRT_BW(DOM_BOX, LM, PY, MD);       \
  } else {                               \
    NGPRT_BW(DOM_CONTRACT, LM, PY, MD);  \
  }
  for (int64_t at = 0; at < n; at += kLaunchRays) {
    const int64_t m = n - at < kLaunchRays ? n - at : kLaunchRays;
    const dim3 g(unsigned(backward_blocks(m, n)));
    auto from = [at](const float* p, int width) { return p ? p + width * at : nullptr; };
    float* part = partial + backward_blocks(at, n) * kMlpParams;
    DetRecords rec = det;
    if (rec.off) rec.off += at;
    if (S.model == NGPRT_MODEL_BAKED) {
      // L <= 2 fine levels: coarse rows of at most 12 channels
      if (S.L <= 2 && S.pyr_n > 0) {
        NGPRT_BW_DOM(2, true, 1)
      } else if (S.L <= 2) {
        NGPRT_BW_DOM(2, false, 1)
      } else if (S.pyr_n > 0) {
        NGPRT_BW_DOM(4, true, 1)
      } else {
        NGPRT_BW_DOM(4, false, 1)
      }
    } else if (S.pyr_n > 0) {
      NGPRT_BW_DOM(16, true, 0)
    } else if (S.L <= 8) {
      NGPRT_BW_DOM(8, false, 0)
    } else {
      NGPRT_BW_DOM(16, false, 0)
    }
  }
#undef NGPRT_BW_DOM
#undef NGPRT_BW
#undef NGPRT_BW_S
  int rc = check_launch(ctx, "backward_kernel");
  if (rc || ups) return rc;
  return launch_partial_sums(ctx, partial, blocks, kMlpParams, partial + size_t(blocks) * kMlpParams, gmlp, st);
}

int launch_adam(int64_t n, float* p, const float* g, float* m, float* v, int32_t step, float lr, float b1,
                float b2, float eps, hipStream_t st) {
  const double c1 = 1.0 / (1.0 - std::pow(double(b1), double(step)));
  const double c2 = 1.0 / (1.0 - std::pow(double(b2), double(step)));
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(adam_kernel, dim3(unsigned(blocks)), dim3(256), 0, st, n, p, g, m, v, lr, b1, b2, eps,
                     float(c1), float(c2));
  return hipGetLastError() == hipSuccess ? NGPRT_OK : NGPRT_E_HIP;
}

}  // namespace ngprt
