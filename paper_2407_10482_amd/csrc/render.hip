// Launches of the render kernels (render_kernel.h) and the point evaluation of
// the parity checks.
#include <hip/hip_runtime.h>

#include "render_kernel.h"

namespace ngprt {

template <int DT, int LMAX, int MODEL>
__global__ void __launch_bounds__(256) eval_points_kernel(SceneArgs S, int64_t n,
                                                          const float* __restrict__ pos,
                                                          int32_t* idx, float* fused, float* weights) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float p[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
  float u[3];
  for (int a = 0; a < 3; ++a) u[a] = (p[a] - S.lo) * S.inv_ext;
  float f[8], w[LMAX];
  int32_t id[LMAX * 8];
  PointSink<LMAX> sink{w, id, S.L};
  eval_sample<MODEL, DT, LMAX>(S, u, f, sink);
  if (fused)
    for (int j = 0; j < 8; ++j) fused[i * 8 + j] = f[j];
  if (weights)
    for (int l = 0; l < S.L; ++l) weights[i * S.L + l] = w[l];
  if (idx)
    for (int l = 0; l < S.L; ++l)
      for (int k = 0; k < 8; ++k) idx[(i * S.L + l) * 8 + k] = id[l * 8 + k];
}

// Lanes a ray of a render without a proposal.  64 rays a wave leave most of the
// chip idle in a small launch, and every ray's march and its 15 to 20 lookups are
// serial chains that its lanes shorten; but lanes past a ray's last sample look
// up for nothing, and each lane of a contracted march follows its ray through
// all lanes' points, so the lanes cost more the fewer samples the rays take and
// the fuller the chip is.  Measured, 1 / 8 / 16 lanes a ray (ms), scenes of 15 to
// 17 samples a ray:
//   rays                     16,384             32,768             49,152             65,536             81,760
//   F32, 8 levels, box       .253 / .108 / .076 .265 / .128 / .129 .317 / .137 / .184 .325 / .179 / .239 .305 / .206 / .274
//   baked, pyramid, box      .213 / .089 / .066 .209 / .097 / .099 .233 / .108 / .124 .230 / .153 / .170 .232 / .164 / .195
//   F32, 16 levels, contr.   1.13 / .660 / .554 1.09 / .708 / .671 1.15 / .965 / .883 1.32 / 1.07 / 1.12 1.46 / 1.19 / 1.25
//   baked, pyramid, contr.   1.50 / .799 / .546 1.76 / .907 / .588 1.80 / .933 / .788 1.87 / .893 / .959 1.94 / 1.06 / 1.09
// and with one sample a ray (solid surfaces):
//   F32, 8 levels, box       .057 / .052 / .050 .058 / .060 / .088 .058 / .071 / .114 .058 / .088 / .154 .064 / .093 / .173
//   F32, 16 levels, contr.   .420 / .335 / .372 .415 / .396 / .501 .423 / .515 / .723 .410 / .587 / .921 .441 / .652 / 1.04
// Sixteen to where eight are no slower on the first, eight to where one lane is
// as good.  (Contracted rays that meet nothing at all pay most, .26 / .58 / 1.00 at
// 49,152; any share of rays that do sample hides it: one lane a ray is then bound
// by its longest rays.)  Rays cut off after at most three samples are of the
// second kind whatever the scene: one lane beyond 16,384 (box, one sample: 16
// lanes .050 at 16,384, .114 at 49,152).
static int render_lanes(const SceneArgs& S, int domain, int64_t n) {
  if (n > (S.max_samples < 4 ? 16384 : 81920)) return 1;
  return n <= (domain == DOM_BOX ? 28672 : 61440) ? kSmallSlots : kMidSlots;
}

int launch_render(ngprt_ctx* ctx, int64_t n, const float* o, const float* d, const RayOut& out,
                  const float* prop, bool use_net, float* prop_out, const ngprt_proposal_cfg& pc,
                  int32_t* fallback, hipStream_t st) {
  SceneArgs S = scene_args(ctx);
  if ((n + 63) / 64 > 0x7FFFFFFF) return fail(ctx, NGPRT_E_SHAPE, "too many rays for one launch");
  MarchRecord rec{nullptr, nullptr, nullptr, 0};
  const uint2* net_w = use_net ? reinterpret_cast<const uint2*>(ctx->prop_net) : nullptr;
  const float* net_b = use_net ? reinterpret_cast<const float*>(
                                     reinterpret_cast<const char*>(ctx->prop_net) + kPropTiles * 64 * 8)
                               : nullptr;
  ProposalArgs pa{prop,         net_w,           net_b,        use_net ? prop_out : nullptr,
                  pc.conf_threshold, pc.margin, pc.use_near, pc.far_guard, fallback};
  const bool ext = prop || use_net || out.t_first || out.t_far || out.t_half || out.dist_loss;
#define NGPRT_FAMILY(f) f(S, ctx->desc.domain, ctx->desc.table_dtype, st, n, o, d, out, rec, ctx->mlp, 0, pa)
  const int lanes = prop || use_net ? 1 : render_lanes(S, ctx->desc.domain, n);
  if (lanes == kSmallSlots) NGPRT_FAMILY(render_small);
  else if (lanes == kMidSlots) NGPRT_FAMILY(render_mid);
  else if (ext) NGPRT_FAMILY(render_ext);
  else NGPRT_FAMILY(render_plain);
#undef NGPRT_FAMILY
  int rc = check_launch(ctx, "render_kernel");
  if (rc == NGPRT_OK && S.view_mlp) rc = launch_view_mlp(ctx, n, d, out.c_d, out.feat, out.rgb, st);
  return rc;
}

int launch_march(ngprt_ctx* ctx, int64_t n, const float* o, const float* d, int32_t cap,
                 int32_t* sk, int32_t* ns, int32_t* nr, int naive, hipStream_t st) {
  SceneArgs S = scene_args(ctx);
  if ((n + 63) / 64 > 0x7FFFFFFF) return fail(ctx, NGPRT_E_SHAPE, "too many rays for one launch");
  MarchRecord rec{sk, ns, nr, cap};
  RayOut out{};
  ProposalArgs pa{nullptr, nullptr, nullptr, nullptr, 0.0f, 0.0f, 0, 0.0f, nullptr};
  render_march(S, ctx->desc.domain, ctx->desc.table_dtype, st, n, o, d, out, rec, ctx->mlp, naive, pa);
  return check_launch(ctx, "march_kernel");
}

int launch_eval_points(ngprt_ctx* ctx, int64_t n, const float* pos, int32_t* idx, float* fused,
                       float* weights, hipStream_t st) {
  SceneArgs S = scene_args(ctx);
  const int64_t blocks = (n + 255) / 256;
  if (blocks > 0x7FFFFFFF) return fail(ctx, NGPRT_E_SHAPE, "too many points for one launch");
  dim3 g = dim3(unsigned(blocks));
  const int dt = ctx->desc.table_dtype;
#define NGPRT_EV(DTV, LM, MD)                                                                   \
  hipLaunchKernelGGL((eval_points_kernel<DTV, LM, MD>), g, dim3(256), 0, st, S, n, pos, idx, fused, \
                     weights)
#define NGPRT_EV_DT(DTV)                   \
  if (dt == DTV) {                         \
    if (S.model == 1) NGPRT_EV(DTV, 4, 1); \
    else if (S.L <= 8) NGPRT_EV(DTV, 8, 0); \
    else NGPRT_EV(DTV, 16, 0);              \
  }
  if (S.model == 1 && S.gen)   // the ablation aggregations: float32 tables only (checked at create)
    NGPRT_EV(DT_F32, 4, 5);
  else {
    NGPRT_EV_DT(DT_F32)
  }
  NGPRT_EV_DT(DT_BF16)
  NGPRT_EV_DT(DT_FP8)
#undef NGPRT_EV_DT
#undef NGPRT_EV
  return check_launch(ctx, "eval_points_kernel");
}

}  // namespace ngprt
