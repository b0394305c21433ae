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

// Launches of at most this many rays take kSmallSlots lanes a ray: 64 rays a
// wave leave most of the chip idle there, and every ray's march and its 15 to
// 20 lookups are serial chains that its lanes shorten.  Measured, one against
// sixteen lanes a ray (ms; 16,384 / 49,152 / 65,536 / 98,304 / 131,072 rays):
// float32, 8 levels in the box 0.305 / 0.307 / 0.329 / 0.295 / 0.299 against
// 0.080 / 0.194 / 0.244 / 0.329 / 0.424; 16 levels, contracted, 1.60 / 1.15 /
// 1.30 / 1.45 / 1.76 against 0.55 / 0.89 / 1.11 / 1.42 / 1.60; baked with the
// pyramid in the box 0.250 / 0.230 / 0.230 / 0.248 / 0.233 against 0.068 /
// 0.130 / 0.179 / 0.224 / 0.288: the lines cross around 90,000.
constexpr int64_t kSmallRays = 81920;

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
  if (!prop && !use_net && n <= kSmallRays) NGPRT_FAMILY(render_small);
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
