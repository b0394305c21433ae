// Render kernels of one family (render_kernel.h): the render with label outputs or a proposal.
#include "render_kernel.h"

namespace ngprt {

void render_ext(NGPRT_DISPATCH_ARGS) {
  dispatch<MODE_RENDER_EXT, 1>(S, dom, dt, st, n, o, d, out, rec, mlp, naive, pa);
}

}  // namespace ngprt
