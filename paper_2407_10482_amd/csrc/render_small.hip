// Render kernels of one family (render_kernel.h): small launches, several lanes a ray.
#include "render_kernel.h"

namespace ngprt {

void render_small(NGPRT_DISPATCH_ARGS) {
  dispatch<MODE_RENDER_EXT, kSmallSlots>(S, dom, dt, st, n, o, d, out, rec, mlp, naive, pa);
}

}  // namespace ngprt
