// Render kernels of one family (render_kernel.h): the plain render.
#include "render_kernel.h"

namespace ngprt {

void render_plain(NGPRT_DISPATCH_ARGS) {
  dispatch<MODE_RENDER, 1>(S, dom, dt, st, n, o, d, out, rec, mlp, naive, pa);
}

}  // namespace ngprt
