// Render kernels of one family (render_kernel.h): the march alone.
#include "render_kernel.h"

namespace ngprt {

void render_march(NGPRT_DISPATCH_ARGS) {
  dispatch<MODE_MARCH, 1>(S, dom, dt, st, n, o, d, out, rec, mlp, naive, pa);
}

}  // namespace ngprt
