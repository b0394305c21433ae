// Render kernels of one family (render_kernel.h): launches between the small and the large ones.
#include "render_kernel.h"

namespace ngprt {

void render_mid(NGPRT_DISPATCH_ARGS) {
  dispatch<MODE_RENDER_EXT, kMidSlots>(S, dom, dt, st, n, o, d, out, rec, mlp, naive, pa);
}

}  // namespace ngprt
