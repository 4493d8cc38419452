// Launches of the one-launch forward layer for wide layers (layer_forward_wide.hpp).
#include "layer_forward_wide.hpp"

namespace snn {

hipError_t layer_forward_wide(hipStream_t st, const LayerForwardArgs &a) {
  const dim3 grid((unsigned)(((a.B + 1) / 2 + 7) / 8 * 8 * a.parts));
  if (a.nt_store) hipLaunchKernelGGL(lif_layer_forward_wide_kernel<NT>, grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL(lif_layer_forward_wide_kernel<0>, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace snn
