// Launches of the one-launch reverse layer below a wide layer (layer_reverse_wide.hpp).
#include "layer_reverse_wide.hpp"

namespace snn {

template <int SURR>
static hipError_t launch(hipStream_t st, const LayerReverseArgs &a) {
  const int grid = (a.B + 7) / 8 * 8 * ((a.ld + ReverseWide::BN - 1) / ReverseWide::BN);
  if (a.nt_store) hipLaunchKernelGGL((lif_layer_reverse_wide_kernel<SURR, NT>), dim3((unsigned)grid), dim3(256), 0, st, a);
  else hipLaunchKernelGGL((lif_layer_reverse_wide_kernel<SURR, 0>), dim3((unsigned)grid), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t layer_reverse_wide(hipStream_t st, const LayerReverseArgs &a, int surrogate) {
  switch (surrogate) {
    case 0: return launch<0>(st, a);
    case 1: return launch<1>(st, a);
    case 2: return launch<2>(st, a);
    case 3: return launch<3>(st, a);
    case 4: return launch<4>(st, a);
    default: return launch<5>(st, a);
  }
}

}  // namespace snn
