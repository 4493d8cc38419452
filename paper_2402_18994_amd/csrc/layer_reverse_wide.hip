// Launches of the one-launch reverse layer below a wide layer (layer_reverse_wide.hpp).
#include "layer_reverse_wide.hpp"

namespace snn {

template <int SURR>
static hipError_t launch(hipStream_t st, const LayerReverseArgs &a) {
  const dim3 grid((unsigned)((a.B + 7) / 8 * 8 * ((a.ld + ReverseWide::BN - 1) / ReverseWide::BN)));
#define SNN_LRW(POL, AD) hipLaunchKernelGGL((lif_layer_reverse_wide_kernel<SURR, POL, AD>), grid, dim3(256), 0, st, a)
  if (a.A) { if (a.nt_store) SNN_LRW(NT, true); else SNN_LRW(0, true); }
  else { if (a.nt_store) SNN_LRW(NT, false); else SNN_LRW(0, false); }
#undef SNN_LRW
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
