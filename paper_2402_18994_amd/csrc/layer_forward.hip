// Launches of the one-launch forward layers (layer_forward.hpp): which variant of the kernel runs.
#include "layer_forward_short.hpp"

namespace snn {

template <int TN, int READOUT, int NL, bool PK, int TS, int LS, int NP, bool FULL>
static hipError_t launch(hipStream_t st, const LayerForwardArgs &a, unsigned grid) {
  hipLaunchKernelGGL((lif_layer_forward_kernel<TN, 3, READOUT, NL, PK, TS, LS, NP, FULL>), dim3(grid), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <int TN, int READOUT, bool PK, int NP, bool FULL>
static hipError_t launch_layers(hipStream_t st, const LayerForwardArgs &a, const LayerForwardVariant &v, unsigned grid) {
  return v.layers == 2 ? launch<TN, READOUT, 2, PK, 1, 1, NP, FULL>(st, a, grid) : launch<TN, READOUT, 1, PK, 1, 1, NP, FULL>(st, a, grid);
}

template <int TN, int READOUT, bool PK>
static hipError_t launch_readout(hipStream_t st, const LayerForwardArgs &a, const LayerForwardVariant &v, unsigned grid) {
  if constexpr (TN == 2) {                              // on request, rounded weights and whole parts only
    if (v.layer_split) return launch<2, READOUT, 2, PK, 1, 2, 1, true>(st, a, grid);
    if (v.time_split) return v.layers == 2 ? launch<2, READOUT, 2, PK, 2, 1, 1, true>(st, a, grid) : launch<2, READOUT, 1, PK, 2, 1, 1, true>(st, a, grid);
  }
  if constexpr (READOUT != 1) {
    if (v.planes == 3) return v.full ? launch_layers<TN, READOUT, PK, 3, true>(st, a, v, grid) : launch_layers<TN, READOUT, PK, 3, false>(st, a, v, grid);
  }
  return v.full ? launch_layers<TN, READOUT, PK, 1, true>(st, a, v, grid) : launch_layers<TN, READOUT, PK, 1, false>(st, a, v, grid);
}

template <int TN, bool PK>
static hipError_t launch_packed(hipStream_t st, const LayerForwardArgs &a, const LayerForwardVariant &v, unsigned grid) {
  switch (v.readout) {
    case 0: return launch_readout<TN, 0, PK>(st, a, v, grid);
    case 1: return launch_readout<TN, 1, PK>(st, a, v, grid);
    case 2: return launch_readout<TN, 2, PK>(st, a, v, grid);
    default: return launch_readout<TN, 3, PK>(st, a, v, grid);
  }
}

template <int TN, bool READOUT, int NL, bool PK>
static hipError_t launch_slots(hipStream_t st, const LayerForwardArgs &a, const LayerForwardVariant &v, unsigned grid) {
  if (v.planes == 3) hipLaunchKernelGGL((lif_layer_forward_short_kernel<TN, READOUT, NL, PK, 3>), dim3(grid), dim3(256), 0, st, a);
  else hipLaunchKernelGGL((lif_layer_forward_short_kernel<TN, READOUT, NL, PK, 1>), dim3(grid), dim3(256), 0, st, a);
  return hipGetLastError();
}
template <int TN>
static hipError_t launch_short(hipStream_t st, const LayerForwardArgs &a, const LayerForwardVariant &v) {
  const int groups = (a.B + (128 >> a.slot_log2) - 1) >> (7 - a.slot_log2);
  const unsigned grid = (unsigned)((groups + 7) / 8 * 8 * a.parts);
  const int which = (v.readout ? 4 : 0) + (v.layers == 2 ? 2 : 0) + (v.packed ? 1 : 0);
  switch (which) {
    case 0: return launch_slots<TN, false, 1, false>(st, a, v, grid);
    case 1: return launch_slots<TN, false, 1, true>(st, a, v, grid);
    case 2: return launch_slots<TN, false, 2, false>(st, a, v, grid);
    case 3: return launch_slots<TN, false, 2, true>(st, a, v, grid);
    case 4: return launch_slots<TN, true, 1, false>(st, a, v, grid);
    case 5: return launch_slots<TN, true, 1, true>(st, a, v, grid);
    case 6: return launch_slots<TN, true, 2, false>(st, a, v, grid);
    default: return launch_slots<TN, true, 2, true>(st, a, v, grid);
  }
}

template <bool PK, int NP>
static hipError_t launch_adaptive(hipStream_t st, const LayerForwardArgs &a) {
  const int groups = (a.B + (128 >> a.slot_log2) - 1) >> (7 - a.slot_log2);
  const unsigned grid = (unsigned)((groups + 7) / 8 * 8 * a.parts);
  hipLaunchKernelGGL((lif_layer_forward_short_kernel<1, false, 1, PK, NP, true>), dim3(grid), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t layer_forward(hipStream_t st, const LayerForwardArgs &a, const LayerForwardVariant &v) {
  if (v.adaptive) {
    if (v.packed) return v.planes == 3 ? launch_adaptive<true, 3>(st, a) : launch_adaptive<true, 1>(st, a);
    return v.planes == 3 ? launch_adaptive<false, 3>(st, a) : launch_adaptive<false, 1>(st, a);
  }
  if (v.slots) return v.neurons == 64 ? launch_short<1>(st, a, v) : launch_short<2>(st, a, v);
  const unsigned grid = (unsigned)((a.B + 7) / 8 * 8 * a.parts * (v.time_split || v.layer_split ? 2 : 1));
  if (v.neurons == 64) return v.packed ? launch_packed<1, true>(st, a, v, grid) : launch_packed<1, false>(st, a, v, grid);
  return v.packed ? launch_packed<2, true>(st, a, v, grid) : launch_packed<2, false>(st, a, v, grid);
}

}  // namespace snn
