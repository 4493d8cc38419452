// Launches of the one-launch reverse layers (layer_reverse.hpp): which variant of the kernel runs.
#include "layer_reverse.hpp"

namespace snn {

template <int KS, int SURR, bool F32, bool FULL, bool SLOTS = false>
static hipError_t launch(hipStream_t st, const LayerReverseArgs &a) {
  const int groups = SLOTS ? (a.B + (64 >> a.slot_log2) - 1) >> (6 - a.slot_log2) : a.B;
  const int grid = (groups + 7) / 8 * 8 * ((a.ld + 63) / 64);
  hipLaunchKernelGGL((lif_layer_reverse_kernel<KS, SURR, F32, FULL, SLOTS>), dim3((unsigned)grid), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <int KS, int SURR>
static hipError_t launch_columns(hipStream_t st, const LayerReverseArgs &a, bool f32) {
  if (a.slot_log2 < 6) return f32 ? launch<KS, SURR, true, false, true>(st, a) : launch<KS, SURR, false, false, true>(st, a);
  const bool full = a.ld % 64 == 0;
  if (f32) return full ? launch<KS, SURR, true, true>(st, a) : launch<KS, SURR, true, false>(st, a);
  return full ? launch<KS, SURR, false, true>(st, a) : launch<KS, SURR, false, false>(st, a);
}

template <int SURR>
static hipError_t launch_surrogate(hipStream_t st, const LayerReverseArgs &a, bool f32) {
  if (a.ldc <= 32) return launch_columns<1, SURR>(st, a, f32);
  if (a.ldc <= 64) return launch_columns<2, SURR>(st, a, f32);
  return launch_columns<4, SURR>(st, a, f32);
}

hipError_t layer_reverse(hipStream_t st, const LayerReverseArgs &a, int surrogate, bool f32) {
  switch (surrogate) {
    case 0: return launch_surrogate<0>(st, a, f32);
    case 1: return launch_surrogate<1>(st, a, f32);
    case 2: return launch_surrogate<2>(st, a, f32);
    case 3: return launch_surrogate<3>(st, a, f32);
    case 4: return launch_surrogate<4>(st, a, f32);
    default: return launch_surrogate<5>(st, a, f32);
  }
}

}  // namespace snn
