// Launches of the paired recurrent layers (rlif_pair.hpp).
#include "rlif_pair.hpp"

namespace snn {

static int pair_steps(int ld) { return ld <= 64 ? 2 : ld <= 128 ? 4 : 6; }   // of 32 neurons

template <int K1, int K2>
static hipError_t launch(hipStream_t st, const RlifPairArgs &a, bool reverse) {
  const dim3 grid((a.B + 3) / 4), block(64 * ((a.lo.ld + 31) / 32 + (a.up.ld + 31) / 32));
  if (reverse) hipLaunchKernelGGL((rlif_pair_reverse_kernel<K1, K2>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((rlif_pair_forward_kernel<K1, K2>), grid, block, 0, st, a);
  return hipGetLastError();
}
template <int K1>
static hipError_t launch_upper(hipStream_t st, const RlifPairArgs &a, bool reverse) {
  switch (pair_steps(a.up.ld)) {
    case 2: return launch<K1, 2>(st, a, reverse);
    case 4: return launch<K1, 4>(st, a, reverse);
    default: return launch<K1, 6>(st, a, reverse);
  }
}
static hipError_t launch_pair(hipStream_t st, const RlifPairArgs &a, bool reverse) {
  switch (pair_steps(a.lo.ld)) {
    case 2: return launch_upper<2>(st, a, reverse);
    case 4: return launch_upper<4>(st, a, reverse);
    default: return launch_upper<6>(st, a, reverse);
  }
}
hipError_t rlif_pair_forward(hipStream_t st, const RlifPairArgs &a) { return launch_pair(st, a, false); }
hipError_t rlif_pair_reverse(hipStream_t st, const RlifPairArgs &a) { return launch_pair(st, a, true); }

}  // namespace snn
