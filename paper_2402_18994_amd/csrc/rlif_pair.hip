// Launches of the paired recurrent layers (rlif_pair.hpp).
#include "rlif_pair.hpp"

namespace snn {

static int pair_steps(int ld) { return ld <= 64 ? 2 : ld <= 128 ? 4 : 6; }   // of 32 neurons

struct PairLaunch {
  hipStream_t st;
  const RlifPairArgs &a;
  bool reverse;
  dim3 grid() const { return dim3((unsigned)((a.B + 3) / 4)); }
  dim3 block() const {                                    // the product between the layers: a wavefront per 32 receiving neurons
    const int lo = (a.lo.ld + 31) / 32, up = (a.up.ld + 31) / 32;
    return dim3((unsigned)(64 * (lo + up + (reverse ? lo : up))));
  }
};
template <int K1, int K2>
static hipError_t launch(const PairLaunch &p) {
#define SNN_PAIR(SU) hipLaunchKernelGGL((rlif_pair_reverse_kernel<SU, K1, K2>), p.grid(), p.block(), 0, p.st, p.a)
  if (!p.reverse) hipLaunchKernelGGL((rlif_pair_forward_kernel<K1, K2>), p.grid(), p.block(), 0, p.st, p.a);
  else switch (p.a.surrogate) {
    case 0: SNN_PAIR(0); break;
    case 1: SNN_PAIR(1); break;
    case 2: SNN_PAIR(2); break;
    case 3: SNN_PAIR(3); break;
    case 4: SNN_PAIR(4); break;
    default: SNN_PAIR(5); break;
  }
#undef SNN_PAIR
  return hipGetLastError();
}
template <int K1>
static hipError_t launch_upper(const PairLaunch &p) {
  switch (pair_steps(p.a.up.ld)) {
    case 2: return launch<K1, 2>(p);
    case 4: return launch<K1, 4>(p);
    default: return launch<K1, 6>(p);
  }
}
static hipError_t launch_pair(const PairLaunch &p) {
  switch (pair_steps(p.a.lo.ld)) {
    case 2: return launch_upper<2>(p);
    case 4: return launch_upper<4>(p);
    default: return launch_upper<6>(p);
  }
}
hipError_t rlif_pair_forward(hipStream_t st, const RlifPairArgs &a) { return launch_pair({st, a, false}); }
hipError_t rlif_pair_reverse(hipStream_t st, const RlifPairArgs &a) { return launch_pair({st, a, true}); }

}  // namespace snn
