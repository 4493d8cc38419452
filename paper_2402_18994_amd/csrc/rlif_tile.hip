// Launches of the recurrent kernels for layers of up to 256 neurons (rlif_tile.hpp).
#include "rlif_tile.hpp"

namespace snn {

// Steps of 32 neurons of the contraction, rounded up to the sizes the kernels are compiled for.
static int tile_steps(int ld) { return ld <= 64 ? 2 : ld <= 128 ? 4 : ld <= 192 ? 6 : 8; }

hipError_t rlif_tile_forward(hipStream_t st, bool fp32, int T, int B, int ld, const float *I, float *V, uint8_t *S,
                             const uint16_t *QRf, int ldqr, long long qr_plane, const float *beta, float theta) {
  const dim3 grid((B + 3) / 4), block(64 * ((ld + 31) / 32));
#define SNN_RTF(KS)                                                                                                    \
  do {                                                                                                                 \
    if (fp32) hipLaunchKernelGGL((rlif_tile_forward_kernel<3, KS>), grid, block, 0, st, I, V, S, QRf, ldqr, qr_plane, T, B, ld, beta, theta); \
    else hipLaunchKernelGGL((rlif_tile_forward_kernel<1, KS>), grid, block, 0, st, I, V, S, QRf, ldqr, qr_plane, T, B, ld, beta, theta); \
  } while (0)
  switch (tile_steps(ld)) { case 2: SNN_RTF(2); break; case 4: SNN_RTF(4); break; case 6: SNN_RTF(6); break; default: SNN_RTF(8); break; }
#undef SNN_RTF
  return hipGetLastError();
}

template <int NP, int SURR>
static hipError_t reverse(hipStream_t st, int T, int B, int ld, const float *dS, const float *V, uint32_t *dI, const uint16_t *QRb,
                          int ldqr, long long qr_plane, const float *beta, float theta, float slope, float *db_part) {
  const dim3 grid((B + 3) / 4), block(64 * ((ld + 31) / 32));
#define SNN_RTR(KS)                                                                                                    \
  hipLaunchKernelGGL((rlif_tile_reverse_kernel<NP, SURR, KS>), grid, block, 0, st, dS, V, dI, QRb, ldqr, qr_plane, T, B, ld, beta, theta, slope, db_part)
  switch (tile_steps(ld)) { case 2: SNN_RTR(2); break; case 4: SNN_RTR(4); break; case 6: SNN_RTR(6); break; default: SNN_RTR(8); break; }
#undef SNN_RTR
  return hipGetLastError();
}

hipError_t rlif_tile_reverse(hipStream_t st, bool fp32, int T, int B, int ld, const float *dS, const float *V, uint32_t *dI,
                             const uint16_t *QRb, int ldqr, long long qr_plane, const float *beta, float theta, int surrogate,
                             float slope, float *db_part) {
#define SNN_RTS(SU)                                                                                                    \
  return fp32 ? reverse<3, SU>(st, T, B, ld, dS, V, dI, QRb, ldqr, qr_plane, beta, theta, slope, db_part)              \
              : reverse<1, SU>(st, T, B, ld, dS, V, dI, QRb, ldqr, qr_plane, beta, theta, slope, db_part)
  switch (surrogate) {
    case 0: SNN_RTS(0);
    case 1: SNN_RTS(1);
    case 2: SNN_RTS(2);
    case 3: SNN_RTS(3);
    case 4: SNN_RTS(4);
    default: SNN_RTS(5);
  }
#undef SNN_RTS
}

}  // namespace snn
