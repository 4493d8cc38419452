// Launches of the recurrent kernels for layers of up to 256 neurons (rlif_tile.hpp).
#include "rlif_tile.hpp"

namespace snn {

// Sixteen samples a workgroup instead of four once the four-sample grid is more than two workgroups a compute unit (256
// of them) and their wavefronts share the SIMDs: us at T = 32, rounded weights, forward / reverse, four and
// sixteen samples: 128 neurons, B = 2048: 18.2 / 23.7 and 19.5 / 23.8, 2304: 25.4 / 32.6 and 19.7 / 23.4, 8192: 77.5 /
// 88.6 and 52.3 / 81.6; 64 neurons, 2048: 10.7 / 14.1 and 12.5 / 13.5, 8192: 31.5 / 39.8 and 23.4 / 32.0; 32 neurons,
// 4096: 9.9 / 13.0 and 9.5 / 13.2, 8192: 16.9 / 21.1 and 13.2 / 17.4.  (fp32, 128 neurons, 2304: 32.6 / 39.7 and 21.0 / 36.4;
// 64, 3072: 15.7 / 19.0 and 13.8 / 22.2, 4608: 24.4 / 28.7 and 17.5 / 27.1: three planes of g times three
// of R share the columns of four samples.)
static bool sixteen(int B, int ld, bool three_planes_of_g = false) {
  return ld <= 128 && B > 2048 && (long long)B * ((ld + 31) / 32) >= (three_planes_of_g ? 9216 : 6144);
}

// Steps of 32 neurons of the contraction, each compiled: a step that multiplies nothing lies in the chain of every time step
// all the same (T = 200, B = 64, forward / reverse, us with a step too many and with those it needs: 30 neurons 30.1 / 37.6 and 29.6 /
// 32.2, 90: 43.7 / 57.0 and 42.6 / 50.5, 130: 68.5 / 79.2 and 62.5 / 70.0, 200: 87.5 / 99.9 and 77.5 / 85.5, fp32 130: 137 / 159 and
// 119 / 143).
static int tile_steps(int ld) { return (ld + 31) / 32; }

hipError_t rlif_tile_forward(hipStream_t st, bool fp32, int T, int B, int ld, const float *I, float *V, uint8_t *S,
                             const uint16_t *QRf, int ldqr, long long qr_plane, const float *beta, float theta) {
  if (sixteen(B, ld)) {
    const dim3 grid((B + 15) / 16), block(64 * ((ld + 15) / 16));
#define SNN_RTF(NP, KS) hipLaunchKernelGGL((rlif_tile16_forward_kernel<NP, KS>), grid, block, 0, st, I, V, S, QRf, ldqr, qr_plane, T, B, ld, beta, theta)
    if (ld <= 64) { if (fp32) SNN_RTF(3, 2); else SNN_RTF(1, 2); }
    else if (fp32) SNN_RTF(3, 4);
    else SNN_RTF(1, 4);
#undef SNN_RTF
    return hipGetLastError();
  }
  const dim3 grid((B + 3) / 4), block(64 * ((ld + 31) / 32));
#define SNN_RTF(KS)                                                                                                    \
  do {                                                                                                                 \
    if (fp32) hipLaunchKernelGGL((rlif_tile_forward_kernel<3, KS>), grid, block, 0, st, I, V, S, QRf, ldqr, qr_plane, T, B, ld, beta, theta); \
    else hipLaunchKernelGGL((rlif_tile_forward_kernel<1, KS>), grid, block, 0, st, I, V, S, QRf, ldqr, qr_plane, T, B, ld, beta, theta); \
  } while (0)
  switch (tile_steps(ld)) {
    case 1: SNN_RTF(1); break;
    case 2: SNN_RTF(2); break;
    case 3: SNN_RTF(3); break;
    case 4: SNN_RTF(4); break;
    case 5: SNN_RTF(5); break;
    case 6: SNN_RTF(6); break;
    case 7: SNN_RTF(7); break;
    default: SNN_RTF(8); break;
  }
#undef SNN_RTF
  return hipGetLastError();
}

template <int NP, int SURR>
static hipError_t reverse(hipStream_t st, int T, int B, int ld, const float *dS, const float *V, uint32_t *dI, const uint16_t *QRb,
                          int ldqr, long long qr_plane, const float *beta, float theta, float slope, float *db_part) {
  if (sixteen(B, ld, NP == 3)) {
    const dim3 grid((B + 15) / 16), block(64 * ((ld + 15) / 16));
#define SNN_RTR(KS)                                                                                                    \
  hipLaunchKernelGGL((rlif_tile16_reverse_kernel<NP, SURR, KS>), grid, block, 0, st, dS, V, dI, QRb, ldqr, qr_plane, T, B, ld, beta, theta, slope, db_part)
    if (ld <= 64) SNN_RTR(2); else SNN_RTR(4);
#undef SNN_RTR
    return hipGetLastError();
  }
  const dim3 grid((B + 3) / 4), block(64 * ((ld + 31) / 32));
#define SNN_RTR(KS)                                                                                                    \
  hipLaunchKernelGGL((rlif_tile_reverse_kernel<NP, SURR, KS>), grid, block, 0, st, dS, V, dI, QRb, ldqr, qr_plane, T, B, ld, beta, theta, slope, db_part)
  switch (tile_steps(ld)) {
    case 1: SNN_RTR(1); break;
    case 2: SNN_RTR(2); break;
    case 3: SNN_RTR(3); break;
    case 4: SNN_RTR(4); break;
    case 5: SNN_RTR(5); break;
    case 6: SNN_RTR(6); break;
    case 7: SNN_RTR(7); break;
    default: SNN_RTR(8); break;
  }
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
