// Which layers run on the kernels for wide layers (host arithmetic only).
#pragma once
#include <algorithm>

namespace snn {

// Below a WIDE layer (more than 128 columns; rounded weights) the whole reverse layer can run as one launch whose dS
// product walks the long contraction (layer_reverse_wide.hpp).  Where: by a model of both, us, with 15 % in favour of the
// two launches.  One launch: a workgroup takes 9 us and 0.62 per stage of 32 columns for each block of 128 steps, 256
// workgroups at a time.  Two: 1.2 per GFLOP and 5 TB/s of dX and dS for the product, 12 bytes per neuron and step
// at 5.2 TB/s for the scan, or 48 ns a step where there are few chains.  us per step, apart and in one: 700-512-512-20, T = B = 256
// 535 and 467; 700-1024-1024-20, T = 256, B = 512 2488 and 2260; 200-256-256-20, B = 256: T = 50 85.6 84.5, 70 95.8 91.2, 128 120 108,
// 140 (a second block of 12) 142 133, T = 500, B = 64 170 186; 200-512-512-20: T = 128, B = 32 / 64 / 256 85.1 89.2 / 98.5 96.5 / 258 226, T =
// 256, B = 32 / 64 126 137 / 150 149, T = 200, B = 128 222 181; 100-300-1000-20, T = 256, B = 64 188 196, T = 500, B = 128 677 657; 100-2048-2048-10, T =
// 128, B = 32 / 64 / 256 342 309 / 525 477 / 1592 1559, T = 50, B = 256 802 888.  Of 70 networks drawn at
// random where it takes the one launch two are more than 0.6 % slower with it (700-1280-640-20, T = 89, B = 51 165 169, 2.5 %; 1.0 %), the median is 7 %
// faster.
// Adaptive thresholds, below any layer (a scan takes 16 bytes and 62 ns; 12 us a block): 700-256-256-20, T = B = 128 127.2
// 121.9; 700-256-20: T = 128, B = 64 / 128 / 256 61.0 63.1 / 75.7 72.8 / 115 101, T = 200, B = 128 102.4 102.7; 700-100-20, T = 128, B =
// 128 / 256 59.8 62.0 / 74.8 73.3; 200-1000-20, T = 100, B = 32 74.4 72.5, T = B = 128 184 138; 700-512-512-20, T = 64, B = 16 81.9
// 92.8, T = 300, B = 256 883 790.  Of 70 drawn networks that it takes none is more than 0.5 % slower.
// `ld`: the layer's padded neurons; `columns`: those of the layer above.
inline bool reverse_wide_pays(int T, int B, int ld, int columns, bool adaptive) {
  const double M = (double)T * B, N = ld;
  const long long groups = (long long)B * ((ld + 255) / 256);
  const double rounds = groups <= 512 ? (double)((groups + 255) / 256) : groups / 256.;
  const double one = 4. + ((T + 127) / 128) * rounds * ((adaptive ? 12. : 9.) + 0.62 * ((columns + 31) / 32));
  const double product = 3. + 2.4e-9 * M * N * columns + 4. * M * (N + columns) / 5e6;
  const double scan = adaptive ? std::max(0.062 * T + 2., 2. + 16. * M * N / 5.2e6) : std::max(0.048 * T + 1., 2. + 12. * M * N / 5.2e6);
  return 1.15 * one < product + scan + 2.;
}

// A feed-forward layer of more than 128 neurons on rounded weights can run on the kernel for wide layers
// (layer_forward_wide.hpp): workgroups of two samples and 128 neurons.
// Against one launch of workgroups of one sample and 128 neurons (layer_forward.hpp), where those are so many that both
// fill the chip more than once, beyond 64 steps, and the last part is not half empty (us per step, before and so; workgroups
// before: 700-512-512-20: T = 128, B = 64, 256: 111.6 120.4, T = 200, B = 128, 512: 241.4 245.2, T = 100 140.3 138.6, T = 128, B = 255,
// 1020: 266 256, T = B = 256, 1024: 480 442, T = 50 148.6 154.9, T = 70 177.8 169.1; 700-1024-1024-20: B = 64, 512: T = 128 194.9 194.0,
// T = 500 590 595, T = 256, B = 512, 4096: 2267 2169; 700-256-256-20: T = 140, B = 256, 512: 177.1 177.6, T = 300, B = 200, 400: 282 287).
// Against product and scan apart (above 1024 neurons or inputs) by a model of both, us, with 10 % in favour of those: 10.5
// and half a us per 64 inputs for each block of 128 steps, 256 workgroups at a time; 1.25 per GFLOP (0.75 where the currents
// stream past the caches) and 5 TB/s of currents for the product, 9 bytes at 6 TB/s or 43 ns a step for the scan.  700-2048-2048-10:
// T = 128, B = 32 / 64 / 255 362 280 / 566 474 / 1764 1525, T = 500, B = 128 3658 3092, T = 500, B = 16 621 614, T = 1000, B = 8 701 804.  Of 70
// drawn networks that either rule takes one is slower (623-640-640-10, T = 125, B = 254 342 347, 1.5 %).
// Whether a context's options leave it a choice: 64 neurons or two workgroups to a sample ask for the kernel that has them.
inline bool forward_wide_allowed(int layer_forward, int layer_max_neurons, int layer_neurons, int layer_time_split) {
  return layer_forward >= 4 && layer_max_neurons >= 1024 && layer_neurons == 128 && !layer_time_split;
}
// `one_launch`: the layer would run as one launch of that kernel; `top_scan`: as a scan that forms the readout's currents;
// `streams`: its currents stream past the caches.
inline bool forward_wide_pays(int T, int B, int ld, int fan_in, bool one_launch, bool top_scan, bool streams) {
  const long long parts = (ld + 127) / 128;
  if (one_launch) return T > 64 && (ld + 63) / 64 == 2 * parts && B * parts >= 768;
  if (top_scan) return false;
  const double M = (double)T * B, N = ld, rounds = std::max(1., (B + 1) / 2 * parts / 256.);
  const double one = 4. + ((T + 127) / 128) * rounds * (10.5 + 0.5 * ((fan_in + 63) / 64));
  const double product = 3. + (streams ? 1.5e-9 : 2.5e-9) * M * N * fan_in + 4. * M * N / 5e6;
  const double scan = std::max(0.043 * T + 2., 2. + 9. * M * N / 6e6);
  return 1.1 * one < product + scan;
}

}  // namespace snn
