// How the contraction of the weight-gradient products is split over workgroups (host arithmetic only).
#pragma once
#include <vector>

namespace snn {

inline long long round_up(long long x, long long m) { return (x + m - 1) / m * m; }

constexpr long long SHORT_ROWS = 8192, SHORT_TILES = 32;  // a short contraction on few tiles: see below

// Contraction splits of the weight-gradient products, which share one launch with `tiles`
// output tiles in total over M rows each.  `weights`: elements of all gradient matrices (a
// split writes that many partial sums); `row_bytes`: operand bytes the products read per row
// of the contraction.  Measured facts behind the rule:
//   * the splits of a tile are dealt round-robin to the 8 XCDs (see gemm_body), so a count
//     that is not a multiple of 8 leaves some XCDs with a split more than others and the
//     launch lasts as long as the fullest (700-512-512-20, T*B = 65536: 21 splits 253 us,
//     24 splits 225 us, 32 splits 180 us);
//   * 512 workgroups run at once (two per compute unit).  Slightly more than that (24 splits
//     x 22 tiles = 528) is the worst case: the stragglers run a whole workgroup's work alone.
//     Either everything fits at once, or there are at least 1.3 rounds of shorter workgroups;
//   * every split writes and the reduction re-reads all partial sums: with large matrices
//     (2048 wide: 56 MB per split) more splits cost more than they gain (64 splits: 10.2 ms
//     against 3.3 ms with 8), and 16 splits never beat 8 at 1024 wide.
//   * the kernel on transposing LDS reads (wgrad_tr.hpp) multiplies as fast with one workgroup per
//     compute unit as with two (its MFMAs are fed by the wavefront's own instruction stream), so for
//     it (`one_per_cu`) half as many splits cover the chip at the same product time and half the
//     partial sums (700-128-128-20, T*B = 32768: 32 splits 19.1 us + 4.4 us for the update against
//     64 splits 20.7 + 6.5);
//   * 2..7 splits would leave whole XCDs without work (a split lives on one XCD): 8 then;
//   * a short contraction on few tiles leaves most of the chip empty, and its time is that of one split
//     plus that of the partial sums: 8 to 13 ns a row of a split and 1.25 ps a partial sum (written and read).
//     Splits are doubled as long as that shortens the sum of both, a workgroup per compute
//     unit at most; beyond 64 the launch itself is the longer part.  us, 64 / 128 / 256 / 512 rows a split, * the
//     rule's: steps of 700-128-128-20, T*B = 1536: 49.5 48.5 48.4 50.1 (192 rows: 47.4*), 4096: 54.3 53.4 51.8* 52.3,
//     8192: 66.2 57.8 54.7* 55.5; of 100-64-10 in fp32, 512: 35.4* 37.0 38.7 42.2, 2048: 37.2* 38.5 40.2 45.0, 8192:
//     44.3 43.8* 45.0 49.4; of 700-256-256-20, 1024: 65.5 61.6* 62.2 64.1, 4096: 83.8 74.6 69.9 69.0*.  With M / 64 splits
//     below 2048 rows and M / 256 from there on the count fell from 16 to 8 at 2048 rows (100-64-10: 33.8 us), and
//     large matrices paid for partial sums (700-128-128-20, 1536: 49.5 us).
inline int choose_splits(long long M, int tiles, long long weights, long long row_bytes, long long *per_split, bool one_per_cu) {
  const long long target = 512;                          // workgroups resident at once
  if (tiles < 1) tiles = 1;
  if (one_per_cu && M <= SHORT_ROWS && tiles <= SHORT_TILES) {
    long long want = 1;
    while (want < 64 && 2 * want * tiles <= target / 2 && 128 * want <= M && 2 * want * want * weights < 8000 * M) want *= 2;
    *per_split = round_up((M + want - 1) / want, 64);
    return (int)((M + *per_split - 1) / *per_split);
  }
  const long long max_by_len = M / 256;                  // at least four 64-row tiles per workgroup
  long long want = target / tiles;
  if (want > max_by_len) want = max_by_len;
  if (want < 1) want = 1;
  if (want > 1 && want < 8 && max_by_len >= 8) want = 8;
  if (want >= 8) {
    want = want / 8 * 8;                                 // all at once, balanced over the XCDs
    // when that leaves more than 15 % of the chip idle: more, shorter workgroups, as long as
    // each keeps 16 tiles of the contraction and the partial sums stay below a quarter of the
    // operand bytes
    const long long more = ((target * 13 / 10 + tiles - 1) / tiles + 7) / 8 * 8;
    if (want * tiles * 100 < target * 85 && M / more >= 1024 && more * weights * 4 * 4 <= M * row_bytes) want = more;
    const long long half = (target / 2 / tiles) / 8 * 8; // one workgroup per compute unit
    if (one_per_cu && half >= 8 && half < want && half * tiles * 100 >= target / 2 * 85) want = half;
  }
  long long per = round_up((M + want - 1) / want, 64);
  *per_split = per;
  return (int)((M + per - 1) / per);
}

// A product of at most 32 columns: three of the four wavefronts of a 128-column tile multiply nothing, which shows
// once it takes longer than a launch.  Alone it takes tiles of 128 x 32 of the general kernel then: fp32, 512 x 16:
// T*B = 16384 13.4 us with the wide tile and 14.4 with the narrow one, 32768 18.4 and 16.8, 262144 84.3 and 71.1; 100 x 16,
// one tile: 29.3 and 29.3 at 262144; the step of 700-32-10 on rounded weights (two pieces a word instead of
// three) at 262144 254 us and 239, at 131072 (700-32-20) 126.7 and 124.3.  Beside wider products it stays in their launch, but
// with splits as if alone, for two workgroups a compute unit: steps of 700-512-20 in fp32 at 131072 938 us with
// the launch's splits, 904 with its own, 917 in a launch of its own; 700-2048-20 on rounded weights at 65536 1185,
// 1153 and 1180.
inline bool long_and_narrow(long long M, int rows, int cols, bool fp32) {
  const long long t = (rows + 127) / 128;
  return cols <= 32 && t >= 2 && t * M >= (fp32 ? 1 << 17 : 3 << 18);
}

// A product of the merged weight-gradient launch: dW or dR, rows x cols.
struct WgradProduct { int rows, cols; };

// The merged launch of a network: `sizes` of its L + 1 layers, `recurrent` flags of the first L.
struct WgradLaunch {
  std::vector<WgradProduct> products;                    // those whose splits are the launch's
  std::vector<bool> own;                                 // per layer: dW is long and narrow beside wider products, splits of its own
  bool narrow = false;                                   // every dW is narrow and one is long
  long long weights = 0, row_bytes = 0;                  // what `products` write per split / read per row
};
inline WgradLaunch wgrad_launch(long long M, int L, const int *sizes, const std::vector<bool> &recurrent, bool fp32) {
  WgradLaunch w;
  bool any_long = false, all_narrow = true;
  for (int l = 0; l < L; ++l) {
    any_long = any_long || long_and_narrow(M, sizes[l], sizes[l + 1], fp32);
    all_narrow = all_narrow && sizes[l + 1] <= 32;
  }
  w.narrow = any_long && all_narrow;
  for (int l = 0; l < L; ++l) {
    const int K = sizes[l], N = sizes[l + 1];
    w.own.push_back(!all_narrow && long_and_narrow(M, K, N, fp32));
    if (!w.own[l]) {
      w.products.push_back({K, N});
      w.weights += (long long)K * N;
      w.row_bytes += K + 4ll * N;                        // spike bytes below, 4-byte current gradients
    }
    if (recurrent[l]) {
      w.products.push_back({N, N});
      w.weights += (long long)N * N;
      w.row_bytes += N + (w.own[l] ? 4ll * N : 0);
    }
  }
  return w;
}

// Tiles of 256 x 128 on the kernel of transposing LDS reads (rounded weights), one workgroup per compute unit: that kernel
// has one tile for products of any width.
inline int wgrad_tall_tiles(const WgradProduct &p) { return ((p.rows + 255) / 256) * ((p.cols + 127) / 128); }
inline int wgrad_flat_tiles(const WgradProduct &p) { return ((p.rows + 127) / 128) * ((p.cols + 127) / 128); }

// Splits of tall tiles: any count, for the workgroups of an XCD (32 compute units; each product's workgroups are dealt
// evenly over the XCDs) to take the fewest rounds for their length, 18 ns a row and 5 us a round, with the partial sums.  A long and narrow product beside them has splits of its own (see
// long_and_narrow) that come to about one workgroup for every compute unit, whatever its height: a round in front of
// the others', the same for each count.  The launch alone in one sweep, us, * the choice: 700-512-512-20, T*B = 65536: 8 splits 165, 9 155, 10 146,
// 11 140*, 12 224, 16 178, 23 147; 700-1024-1024-20, 131072: 4 730, 8 722, 9 701*; 700-256-256-20, 65536: 16 91, 24 72, 26 68, 28
// 67*, 32 97; 300-1024-20, 65536: 8 156, 10 133, 12 124*, 14 188.
inline long long tall_slots(const WgradLaunch &w, int splits) {
  long long slots = 0;                                   // workgroups of an XCD
  for (const WgradProduct &p : w.products) slots += ((long long)wgrad_tall_tiles(p) * splits + 7) / 8;
  return slots;
}
inline int choose_splits_tall(long long M, const WgradLaunch &w, long long *per_split) {
  int best = 1;
  double best_us = 0.;
  for (int want = 1; want <= 64 && (want == 1 || 256ll * want <= M); ++want) {
    const long long per = round_up((M + want - 1) / want, 64);
    const int splits = (int)((M + per - 1) / per);
    const double us = (tall_slots(w, splits) + 31) / 32 * (per * 18e-3 + 5.) + (splits > 1 ? splits * w.weights * 1.25e-6 : 0.);
    if (want == 1 || us < best_us) { best = want; best_us = us; }
  }
  *per_split = round_up((M + best - 1) / best, 64);
  return (int)((M + *per_split - 1) / *per_split);
}

// Whether tall tiles are the faster form: by a model of both launches, us, with 7 in favour of 128 x 128 tiles.  Either
// launch takes a time for its rows and one for the rounds of its workgroups and writes its partial sums, which the update
// reads (dW from one split goes straight to its place); 128 x 128 tiles read more of the operands from memory once those do
// not stay in the caches (`row_bytes`: bytes of all operands per row of the contraction; 120 MB).  The model is within 6 % (tall)
// and 9 % of 203 launches at 512 to 250000 rows.  Of 165 steps measured where it takes tall tiles four are 1 to 2.1 % slower with
// them and 136 more than 2 % faster (1.31 times at most); of 102 where it does not, three would be more than 4 % faster.
// us per step, 128 x 128 and 256 x 128, * the choice: 700-512-512-20, T*B = 10000 126.0* 125.6, 16384 155 152*, 32768 272 260*, 65536
// 471 456*; 700-256-256-20, 32768 143.1* 143.4, 51200 229 218*, 65536 277 256*; 300-1024-20 (512 rows for 300), 32768 175* 187, 65536
// 380 366*; 700-512-20, 40960 162* 167, 57344 249 222*; 700-1024-1024-20, 8192 196 191*, 131072 2415 2242*; 700-1472-1472-10, 1536 249
// 195*; 700-2048-2048-20, 4096 368 348*; 398-1911-1911-1911-10, 3503 559* 590; 700-1542-1542-20, 5300 406* 416; 700-1664-1664-10,
// 11235 575 543*.
inline bool wgrad_tall_pays(long long M, const WgradLaunch &w) {
  long long tiles = 0, tiles_tall = 0, per, per_tall, slots = 0;
  for (const WgradProduct &p : w.products) {
    tiles += wgrad_flat_tiles(p);
    tiles_tall += wgrad_tall_tiles(p);
  }
  const int splits = choose_splits(M, (int)tiles, w.weights, w.row_bytes, &per, true), splits_tall = choose_splits_tall(M, w, &per_tall);
  for (const WgradProduct &p : w.products)               // workgroups of the fullest XCD, splits dealt round-robin
    slots += splits == 1 ? (wgrad_flat_tiles(p) + 7) / 8 : (long long)wgrad_flat_tiles(p) * ((splits + 7) / 8);
  const long long rounds = (slots + 31) / 32, rounds_tall = (tall_slots(w, splits_tall) + 31) / 32;
  const double from_memory = M * w.row_bytes * 1e-6 - 120.;
  const double flat = 22e-6 * M * tiles + 6.5e-3 * rounds * per + 0.6e-6 * splits * w.weights + (from_memory > 0. ? 0.1 * from_memory : 0.);
  const double tall = 3. + 27e-6 * M * tiles_tall + 13.3e-3 * rounds_tall * per_tall + 0.72e-6 * splits_tall * w.weights;
  const double update = 1e-6 * w.weights * (splits_tall - splits + 3 * ((splits_tall > 1) - (splits > 1)));
  return flat - tall - update >= 7.;
}

// Tiles of the general kernel.
inline int wgrad_tiles(int rows, int cols, bool tall) {
  int bn = cols <= 32 ? 32 : (cols <= 64 ? 64 : 128);
  const int bm = tall && cols > 64 ? 256 : 128;
  return ((rows + bm - 1) / bm) * ((cols + bn - 1) / bn);
}

}  // namespace snn
