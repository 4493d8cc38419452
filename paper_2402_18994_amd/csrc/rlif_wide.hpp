// Time loops of recurrent layers too wide for one workgroup, on rounded weights (up to 2048 neurons):
// V_{t+1} = beta V_t + I_t + S_t R - theta S_t, and the reverse recursion, all steps in a launch (one for every
// 8 * (32 / members of a group) tiles of the batch).
//
// A tile of 16 samples belongs to a group of workgroups on ONE XCD: member m owns neurons 64 m .. 64 m + 63,
// keeps their rows of R in registers for all steps (eight wavefronts, each an eighth of the
// contraction: 128 registers at 2048 neurons) and the state of its 64 x 16 neurons as two values a
// thread.  What a step needs from the other members goes through memory with device-scope accesses:
//   * forward: spikes as bits, 64-bit words {32 neurons of a sample, step} that are their own flags: a
//     wavefront polls the words of its share of the contraction until each carries the step;
//   * reverse: the hi/lo words of g, 64 KB to 128 KB per tile, behind one flag per member that is raised
//     when the member's words are acknowledged.
// Two buffers by parity of the step: a member overwrites step s only after it has seen step s + 1 of
// every member, which they published after they had read step s.
//
// Why one XCD: a device-scope load that finds its line in the XCD's own L2 is a short round trip.  32
// members exchanging a word each take 0.7-1.1 us per step within an XCD, 3.1 us when the members are
// spread over the chip (32 neurons x 32 samples per workgroup, the form before); 128 KB of g per
// member adds 2 us, which is what the L2 delivers to a compute unit (29 bytes a clock).  Workgroup i is
// dealt to XCD i % 8; nothing but speed depends on that, every access is at device scope.
// 700-2048(rec)-2048-2048-20, T = 512, B = 128: forward loop 2.83 -> 1.30 ms
// (2.5 us a step: 0.9 until the words are in, 0.3 products, 0.8 sum over the wavefronts and its wait, 0.4
// update and publication), reverse loop 6.08 -> 2.46 ms (4.8 us: 1.3 until the flags are up, 1.8 loads of
// g and products, 0.8 sum, 0.8 publication and its acknowledgement); a launch per step was the reverse loop.
//
// Every workgroup that waits must be resident with those it waits for: these launches are made only
// if the grid fits the compute units at a workgroup each and is ordered behind the other grids of this kind
// (one_grid.hpp; not on a stream that is being captured).  Otherwise (or with SNN_OPT_RLIF_PERSIST = 0) kernels of
// one step are launched T times, which exchange through S and dI and wait for nobody: the same sums in the
// same order, the same bits.  (100-2048(rec)-20, T = 64, B = 128: 576 us forward and 821 reverse, 161 and
// 279 in one launch; 512 neurons: 238 and 267, 99 and 145.  The kernels of the one launch cut to a
// step, exchange and waits included, took 867 and 1348, 323 and 488.)
// A wait polls at most 2^18 times (SNN_OPT_WAIT_LIMIT_LOG2); on a time-out the workgroup sets bit 1 of the
// error word and a flag that ends all waiting everywhere, so the grid drains and the host reports it.
#pragma once
#include "surrogate.hpp"

namespace snn {

struct RlifWide {
  static constexpr int NB = 64, SB = 16;                  // neurons and samples of a workgroup
  static constexpr int MAXN = 2048;                       // widest layer
  static constexpr int SLOTS = 32;                        // workgroups per XCD
  static constexpr int GROUPS = 8 * (SLOTS / 5);          // most groups (layers of 257 neurons have five members)
  // exchange space: abort flag, member flags [group][32] (reverse), words [parity][group][member][sample][2]
  // (forward), g [parity][group][member][half of the neurons][16-neuron piece][4-neuron group][sample][4] (reverse)
  static constexpr size_t FLAGS = 256, FLAG_BYTES = GROUPS * SLOTS * 4;
  static constexpr size_t WORDS = FLAGS + FLAG_BYTES, WORD_BYTES = 2ull * 256 * SB * 2 * 8;
  static constexpr size_t G = WORDS + WORD_BYTES, G_BYTES = 2ull * 256 * SB * NB * 4;
  static constexpr size_t BYTES = G + G_BYTES;
  static constexpr int RP = NB + 4;                       // floats between the samples of a partial sum in LDS
};

struct RlifWideArgs {
  const float *X;                                         // I (forward), dS (reverse)
  float *V;                                               // written (forward), read (reverse)
  uint8_t *S;
  uint32_t *dI;
  float *gs;                                              // [B][ld] g between launches of a step each
  const uint16_t *R;                                      // R^T [to][from] (forward), R [from][to] (reverse)
  int ldr, T, B, ld, P, groups;                           // P: members of a group
  const float *beta_v;
  float theta, slope;
  int surrogate;
  float *db_part;
  char *space;
  int *err;
  int max_polls;
  uint32_t tag_bias;                                      // 0, or (tests) what makes every wait expect a step nobody publishes
  int tile0;                                              // first tile of this launch (group g takes tile0 + g)
  uint32_t tag0;                                          // what step t publishes under is tag0 + t
  int step;                                               // the step of a launch of one
};

static bool rlif_wide_layer(int ld) { return ld > 256 && ld <= RlifWide::MAXN; }
hipError_t rlif_wide_forward(hipStream_t st, RlifWideArgs a, int cus, bool persist);
hipError_t rlif_wide_reverse(hipStream_t st, RlifWideArgs a, int cus, bool persist);

}  // namespace snn
