// Reverse pass of a feed-forward LIF layer below a WIDE layer (more than 128 columns) in one launch: the spike gradients
// dS = dX W^T, the surrogate, the reverse scan, dI stored as hi/lo words (rounded weights; see layer_reverse.hpp for
// narrow layers above).  dS never reaches memory.  ADAPT: a layer with adaptive thresholds, below any layer.
//
// As two launches the product writes dS and the scan reads it back, 8 bytes per neuron and step, where the pass cannot do
// without 12 (dX, V, dI).  A workgroup owns one sample and 256 neurons; per block of 128 steps, last block first:
//   1. product: 128 steps x 256 neurons on 2 x 2 wavefronts of 64 x 128, stages of 32 columns, both operands from memory
//      straight into LDS (buffer_load ... lds).  The tile is this wide because the L2 gives a compute unit about 29 bytes a
//      cycle: 32 KiB per 1024 cycles of MFMA (both passes), 48 with 128 x 128.  The words of dX have three buffers (they
//      come from memory: two stages to land), the weights two (they stay in the L2): 80 KiB, so that two workgroups share
//      a compute unit and one multiplies while the other scans.
//   2. scan, 64 steps at a time: the wavefronts that hold these steps put them into LDS (the stages are free), and every
//      thread walks its own neuron: V straight from memory 32 steps ahead (16 with its adaptation), g' = beta g + s (dS -
//      theta g), dI stored.
// The words are split into their bfloat16 planes after the fragment read, lo first; both meet the same weights.
//
// 700-512-512-20, T = B = 256: 87 us (product) + 65 (scan) -> 90, 80 of it what dX, V and dI take at 5 TB/s; 700-1024-1024-20, T = 256,
// B = 512: 537 + 267 -> 675, where 128 steps of a sample lie in 128 different pages of 2 MiB (with the rows of a sample side by
// side the launch takes 557).  Potentials 32 steps ahead of the scan instead of 16: 96 -> 89 and 698 -> 680; 64 steps spill.  No
// difference: the walk through the contraction starting elsewhere in each sample, priorities or a delay between the two
// workgroups of a compute unit.
#pragma once
#include "surrogate.hpp"
#include "gemm_stream.hpp"
#include "layer_reverse.hpp"

namespace snn {

struct ReverseWide {
  static constexpr int BM = 128, BN = 256;
  static constexpr int PB = BM * 128, QB = BN * 64;               // bytes of a stage: words of dX, weights
  static constexpr int QOFF = 3 * PB, LDS_BYTES = 3 * PB + 2 * QB;
  static constexpr int PITCH = BN + 4;                            // floats between rows of dS in LDS
  static_assert(LDS_BYTES == 81920 && 64 * PITCH * 4 <= LDS_BYTES, "two workgroups per compute unit");
};

template <int SURR, int POL, bool ADAPT>
__global__ __launch_bounds__(256, 2) void lif_layer_reverse_wide_kernel(const LayerReverseArgs a) {
  typedef ReverseWide G;
  constexpr int BM = G::BM, BN = G::BN, PB = G::PB, QB = G::QB;
  __shared__ __attribute__((aligned(16))) char lds[G::LDS_BYTES];

  // Workgroup ids are dealt round-robin to the 8 XCDs: the parts of a sample take ids 8 apart.
  const int parts = (a.ld + BN - 1) / BN;
  const int part = (blockIdx.x >> 3) % parts;
  const int b = (blockIdx.x >> 3) / parts * 8 + (blockIdx.x & 7);
  if (b >= a.B) return;
  const int n0 = part * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, h = lane >> 5;
  const u32x4 rp = raw_rsrc(a.dX, (unsigned)a.T * a.B * a.ldc * 4u), rq = raw_rsrc(a.Wq, a.wq_bytes);
  const unsigned lds0 = (unsigned)(uintptr_t)(lds_ptr_t)lds;
  const int nk = (a.ldc + 31) >> 5;                    // stages

  // Global side of the loads.  Words: instruction q of a wavefront fills rows 8 (wave + 4 q) .. + 7 of the stage, 128 bytes
  // each, lane -> row lane / 8, slot lane % 8 holding unit slot ^ (row / 2) % 8.  Weights: rows (neurons) 16 (wave + 4 q) .. +
  // 15, 64 bytes each, lane -> row lane / 4, slot lane % 4 holding chunk slot ^ (row / 4) % 4.  (16 consecutive rows of a
  // fragment read then lie on 16 different groups of four banks.)
  int pv[4], qv[4];
  bool in_last[4];                                     // the unit exists in the last stage
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = 8 * (wave + 4 * q) + (lane >> 3), u = (lane & 7) ^ ((row >> 1) & 7);
    in_last[q] = (nk - 1) * 32 + u * 4 < a.ldc;
    const int n = 16 * (wave + 4 * q) + (lane >> 2), ch = (lane & 3) ^ ((n >> 2) & 3);
    qv[q] = ((n0 + n) * a.ldq + ch * 8) * 2;
  }
  // Fragment reads: steps 64 wm + 32 i + lane % 32, the eight words 16 st + 8 h ..; neurons 128 wn + 32 j + lane % 32, the same columns.
  int fp[2][2], fq[2];
  {
    const int ra = 64 * wm + (lane & 31), rb = 128 * wn + (lane & 31);
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
      for (int e = 0; e < 2; ++e) fp[st][e] = ra * 128 + (((4 * st + 2 * h + e) ^ ((ra >> 1) & 7)) << 4);
      fq[st] = G::QOFF + rb * 64 + (((2 * st + h) ^ ((rb >> 2) & 3)) << 4);
    }
  }

  struct Frag {
    u32x4 q[4], hi[2], lo[2];
  };
  f32x16 acc[4][2];                                    // neurons 32 j, steps 32 i

  auto issue_p = [&](int kt, int buf, int q) {
    u32x4 r = rp;
    if (kt >= nk) r.z = 0;                             // beyond the contraction: same instruction count, nothing fetched
    load_to_lds_b128(r, __builtin_amdgcn_readfirstlane(lds0 + buf * PB + 1024 * wave) + 4096 * q,
                     kt == nk - 1 && !in_last[q] ? OOB : pv[q], kt * 128);
  };
  auto issue_q = [&](int kt, int buf, int q) {
    u32x4 r = rq;
    if (kt >= nk) r.z = 0;
    load_to_lds_b128(r, __builtin_amdgcn_readfirstlane(lds0 + G::QOFF + buf * QB + 1024 * wave) + 4096 * q, qv[q], kt * 64);
  };
  // The 16 MFMAs of step x, one per slot, with what the next step (ST of the stage in buffers U) needs behind them: fragment
  // reads first, `fetch` in the middle, the split of the words last.
  auto half = [&](auto U, auto ST, const Frag &x, Frag &next, auto fetch) {
    constexpr int po = decltype(U)::value % 3 * PB, qo = decltype(U)::value % 2 * QB, st = decltype(ST)::value;
    u32x4 raw[2][2];
    static_for<16>([&](auto N) {
      constexpr int n = decltype(N)::value, i = n & 1, j = (n & 7) >> 1;
      acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x.q[j]),
                                                          __builtin_bit_cast(bf16x8, n < 8 ? x.lo[i] : x.hi[i]), acc[j][i], 0, 0, 0);
      if constexpr (n < 4) {
        raw[n >> 1][n & 1] = *(const u32x4 *)(lds + fp[st][n & 1] + (po + (n >> 1) * 4096));
        next.q[n] = *(const u32x4 *)(lds + fq[st] + (qo + n * 2048));
      }
      fetch(N);
      if constexpr (n >= 12) {
        constexpr int ti = (n - 12) >> 1, e = n & 1;
        const u32x4 w = raw[ti][e];
        next.hi[ti][2 * e] = __builtin_amdgcn_perm(w.y, w.x, 0x05040100u);
        next.hi[ti][2 * e + 1] = __builtin_amdgcn_perm(w.w, w.z, 0x05040100u);
        next.lo[ti][2 * e] = __builtin_amdgcn_perm(w.y, w.x, 0x07060302u);
        next.lo[ti][2 * e + 1] = __builtin_amdgcn_perm(w.w, w.z, 0x07060302u);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // A stage: its first half multiplies the step left over from the stage before.  At its barrier every wavefront has seen
  // its own loads of the stage land (the words of the next stage may still be in flight) and has left stage kt - 1, whose
  // buffers take the weights of stage kt + 1 and the words of stage kt + 2.
  auto stage = [&](auto U, int kt_any, Frag &pend) {
    constexpr int u = decltype(U)::value;
    const int kt = __builtin_amdgcn_readfirstlane(kt_any);
    asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    Frag now;
    half(U, std::integral_constant<int, 0>(), pend, now, [&](auto N) {
      constexpr int n = decltype(N)::value;
      if constexpr (n >= 4 && n < 8) issue_q(kt + 1, (u + 1) % 2, n - 4);
      if constexpr (n >= 8 && n < 12) issue_p(kt + 2, (u + 2) % 3, n - 8);
    });
    half(U, std::integral_constant<int, 1>(), now, pend, [](auto) {});
  };

  // State of neuron n0 + tid.
  const bool mine = n0 + tid < a.ld;
  const float beta = mine ? a.beta_v[n0 + tid] : 0.f, theta = a.theta, slope = a.slope;
  float g = 0.f, ga = 0.f, db = 0.f;                   // (ga: gradient of the adaptation, see lif_reverse_kernel)
  const unsigned vbytes = (unsigned)a.T * a.B * a.ld * 4u;
  const rsrc_t rV = make_rsrc(a.V, vbytes), rdI = make_rsrc(a.dI, vbytes);
  const rsrc_t rA = make_rsrc(a.A, ADAPT ? vbytes : 0u);
  const int row4 = a.B * a.ld * 4, vo = mine ? (b * a.ld + n0 + tid) * 4 : OOB;
  const float *const cell = (const float *)lds + tid;

  for (int t0 = (a.T - 1) / BM * BM; t0 >= 0; t0 -= BM) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = 8 * (wave + 4 * q) + (lane >> 3), u = (lane & 7) ^ ((row >> 1) & 7);
      pv[q] = t0 + row < a.T ? ((t0 + row) * a.B + b) * a.ldc * 4 + u * 16 : OOB;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
    Frag pend;                                         // zeros in front of the first stage
#pragma unroll
    for (int j = 0; j < 4; ++j) pend.q[j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 2; ++i) pend.hi[i] = pend.lo[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < 4; ++q) issue_q(0, 0, q);
#pragma unroll
    for (int q = 0; q < 4; ++q) issue_p(0, 0, q);
#pragma unroll
    for (int q = 0; q < 4; ++q) issue_p(1, 1, q);
    int kt = 0;
    for (; kt + 6 <= nk; kt += 6) {
      static_for<6>([&](auto U) { stage(U, kt + decltype(U)::value, pend); });
    }
    static_for<5>([&](auto U) {
      if (kt + decltype(U)::value < nk) stage(U, kt + decltype(U)::value, pend);
    });
    // The potentials of the first 32 steps (16, with their adaptation) are asked for under the last MFMAs, and those as many
    // steps on as steps are taken.
    constexpr int U = ADAPT ? 8 : 16;
    struct Rows { float v[U], a[ADAPT ? U : 1]; } rows[2];
    auto fetch = [&](Rows &x, int t) {                 // steps t .. t + U - 1 (past T: zeros)
#pragma unroll
      for (int s = 0; s < U; ++s) {
        const int off = t >= 0 && t + s < a.T ? vo : OOB, so = min(max(t + s, 0), a.T - 1) * row4;
        x.v[s] = __uint_as_float(ld_b32<POL>(rV, off, so));
        if (ADAPT) x.a[ADAPT ? s : 0] = __uint_as_float(ld_b32<POL>(rA, off, so));
      }
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the stage loads beyond the range have written their zeros)
#pragma unroll
    for (int k = 1; k >= 0; --k) fetch(rows[k], t0 + BM - 2 * U + U * k);
#pragma unroll
    for (int n = 0; n < 16; ++n)
      acc[(n & 7) >> 1][n & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          __builtin_bit_cast(bf16x8, pend.q[(n & 7) >> 1]), __builtin_bit_cast(bf16x8, n < 8 ? pend.lo[n & 1] : pend.hi[n & 1]),
          acc[(n & 7) >> 1][n & 1], 0, 0, 0);
    lds_barrier();                                     // every wavefront is past its fragment reads

    static_for<2>([&](auto HF) {
      constexpr int hf = 1 - decltype(HF)::value;
      // dS^T: the lane holds step 32 i + lane % 32 of its half, register r neuron 8 (r / 4) + 4 h + r % 4 of the tile.
      if (wm == hf) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const f32x4 x = {acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
              *(f32x4 *)(lds + ((32 * i + (lane & 31)) * G::PITCH + 128 * wn + 32 * j + 8 * q + 4 * h) * 4) = x;
            }
      }
      lds_barrier();
      auto steps = [&](const Rows &x, int s0) {        // steps s0 + U - 1 .. s0 of the half
        const int t = t0 + 64 * hf + s0;
        if (t >= a.T) return;
        float ds[U];
#pragma unroll
        for (int s = 0; s < U; ++s) ds[s] = cell[(s0 + s) * G::PITCH];
#pragma unroll
        for (int s = U - 1; s >= 0; --s) {
          __builtin_amdgcn_raw_buffer_store_b32(pack_hl(g), rdI, t + s < a.T ? vo : OOB, min(t + s, a.T - 1) * row4, POL);
          db = __builtin_fmaf(g, x.v[s], db);
          if constexpr (ADAPT) {
            const float thr = theta + x.a[s], y = x.v[s] - thr;
            const float sq = surr_rcp<SURR>(slope, y) * (ds[s] - thr * g + a.kappa * ga);
            ga = a.gamma * ga - (y > 0.f ? g : 0.f) - sq;
            g = beta * g + sq;
          } else {
            g = beta * g + surr_rcp<SURR>(slope, x.v[s] - theta) * (ds[s] - theta * g);
          }
        }
      };
      const int t = t0 + 64 * hf;
#pragma unroll
      for (int k = 64 / U - 1; k >= 0; --k) {
        steps(rows[k & 1], U * k);
        if (hf || k >= 2) fetch(rows[k & 1], t + U * (k - 2));
      }
      lds_barrier();                                   // the rows are read before the next ones, or the next block's stages, land
    });
  }
  if (a.db_part && mine) a.db_part[b * a.ld + n0 + tid] = db;
}

hipError_t layer_reverse_wide(hipStream_t st, const LayerReverseArgs &a, int surrogate);

}  // namespace snn
