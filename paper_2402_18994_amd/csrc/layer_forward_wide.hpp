// Forward pass of a wide feed-forward LIF layer in one launch (rounded weights): currents I = S_below W, the scan over time,
// V and S stored; I never goes to memory.  The form for layers that are cut in many parts; layer_forward.hpp has the narrow
// ones, with what they take along (readout, a second layer, packed rasters).
//
// A workgroup owns two samples and 128 neurons; per block of 128 steps:
//   1. product: 256 rows (a sample's 128 steps, then the other's) x 128 neurons on 2 x 2 wavefronts of one sample x 64
//      neurons, stages of 64 inputs, both operands from memory straight into LDS.  What bounds 128 rows x 128 neurons is the
//      ingest of the weights, 24 KiB per 512 cycles of MFMA where the L2 gives a compute unit about 29 bytes a cycle; two
//      samples share them: 32 KiB per 1024.  Three buffers for the spike rows (they come from memory), two for the weights
//      (from the L2): 80 KiB, two workgroups to a compute unit, one multiplies while the other scans.
//   2. scan: every wavefront puts 64 steps of its own sample and neurons into LDS (the stages are free) and takes them back
//      a neuron per lane: nothing is exchanged between wavefronts, no barrier stands in the scan.  V leaves a row of 64 neurons
//      at a time; the spikes of four steps are four compare masks, and lane 16 g + i stores neurons 4 i .. + 3 of step g.
// The spike decision is the compare-free one of layer_forward.hpp.
//
// 700-512-512-20, T = B = 256: 67 + 66 -> 66 + 44 us for the two layers; 700-1024-1024-20, T = 256, B = 512: 294 + 338 -> 250 +
// 279, the second one's 805 MB in 161 at 5 TB/s; the 2048 x 2048 layers of T = 512, B = 128: 526 (product) + 210 (scan) -> 445.  The
// product alone takes 157 us of the 279 (1.75 PFLOP/s): what is left is that all compute units write at the same time.
#pragma once
#include "gemm_stream.hpp"
#include "layer_forward.hpp"

namespace snn {

struct ForwardWide {
  static constexpr int BM = 128, BN = 128, KS = 64;               // steps (of each of two samples), neurons, inputs of a stage
  static constexpr int PB = 2 * BM * KS, QB = BN * 2 * KS;        // bytes of a stage: spikes, weights
  static constexpr int QOFF = 3 * PB, LDS_BYTES = 3 * PB + 2 * QB;
  static constexpr int PITCH = 64 + 4;                            // floats between steps of a wavefront's currents
  static_assert(LDS_BYTES == 81920 && 4 * 64 * PITCH * 4 <= LDS_BYTES, "two workgroups per compute unit");
};

template <int POL>
__global__ __launch_bounds__(256, 2) void lif_layer_forward_wide_kernel(const LayerForwardArgs a) {
  typedef ForwardWide G;
  constexpr int BM = G::BM, PB = G::PB, QB = G::QB, KS = G::KS;
  __shared__ __attribute__((aligned(16))) char lds[G::LDS_BYTES];
  const LayerForwardOp &op = a.op[0];

  // Workgroup ids are dealt round-robin to the 8 XCDs: the parts of a pair of samples take ids 8 apart.
  const int part = (blockIdx.x >> 3) % a.parts;
  const int b0 = ((blockIdx.x >> 3) / a.parts * 8 + (blockIdx.x & 7)) * 2;
  if (b0 >= a.B) return;
  const int n0 = part * G::BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, h = lane >> 5;
  const u32x4 rp = raw_rsrc(op.P, op.p_bytes), rq = raw_rsrc(op.Q, op.q_bytes);
  const unsigned lds0 = (unsigned)(uintptr_t)(lds_ptr_t)lds;
  const int nk = (op.kc + KS - 1) / KS;                // stages

  // Global side of the loads.  Spikes: instruction q of a wavefront fills rows 16 (wave + 4 q) .. + 15 of the stage, 64 bytes
  // each, lane -> row lane / 4, slot lane % 4 holding unit slot ^ (row / 4) % 4.  Weights: rows 8 (wave + 4 q) .. + 7, 128
  // bytes each, lane -> row lane / 8, slot lane % 8 holding chunk slot ^ (row / 2) % 8.
  int pv[4], qv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int n = 8 * (wave + 4 * q) + (lane >> 3), ch = (lane & 7) ^ ((n >> 1) & 7);
    qv[q] = ((n0 + n) * op.ldq + ch * 8) * 2;
  }
  // Fragment reads: row 128 wm + 32 i + lane % 32, units 2 h and 2 h + 1 (two steps of eight inputs each); neuron 64 wn +
  // 32 j + lane % 32, chunk 4 h + step.
  int fp[2], fq[4];
  {
    const int ra = 128 * wm + (lane & 31), rb = 64 * wn + (lane & 31);
#pragma unroll
    for (int e = 0; e < 2; ++e) fp[e] = ra * KS + (((2 * h + e) ^ ((ra >> 2) & 3)) << 4);
#pragma unroll
    for (int st = 0; st < 4; ++st) fq[st] = G::QOFF + rb * 2 * KS + (((4 * h + st) ^ ((rb >> 1) & 7)) << 4);
  }

  struct Frag {
    u32x4 q[2];
    bf16x8 p[4];
  };
  f32x16 acc[2][4];                                    // neurons 32 j, steps 32 i
  u32x4 raw[4];                                        // spikes of two steps, per row tile

  auto issue_p = [&](int kt, int buf, int q) {
    u32x4 r = rp;
    if (kt >= nk) r.z = 0;                             // beyond the contraction: same instruction count, nothing fetched
    load_to_lds_b128(r, __builtin_amdgcn_readfirstlane(lds0 + buf * PB + 1024 * wave) + 4096 * q, pv[q], kt * KS);
  };
  auto issue_q = [&](int kt, int buf, int q) {
    u32x4 r = rq;
    if (kt >= nk) r.z = 0;
    load_to_lds_b128(r, __builtin_amdgcn_readfirstlane(lds0 + G::QOFF + buf * QB + 1024 * wave) + 4096 * q, qv[q], kt * 2 * KS);
  };
  // Spike bytes to bfloat16 of value 2 (see SpikeTile): the products come out doubled and are halved on their way to LDS.
  auto convert = [&](uint32_t x0, uint32_t x1) {
    const uint32_t t0 = x0 << 6, t1 = x1 << 6;
    u32x4 d;
    d.x = __builtin_amdgcn_perm(0u, t0, 0x010C000Cu);
    d.y = __builtin_amdgcn_perm(0u, t0, 0x030C020Cu);
    d.z = __builtin_amdgcn_perm(0u, t1, 0x010C000Cu);
    d.w = __builtin_amdgcn_perm(0u, t1, 0x030C020Cu);
    return __builtin_bit_cast(bf16x8, d);
  };
  // The eight MFMAs of step x, one per slot, with what the next step (ST of the stage in buffers U) needs behind them.
  auto quarter = [&](auto U, auto ST, const Frag &x, Frag &next, auto fetch) {
    constexpr int po = decltype(U)::value % 3 * PB, qo = decltype(U)::value % 2 * QB, st = decltype(ST)::value;
    static_for<8>([&](auto N) {
      constexpr int n = decltype(N)::value, i = n & 3, j = n >> 2;
      acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x.q[j]), x.p[i], acc[j][i], 0, 0, 0);
      if constexpr (n < 2) {
        next.q[n] = *(const u32x4 *)(lds + fq[st] + (qo + n * 32 * 2 * KS));
        if constexpr (st % 2 == 0) {
          raw[2 * n] = *(const u32x4 *)(lds + fp[st / 2] + (po + 2 * n * 32 * KS));
          raw[2 * n + 1] = *(const u32x4 *)(lds + fp[st / 2] + (po + (2 * n + 1) * 32 * KS));
        }
      }
      fetch(N);
      if constexpr (n >= 4) next.p[n - 4] = convert(raw[n - 4][2 * (st & 1)], raw[n - 4][2 * (st & 1) + 1]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, 2> I2;
  typedef std::integral_constant<int, 3> I3;
  // A stage; its first quarter multiplies the step left over from the stage before.  At its barrier every wavefront has seen its
  // own loads of the stage land (the spikes of the next stage may still be in flight) and has left stage kt - 1, whose buffers
  // take the weights of stage kt + 1 and the spikes of stage kt + 2.
  auto stage = [&](auto U, int kt_any, Frag &pend) {
    constexpr int u = decltype(U)::value;
    const int kt = __builtin_amdgcn_readfirstlane(kt_any);
    asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    Frag x, y;
    quarter(U, I0(), pend, x, [&](auto N) {
      constexpr int n = decltype(N)::value;
      if constexpr (n == 2 || n == 3) issue_q(kt + 1, (u + 1) % 2, n - 2);
    });
    quarter(U, I1(), x, y, [&](auto N) {
      constexpr int n = decltype(N)::value;
      if constexpr (n == 2 || n == 3) issue_q(kt + 1, (u + 1) % 2, n);
    });
    quarter(U, I2(), y, x, [&](auto N) {
      constexpr int n = decltype(N)::value;
      if constexpr (n == 2 || n == 3) issue_p(kt + 2, (u + 2) % 3, n - 2);
    });
    quarter(U, I3(), x, pend, [&](auto N) {
      constexpr int n = decltype(N)::value;
      if constexpr (n == 2 || n == 3) issue_p(kt + 2, (u + 2) % 3, n);
    });
  };

  // Scan: the lane's sample and neuron
  const int b = b0 + wm, n = n0 + 64 * wn + lane;
  const bool mine = b < a.B && n < op.ld;
  const float beta = n < op.ld ? op.beta_v[n] : 0.f, theta = a.theta;
  const float big = 0x1p100f, mtheta_big = -theta * 0x1p100f, mtheta = -theta;
  float v = 0.f;
  const unsigned vbytes = (unsigned)a.T * a.B * op.ld * 4u;
  const rsrc_t rV = make_rsrc(op.V, vbytes), rS = make_rsrc(op.S, vbytes / 4);
  const int row = a.B * op.ld, vo = mine ? (b * op.ld + n) * 4 : OOB;
  const int sn = n0 + 64 * wn + 4 * (lane & 15), sg = lane >> 4;
  const int so = b < a.B && sn < op.ld ? b * op.ld + sn : OOB;
  const int shift = 4 * (lane & 7);
  char *const own = lds + wave * (64 * G::PITCH * 4);

  for (int t0 = 0; t0 < a.T; t0 += BM) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 16 * (wave + 4 * q) + (lane >> 2), u = (lane & 3) ^ ((r >> 2) & 3);
      const int t = t0 + (r & 127), s = b0 + (r >> 7);
      pv[q] = t < a.T && s < a.B ? (t * a.B + s) * op.ldp + u * 16 : OOB;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
    Frag pend;                                         // zeros in front of the first stage
#pragma unroll
    for (int j = 0; j < 2; ++j) pend.q[j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 4; ++i) pend.p[i] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
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
#pragma unroll
    for (int k = 0; k < 8; ++k)
      acc[k >> 2][k & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, pend.q[k >> 2]), pend.p[k & 3], acc[k >> 2][k & 3], 0, 0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the stage loads beyond the range have written their zeros
    lds_barrier();                                     // every wavefront is past its fragment reads

    static_for<2>([&](auto HF) {
      constexpr int hf = decltype(HF)::value;
      // I^T: the lane holds step 32 i + lane % 32, register r neuron 8 (r / 4) + 4 h + r % 4 of the tile.
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = 0.5f * acc[j][2 * hf + i][4 * q + e];
            *(f32x4 *)(own + ((32 * i + (lane & 31)) * G::PITCH + 32 * j + 8 * q + 4 * h) * 4) = x;
          }
      const float *const cell = (const float *)own + lane;
      auto read = [&](float (&x)[16], int s0) {
#pragma unroll
        for (int s = 0; s < 16; ++s) x[s] = cell[(s0 + s) * G::PITCH];
      };
      auto steps = [&](const float (&x)[16], int s0) {
        const int t = t0 + 64 * hf + s0;
        if (t >= a.T) return;
#pragma unroll
        for (int s4 = 0; s4 < 16; s4 += 4) {
          unsigned long long m[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int ts = min(t + s4 + s, a.T - 1);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rV, t + s4 + s < a.T ? vo : OOB, ts * row * 4, POL);
            m[s] = __builtin_amdgcn_ballot_w64(v > theta);
            float sp;                                  // 1 if v > theta, else 0
            asm("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(sp) : "v"(v), "v"(big), "v"(mtheta_big));
            v = __builtin_fmaf(mtheta, sp, __builtin_fmaf(beta, v, x[s4 + s]));
          }
          // bits 4 i .. + 3 of the mask of step g, one to a byte
          const uint32_t lo = sg & 2 ? (sg & 1 ? (uint32_t)m[3] : (uint32_t)m[2]) : sg & 1 ? (uint32_t)m[1] : (uint32_t)m[0];
          const uint32_t hi = sg & 2 ? (sg & 1 ? (uint32_t)(m[3] >> 32) : (uint32_t)(m[2] >> 32))
                                     : sg & 1 ? (uint32_t)(m[1] >> 32) : (uint32_t)(m[0] >> 32);
          const uint32_t bits = ((lane & 8 ? hi : lo) >> shift) & 15u;
          const int ts = t + s4 + sg;
          // (half a cache line; never non-temporal: 310 us instead of 283 at the second layer of 700-1024-1024-20, T = 256, B = 512)
          __builtin_amdgcn_raw_buffer_store_b32(__umul24(bits, 0x204081u) & 0x01010101u, rS, ts < a.T && so != OOB ? so + ts * row : OOB, 0, 0);
        }
      };
      float xa[16], xb[16];
      read(xa, 0);
      read(xb, 16);
      steps(xa, 0);
      read(xa, 32);
      steps(xb, 16);
      read(xb, 48);
      steps(xa, 32);
      steps(xb, 48);
    });
    lds_barrier();                                     // every wavefront has read its currents: the next block's stages
  }
}

hipError_t layer_forward_wide(hipStream_t st, const LayerForwardArgs &a);

}  // namespace snn
