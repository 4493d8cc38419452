// Reverse pass of a whole feed-forward LIF layer below a narrow layer in one launch: the
// spike gradients dS = dX W^T from the current gradients dX of the layer above (at most 128
// columns: the readout or a narrow spiking layer), the surrogate, the reverse scan
// g_t -> dI_t (Eq. 1-2 differentiated; see lif_reverse_kernel), dI stored as hi/lo words (F32:
// fp32 products; dX and dI are fp32, both operands of dS enter in three bfloat16 pieces).
//
// lif_reverse_top_kernel does the same with one wavefront per 64 chains, each lane walking
// its chain through global memory: per step a load, a store and a share of the dX fetches,
// which is what bounds it (a wavefront issues a memory instruction about every 60 cycles).
// Here a workgroup owns one sample and 64 neurons (two or three workgroups share a compute unit and
// overlap each other's phases: 99.8 us per step at 700-128-128-20 against 104.8 with 128 neurons), and
// per block of 64 steps, last block first:
//   1. V (64 x 64) and dX (64 x ldc words) arrive through 16-byte loads issued one block
//      ahead (they land during the previous block's scan) and go to LDS;
//   2. dS: 32x32x16 bfloat16 MFMAs, the rounded weights of the wavefront's 32 neurons resident
//      in registers, the hi and lo halves of dX as the second operand, lo first; a wavefront
//      holds 32 steps x 32 neurons of the result;
//   3. still in the MFMA layout, every lane turns its elements into the two coefficients of
//      the step: with s = surr(V - theta), g' = beta g + s (dS - theta g) = c1 g + c2,
//      c1 = beta - s theta, c2 = s dS.  The surrogate (a division or an exponential) is
//      computed here by all four wavefronts, not inside the sequential scan;
//   4. scan: one wavefront, a neuron per lane, 64 steps of one fused multiply-add each on
//      LDS (coefficients read 8 steps ahead, g written back in place of c2);
//   5. store: all wavefronts pack g into hi/lo words and write whole rows, 16 bytes per lane.
// SLOTS (at most 32 steps, one block): the block's rows are 64 / SL samples in slots of SL = 16 or 32 steps, a
// wavefront scans a slot; 16 steps in a block of their own leave three of four rows to zeros.
// A layer whose width is no multiple of 64 (not FULL) has columns without neurons in its last part: they
// read zeros, stay zero and are not stored.
// g (and the decay gradient's partial sum) stay in the scanning lanes' registers from block
// to block.  Rows past T read as zero: c2 = 0 there and g, zero at the start, stays zero.
#pragma once
#include "surrogate.hpp"
#include "gemm_stream.hpp"
#include <type_traits>

namespace snn {

struct LayerReverseArgs {
  const uint32_t *dX;      // current gradients of the layer above [T*B][ldc], hi/lo words (F32: fp32)
  int ldc;                 // its padded columns (multiple of 8, at most 128; layer_reverse_wide: any)
  const uint16_t *Wq;      // W[n][c] bfloat16 planes, row n = neuron of this layer, zero beyond the valid columns
  int ldq;
  unsigned wq_bytes, wq_plane;   // all planes; bytes between planes
  const float *V;          // [T*B][ld]
  uint32_t *dI;            // [T*B][ld] hi/lo words
  const float *beta_v;     // [ld]
  float theta, slope;
  float *db_part;          // [B][ld] per-sample parts of the decay gradient, or NULL
  int T, B, ld;
  int nt_store;            // dI streams past the caches
  int slot_log2;           // 6: a block of 64 steps is one sample's; 4 or 5: slots of 16 or 32 steps
  const float *A;          // layer_reverse_wide: adaptation in force at each step [T*B][ld], its decay and its rise per spike, or NULL
  float gamma, kappa;
};
hipError_t layer_reverse(hipStream_t st, const LayerReverseArgs &a, int surrogate, bool f32);

template <int KS, int SURR, bool F32 = false, bool FULL = true, bool SLOTS = false>
__global__ __launch_bounds__(256, 2) void lif_layer_reverse_kernel(const LayerReverseArgs a) {
  constexpr int BM = 64, BN = 64;                     // steps of a block, neurons
  constexpr int NV = BN / 16;                         // 16-byte accesses per thread to a 64 x BN fp32 tile
  constexpr int LPR = BN / 4;                         // lanes per row in those accesses
  constexpr int CP = BN * 4 + 16;                     // bytes between time rows of the fp32 tiles
  constexpr int PITCH = CP / 4;
  constexpr int XP = F32 ? KS * 64 + 16 : KS * 128 + 16;   // bytes between time rows of the dX tile (32 KS words; F32: 32 KS bfloat16 per plane)
  constexpr int XPL = BM * XP, XT = F32 ? 3 * XPL : XPL;   // F32: bytes between planes; bytes of the tile
  constexpr int TILE = BM * CP;
  constexpr int KK = 2 * KS;                          // 16-wide MFMA steps over the columns above
  constexpr int LDS_BYTES = TILE + (XT > 2 * TILE ? XT : 2 * TILE);   // the dX tile shares the space of the coefficient tiles
  static_assert(LDS_BYTES <= 80 * 1024, "two workgroups per compute unit");
  __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
  __shared__ __attribute__((aligned(16))) float betas[BN];
  char *const Vt = lds, *const C1 = lds + TILE, *const C2 = lds + 2 * TILE, *const Xt = C1;

  // Workgroup ids are dealt round-robin to the 8 XCDs: the parts of a sample take ids 8 apart.
  const int parts = FULL ? a.ld / BN : (a.ld + BN - 1) / BN;
  const int part = (blockIdx.x >> 3) % parts;
  const int sl2 = SLOTS ? a.slot_log2 : 6;
  const int b = ((blockIdx.x >> 3) / parts * 8 + (blockIdx.x & 7)) << (6 - sl2);   // the first sample
  if (b >= a.B) return;
  static_assert(!SLOTS || !FULL, "slots: any width");
  const int n0 = part * BN;
  // row of the block at t0: its step and sample, and whether they exist
  auto step = [&](int t0, int row) { return SLOTS ? row & ((1 << sl2) - 1) : t0 + row; };
  auto sample = [&](int row) { return SLOTS ? b + (row >> sl2) : b; };
  auto exists = [&](int t, int s) { return t < a.T && (!SLOTS || s < a.B); };
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, h = lane >> 5;
  const float theta = a.theta, slope = a.slope;
  const unsigned vbytes = (unsigned)a.T * a.B * a.ld * 4u;
  const rsrc_t rV = make_rsrc(a.V, vbytes), rdI = make_rsrc(a.dI, vbytes);
  const rsrc_t rX = make_rsrc(a.dX, (unsigned)a.T * a.B * a.ldc * 4u), rW = make_rsrc(a.Wq, a.wq_bytes);
  if (tid < BN) betas[tid] = FULL || n0 + tid < a.ld ? a.beta_v[n0 + tid] : 0.f;

  // A block's global loads: V as NV x 16 bytes per thread, dX as KK x 16
  // bytes per thread over rows of 8 KS chunks (chunks beyond ldc read as zero).
  u32x4 xv[NV], xd[KK];
  auto fetch = [&](int t0) {                          // t0 < 0: nothing is read
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int row = (256 / LPR) * k + tid / LPR, t = step(t0, row), s = sample(row), col = (tid % LPR) * 4;
      xv[k] = ld_b128(rV, t0 >= 0 && exists(t, s) && (FULL || n0 + col < a.ld) ? ((t * a.B + s) * a.ld + n0 + col) * 4 : OOB, 0);
    }
#pragma unroll
    for (int k = 0; k < KK; ++k) {
      const int idx = k * 256 + tid, row = idx / (8 * KS), ch = idx % (8 * KS), t = step(t0, row), s = sample(row);
      xd[k] = ld_b128(rX, t0 >= 0 && exists(t, s) && ch * 4 + 3 < a.ldc ? ((t * a.B + s) * a.ldc + ch * 4) * 4 : OOB, 0);
    }
  };
  auto fill = [&]() {
#pragma unroll
    for (int k = 0; k < NV; ++k) *(u32x4 *)(Vt + ((256 / LPR) * k + tid / LPR) * CP + (tid % LPR) * 16) = xv[k];
#pragma unroll
    for (int k = 0; k < KK; ++k) {
      const int idx = k * 256 + tid, row = idx / (8 * KS), ch = idx % (8 * KS);
      if constexpr (F32) {
        // split here, once per word; in the product every word would be split by the wavefronts of both
        // neuron halves, one step behind the other (700-128-128-20, T = 500, B = 4: 5 us per block)
        typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
        bf16x4 xp[3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x = __uint_as_float(xd[k][e]);
#pragma unroll
          for (int pl = 0; pl < 3; ++pl) {
            const __bf16 piece = (__bf16)x;
            xp[pl][e] = piece;
            x -= (float)piece;
          }
        }
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *(bf16x4 *)(Xt + pl * XPL + row * XP + ch * 8) = xp[pl];
      } else *(u32x4 *)(Xt + row * XP + ch * 16) = xd[k];
    }
  };

  int t0 = (a.T - 1) / BM * BM;
  fetch(t0);                                          // the first block's loads go out before anything else

  // First MFMA operand: W[n][c], lane -> neuron (lane & 31) of the 32-neuron tile, columns
  // 16 kk + 8 h .. +7.  Resident for the whole kernel.
  // (F32 with 128 columns: the third plane, one of the six products, is fetched per block; resident it makes
  // registers spill, and each spill's reload waits for the next block's loads in flight)
  constexpr int NP = F32 ? 3 : 1, NRES = F32 && KS == 4 ? 2 : NP;
  bf16x8 wf[NP][KK];
  auto weights = [&](int pl) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int n = n0 + 32 * wn + (lane & 31), c = 16 * kk + 8 * h;
      wf[pl][kk] = __builtin_bit_cast(bf16x8, ld_b128(rW, c + 7 < a.ldq ? (n * a.ldq + c) * 2 : OOB, pl * (int)a.wq_plane));
    }
  };
#pragma unroll
  for (int pl = 0; pl < NRES; ++pl) weights(pl);

  float g = 0.f, db = 0.f;                            // state of neuron n0 + tid (wavefront 0; SLOTS: n0 + lane)

  for (int blk = 0; t0 >= 0; t0 -= BM, ++blk) {
    fill();
    if (NRES < NP) weights(NRES);
    __syncthreads();
    fetch(t0 - BM);

    // 2. dS^T tile: rows = neurons, columns = steps; the lane holds step 32 wm + (lane & 31)
    // and register r neuron 8 (r / 4) + 4 h + (r % 4) of its 32-neuron tile.
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    if constexpr (F32) {
      // pieces p of dX and q of W with p + q < 3: every product above 2^-24
      const char *px = Xt + (32 * wm + (lane & 31)) * XP + 16 * h;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        bf16x8 xp[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) xp[pl] = *(const bf16x8 *)(px + pl * XPL + 32 * kk);
#pragma unroll
        for (int s = 2; s >= 0; --s)
#pragma unroll
          for (int pl = 0; pl <= s; ++pl)
            if (s - pl < NRES) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s - pl][kk], xp[pl], acc, 0, 0, 0);
      }
      if constexpr (NRES < NP) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const bf16x8 xp = *(const bf16x8 *)(px + 32 * kk);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[NRES][kk], xp, acc, 0, 0, 0);
        }
      }
    } else {
      bf16x8 hi[KK];
      const char *px = Xt + (32 * wm + (lane & 31)) * XP + 32 * h;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const u32x4 j0 = *(const u32x4 *)(px + 64 * kk), j1 = *(const u32x4 *)(px + 64 * kk + 16);
        u32x4 hh, ll;
        hh.x = __builtin_amdgcn_perm(j0.y, j0.x, 0x05040100u); ll.x = __builtin_amdgcn_perm(j0.y, j0.x, 0x07060302u);
        hh.y = __builtin_amdgcn_perm(j0.w, j0.z, 0x05040100u); ll.y = __builtin_amdgcn_perm(j0.w, j0.z, 0x07060302u);
        hh.z = __builtin_amdgcn_perm(j1.y, j1.x, 0x05040100u); ll.z = __builtin_amdgcn_perm(j1.y, j1.x, 0x07060302u);
        hh.w = __builtin_amdgcn_perm(j1.w, j1.z, 0x05040100u); ll.w = __builtin_amdgcn_perm(j1.w, j1.z, 0x07060302u);
        hi[kk] = __builtin_bit_cast(bf16x8, hh);
        const bf16x8 lo = __builtin_bit_cast(bf16x8, ll);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[0][kk], lo, acc, 0, 0, 0);
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[0][kk], hi[kk], acc, 0, 0, 0);
    }
    __syncthreads();                                  // every wavefront has read the dX tile: C1 takes its place

    // 3. coefficients
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = 32 * wm + (lane & 31), n = 32 * wn + 8 * q + 4 * h;
      const f32x4 vv = *(const f32x4 *)(Vt + t * CP + n * 4);
      const f32x4 bb = *(const f32x4 *)(&betas[n]);
      f32x4 c1, c2;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float s = surr_rcp<SURR>(slope, vv[e] - theta);
        c1[e] = bb[e] - s * theta;
        c2[e] = s * acc[4 * q + e];
      }
      *(f32x4 *)(C1 + t * CP + n * 4) = c1;
      *(f32x4 *)(C2 + t * CP + n * 4) = c2;
    }
    __syncthreads();

    // 4. scan, steps t0 + 63 down to t0: dI_t = g, then g <- c1 g + c2 (and db += g V_t)
    const int scans = SLOTS ? 64 >> sl2 : 1, slot = SLOTS ? wave : 0, rows = 1 << sl2;   // SLOTS: the wavefront's
    if (wave < scans) {
      const int cell = SLOTS ? (slot << sl2) * CP + lane * 4 : tid * 4;
      const float *p1 = (const float *)(C1 + cell), *pv = (const float *)(Vt + cell);
      float *p2 = (float *)(C2 + cell);
      auto scan = [&](auto DB) {
        constexpr bool with_db = decltype(DB)::value;
        constexpr int U = F32 && KS == 4 ? 4 : 8;
        float n1[U], n2[U], nv[U];
        auto read = [&](int s0) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            n1[u] = p1[(s0 + u) * PITCH];
            n2[u] = p2[(s0 + u) * PITCH];
            if (with_db) nv[u] = pv[(s0 + u) * PITCH];
          }
        };
        read((SLOTS ? rows : BM) - U);
        for (int s0 = (SLOTS ? rows : BM) - U; s0 >= 0; s0 -= U) {
          float c1[U], c2[U], vv[U];
#pragma unroll
          for (int u = 0; u < U; ++u) { c1[u] = n1[u]; c2[u] = n2[u]; vv[u] = with_db ? nv[u] : 0.f; }
          if (s0 >= U) read(s0 - U);                  // the next 8 steps' coefficients, before these 8 are taken
#pragma unroll
          for (int u = 0; u < U; ++u) asm volatile("" : "+v"(c1[u]), "+v"(c2[u]));
#pragma unroll
          for (int u = U - 1; u >= 0; --u) {
            p2[(s0 + u) * PITCH] = g;
            if (with_db) db = __builtin_fmaf(g, vv[u], db);
            g = __builtin_fmaf(c1[u], g, c2[u]);
          }
        }
      };
      if (a.db_part) scan(std::true_type()); else scan(std::false_type());
    }
    __syncthreads();

    // 5. store: 16 lanes x 16 bytes per row
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int row = (256 / LPR) * k + tid / LPR, col = (tid % LPR) * 4, t = step(t0, row), s = sample(row);
      const f32x4 gq = *(const f32x4 *)(C2 + row * CP + col * 4);
      u32x4 w;
      if (F32) w = __builtin_bit_cast(u32x4, gq);
      else { w.x = pack_hl(gq[0]); w.y = pack_hl(gq[1]); w.z = pack_hl(gq[2]); w.w = pack_hl(gq[3]); }
      const int vo = exists(t, s) && (FULL || n0 + col < a.ld) ? ((t * a.B + s) * a.ld + n0 + col) * 4 : OOB;
      if (a.nt_store) __builtin_amdgcn_raw_buffer_store_b128(w, rdI, vo, 0, NT);
      else __builtin_amdgcn_raw_buffer_store_b128(w, rdI, vo, 0, 0);
    }
    // The next block's fill writes V and dX, which takes the place of C1 and, when it is larger than
    // C1, of part of C2, which this store phase is still reading.
    if (XT > TILE) __syncthreads();
  }
  if (SLOTS) {
    const int s = b + wave;
    if (a.db_part && wave < (64 >> sl2) && s < a.B && n0 + lane < a.ld) a.db_part[s * a.ld + n0 + lane] = db;
  } else if (a.db_part && tid < BN && (FULL || n0 + tid < a.ld)) a.db_part[b * a.ld + n0 + tid] = db;
}

}  // namespace snn
