// Forward pass of whole feed-forward LIF layers in one launch for rasters of at most 64 steps: several
// samples to a tile (see layer_forward.hpp for the kernel that gives a workgroup one sample).
//
// There the 128 rows of a workgroup's product tile are 128 steps of one sample; at 16 steps seven of
// eight rows are zeros, every workgroup still pulls all of its weights through its compute unit, and
// the scan walks 128 rows.  Here the rows are 128 / SL samples in slots of SL = 16, 32 or 64 steps (the
// least that holds T), so a launch has that many times fewer workgroups and bytes of weights:
//   1. product of the 128 rows on the same streamed pipeline (SpikeTile);
//   2. the tile goes to LDS;
//   3. scan, one chain (slot, neuron) per thread at a time, at most 64 steps per thread for any SL,
//      potentials written back in place;
//   4. all threads store V and S as whole rows;
//   5. the readout as there (READOUT): its scan cuts the rows in segments of 16, and a segment takes its
//      entry state from the segments before it in the same slot.
// 700-200-150-20 fp32, T = 30, B = 500: 150.6 us per step with product and scan apart, 121 so; 700-157-157-20,
// T = 20, B = 209 (forward, loss and logits): 63.8 apart, 66.6 with a sample to a tile, 58 so.
//
// ADAPT: layers with adaptive firing thresholds (see lif_forward_kernel), at any number of steps: the second
// state A needs a tile of its own beside V, which fits for 64 neurons, and the kernel above hands finished rows to
// storing wavefronts that would have to know it.  Rasters of more than 64 steps take SL = 128, a block
// after the other, the two states in the scanning thread's registers.  What bounds it is the chain of a step,
// four dependent operations (decision, adaptation, threshold, distance) where the plain neuron has two.
// 700-256-256-20, T = B = 128, per step: 131 us with product and scan apart, 122 so; 700-40-40-20, T = 128, B = 64: 88 and 77.
#pragma once
#include "layer_forward.hpp"

namespace snn {

template <int TN, bool READOUT, int NL, bool PACKED, int NP, bool ADAPT = false>
__global__ __launch_bounds__(256, 2) void lif_layer_forward_short_kernel(const LayerForwardArgs a) {
  typedef SpikeTile<2, 2, 2, TN, 3> Tile;
  constexpr int BM = Tile::BM, BN = Tile::BN, PI = Tile::PI, QI = Tile::QI, KS = Tile::KSTAGE;
  constexpr int TM = 2, CP = BN * 4 + 16, JP = 36;
  constexpr int STAGES = Tile::lds_bytes(false, NP) > Tile::lds_bytes(PACKED, NP) ? Tile::lds_bytes(false, NP) : Tile::lds_bytes(PACKED, NP);
  constexpr int TILES = (ADAPT ? 2 : 1) * BM * CP, LDS_BYTES = STAGES > TILES ? STAGES : TILES;
  static_assert(!ADAPT || (TN == 1 && !READOUT && NL == 1), "adaptive layers: 64 neurons, alone in their launch");
  static_assert(BM == 128 && LDS_BYTES <= 80 * 1024, "two workgroups per compute unit");
  __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
  __shared__ float x_e[8][32], x_best[8][32];
  __shared__ int x_tb[8][32];

  const int sl2 = a.slot_log2, SL = 1 << sl2, SPT = BM >> sl2;   // steps per slot, samples per workgroup
  const int parts = a.parts;
  const int part = (blockIdx.x >> 3) % parts;
  const int b0 = ((blockIdx.x >> 3) / parts * 8 + (blockIdx.x & 7)) * SPT;   // the parts of a workgroup's samples share an XCD
  if (b0 >= a.B) return;
  const int n0 = part * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, h = lane >> 5;
  const float theta = a.theta;
  const float big = 0x1p100f, mtheta_big = -theta * 0x1p100f, mtheta = -theta;
  // element (t, b) of row r of the tile, or -1
  int t0 = 0;                                         // (only ADAPT has more than one block)
  auto pos = [&](int r) {
    const int t = t0 + (r & (SL - 1)), b = b0 + (r >> sl2);
    return t < a.T && b < a.B ? t * a.B + b : -1;
  };
  float v_in = 0.f, ad_in = 0.f;                      // ADAPT: the states entering a block of 128 steps
  do {
  const int steps = min(SL, (a.T - t0 + 15) & ~15);   // whole groups of 16

  static_for<NL>([&](auto LI) {
    constexpr int li = decltype(LI)::value;
    constexpr bool last = li == NL - 1;
    const LayerForwardOp &op = a.op[li];
    const int ld = op.ld, nk = (op.kc + KS - 1) / KS;
    const u32x4 rp = raw_rsrc(op.P, op.p_bytes), rq = raw_rsrc(op.Q, op.q_bytes);
    const rsrc_t rV = make_rsrc(op.V, (unsigned)a.T * a.B * ld * 4u), rS = make_rsrc(op.S, (unsigned)a.T * a.B * ld);
    // 1. product
    int qv[QI], pv[PI];
#pragma unroll
    for (int q = 0; q < QI; ++q) {
      const int row = Tile::q_row(wave, lane, q);
      qv[q] = ((n0 + row) * op.ldq + Tile::q_chunk(row, lane) * 8) * 2;
    }
#pragma unroll
    for (int q = 0; q < PI; ++q) {
      const int row = Tile::p_row(wave, lane, q), e = pos(row);
      pv[q] = e >= 0 ? e * op.ldp + Tile::p_unit(row, lane) * 16 : OOB;
    }
    f32x16 acc[TM][TN];
    if constexpr (PACKED && li == 0) {
      PackedRows pk;
      pk.rsrc = make_rsrc(op.P, op.p_bytes);
      pk.base = ((t0 >> 3) * a.B + b0) * op.ldp;
      pk.row_stride = a.B * op.ldp;
      pk.rows = ((a.T + 7) >> 3) - (t0 >> 3);
      pk.kbytes = op.ldp;
      pk.slot_log2 = sl2 - 3;
      pk.samples = a.B - b0;
      if constexpr (NP == 3) Tile::template run_planes<true>(lds, rp, rq, pv, qv, op.q_plane, nk, wave, lane, acc, &pk);
      else Tile::template run<true>(lds, rp, rq, pv, qv, nk, wave, lane, acc, &pk);
    } else {
      if constexpr (NP == 3) Tile::run_planes(lds, rp, rq, pv, qv, op.q_plane, nk, wave, lane, acc);
      else Tile::run(lds, rp, rq, pv, qv, nk, wave, lane, acc);
    }

    // 2. (the lane holds row lane & 31 of its row tile, register r neuron 8 (r / 4) + 4 h + r % 4)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 x = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *(f32x4 *)(lds + ((wm * TM + i) * 32 + (lane & 31)) * CP + ((wn * TN + j) * 32 + 8 * q + 4 * h) * 4) = x;
        }
    __syncthreads();

    // the readout's weights arrive under the scan
    bf16x8 wr[NP][READOUT && last ? BN / 16 : 1];
    if constexpr (READOUT && last) {
      const rsrc_t rQ = make_rsrc(a.Qr, a.qr_bytes);
#pragma unroll
      for (int pl = 0; pl < NP; ++pl)
#pragma unroll
        for (int kk = 0; kk < BN / 16; ++kk) {
          const int n = 16 * kk + 8 * h;
          wr[pl][kk] = __builtin_bit_cast(bf16x8, ld_b128(rQ, n < a.ldqr ? ((lane & 31) * a.ldqr + n) * 2 : OOB, pl * (int)a.qr_plane));
        }
    }

    // 3. scan (the spike decision without a compare, see layer_forward.hpp)
    const float beta = n0 + tid % BN < ld ? op.beta_v[n0 + tid % BN] : 0.f;
    for (int q = tid; q < SPT * BN; q += 256) {       // (256 is a multiple of BN: the same neuron each time)
      constexpr int U = 16;
      float *cell = (float *)(lds + (q / BN << sl2) * CP + (q % BN) * 4);
      float v = ADAPT ? v_in : 0.f, ad = ADAPT ? ad_in : 0.f, nxt[U];
#pragma unroll
      for (int u = 0; u < U; ++u) nxt[u] = cell[u * (CP / 4)];
      for (int s0 = 0; s0 < steps; s0 += U) {
        float cur[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cur[u] = nxt[u];
        if (s0 + U < steps) {
#pragma unroll
          for (int u = 0; u < U; ++u) nxt[u] = cell[(s0 + U + u) * (CP / 4)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" : "+v"(cur[u]));
#pragma unroll
        for (int u = 0; u < U; ++u) {
          cell[(s0 + u) * (CP / 4)] = v;
          float s;
          if constexpr (ADAPT) {
            cell[(BM + s0 + u) * (CP / 4)] = ad;
            const float thr = theta + ad;
            asm("v_mul_f32 %0, %1, %2 clamp" : "=v"(s) : "v"(v - thr), "v"(big));
            v = __builtin_fmaf(-thr, s, __builtin_fmaf(beta, v, cur[u]));
            ad = __builtin_fmaf(op.gamma, ad, op.kappa * s);
            continue;
          }
          asm("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(s) : "v"(v), "v"(big), "v"(mtheta_big));
          v = __builtin_fmaf(mtheta, s, __builtin_fmaf(beta, v, cur[u]));
        }
      }
      if (ADAPT && SL == BM) { v_in = v; ad_in = ad; }
    }
    __syncthreads();

    // 4. store
    constexpr int VL = BN / 4, SLC = BN / 16;         // pieces per row of V and of S
#pragma unroll
    for (int p0 = 0; p0 < BM * VL; p0 += 256) {
      const int p = p0 + tid, row = p / VL, col = (p % VL) * 4, e = pos(row);
      const u32x4 x = *(const u32x4 *)(lds + row * CP + col * 4);
      const int vo = e >= 0 && n0 + col < ld ? (e * ld + n0 + col) * 4 : OOB;
      if (a.nt_store) __builtin_amdgcn_raw_buffer_store_b128(x, rV, vo, 0, NT);
      else __builtin_amdgcn_raw_buffer_store_b128(x, rV, vo, 0, 0);
      if constexpr (ADAPT) {
        const u32x4 xa = *(const u32x4 *)(lds + (BM + row) * CP + col * 4);
        const rsrc_t rA = make_rsrc(op.A, (unsigned)a.T * a.B * ld * 4u);
        if (a.nt_store) __builtin_amdgcn_raw_buffer_store_b128(xa, rA, vo, 0, NT);
        else __builtin_amdgcn_raw_buffer_store_b128(xa, rA, vo, 0, 0);
      }
    }
#pragma unroll
    for (int p0 = 0; p0 < BM * SLC; p0 += 256) {
      const int p = p0 + tid, row = p / SLC, col = (p % SLC) * 16, e = pos(row);
      u32x4 x;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 f = *(const f32x4 *)(lds + row * CP + (col + 4 * q) * 4);
        if constexpr (ADAPT) {                        // (the same difference as in the scan, against zero)
          const f32x4 fa = *(const f32x4 *)(lds + (BM + row) * CP + (col + 4 * q) * 4);
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) f[e4] = f[e4] - (theta + fa[e4]) > 0.f ? INFINITY : -INFINITY;
        }
        x[q] = (f[0] > theta ? 1u : 0u) | (f[1] > theta ? 0x100u : 0u) | (f[2] > theta ? 0x10000u : 0u) |
               (f[3] > theta ? 0x1000000u : 0u);
      }
      const int so = e >= 0 && n0 + col + 16 <= ld ? e * ld + n0 + col : OOB;
      if (a.nt_store) __builtin_amdgcn_raw_buffer_store_b128(x, rS, so, 0, NT);
      else __builtin_amdgcn_raw_buffer_store_b128(x, rS, so, 0, 0);
      if (ld & 8) {                                   // the row's last eight neurons are half a piece
        const u32x2 x8 = {x.x, x.y};
        st_b64(rS, e >= 0 && n0 + col + 8 == ld ? e * ld + n0 + col : OOB, 0, x8);
      }
    }

    if constexpr (READOUT && last) {
      // 5. currents of the readout: a wavefront takes 32 rows, the lane ends up with its row's
      const int row = 32 * wave + (lane & 31), e = pos(row);
      f32x16 jt;
#pragma unroll
      for (int r = 0; r < 16; ++r) jt[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < BN / 16; ++kk) {
        const f32x4 p0 = *(const f32x4 *)(lds + row * CP + (16 * kk + 8 * h) * 4);
        const f32x4 p1 = *(const f32x4 *)(lds + row * CP + (16 * kk + 8 * h + 4) * 4);
        u32x4 sp;
        sp.x = (p0[0] > theta ? 0x3F80u : 0u) | (p0[1] > theta ? 0x3F800000u : 0u);
        sp.y = (p0[2] > theta ? 0x3F80u : 0u) | (p0[3] > theta ? 0x3F800000u : 0u);
        sp.z = (p1[0] > theta ? 0x3F80u : 0u) | (p1[1] > theta ? 0x3F800000u : 0u);
        sp.w = (p1[2] > theta ? 0x3F80u : 0u) | (p1[3] > theta ? 0x3F800000u : 0u);
#pragma unroll
        for (int pl = NP - 1; pl >= 0; --pl)
          jt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[pl][kk], __builtin_bit_cast(bf16x8, sp), jt, 0, 0, 0);
      }
      const rsrc_t rJ = make_rsrc(a.J, (unsigned)a.T * a.B * a.ldj * 4u);
      __syncthreads();                                // V has been read: the tile's space is free
      float *Jt = (float *)lds;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 8 * q + 4 * h;
        const f32x4 x = {jt[4 * q], jt[4 * q + 1], jt[4 * q + 2], jt[4 * q + 3]};
        st_b128(rJ, e >= 0 && c + 3 < a.ldj ? (e * a.ldj + c) * 4 : OOB, 0, __builtin_bit_cast(u32x4, x));
        *(f32x4 *)&Jt[row * JP + c] = x;
      }
      __syncthreads();

      // LI scan: thread -> segment of 16 rows tid / 32, class tid % 32
      const int g = tid >> 5, c = tid & 31, per = SL >> 4;       // segments per slot
      const int slot = g / per, first = slot * per, ts0 = 16 * (g - first), b = b0 + slot;
      const float beta_r = c < a.ldj ? a.beta_r[c] : 0.f;
      float bseg = beta_r;
#pragma unroll
      for (int i = 1; i < 16; i *= 2) bseg *= bseg;
      float j[16], e0 = 0.f;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        j[k] = Jt[(16 * g + k) * JP + c];
        e0 = beta_r * e0 + j[k];
      }
      x_e[g][c] = e0;
      __syncthreads();
      float y = 0.f;
      for (int v = first; v < g; ++v) y = bseg * y + x_e[v][c];
      float best = -INFINITY, ysum = 0.f;
      int tb = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        y = beta_r * y + j[k];
        Jt[(16 * g + k) * JP + c] = y;
        if (ts0 + k < a.T) {
          ysum += y;
          if (y > best) { best = y; tb = ts0 + k; }
        }
      }
      x_best[g][c] = a.integral ? ysum : best;
      x_tb[g][c] = a.integral ? 0 : tb;
      __syncthreads();
      const rsrc_t rY = make_rsrc(a.Y, (unsigned)a.T * a.B * a.ldj * 4u);
#pragma unroll
      for (int k = 0; k < BM / 32; ++k) {             // 8 lanes x 16 bytes per row, 32 rows per instruction
        const int r = 32 * k + (tid >> 3), cc = (tid & 7) * 4, er = pos(r);
        const u32x4 x = *(const u32x4 *)&Jt[r * JP + cc];
        st_b128(rY, er >= 0 && cc + 3 < a.ldj ? (er * a.ldj + cc) * 4 : OOB, 0, x);
      }
      // first maximiser over the slot's segments (integral loss: the sum of their sums, in order)
      best = x_best[first][c];
      tb = x_tb[first][c];
      for (int v = first + 1; v < first + per; ++v) {
        const float bv = x_best[v][c];
        if (a.integral) best += bv;
        else if (bv > best) { best = bv; tb = x_tb[v][c]; }
      }
      const bool valid = b < a.B, live = valid && c < a.C;
      const int p = b * a.ldj + c;
      if (live && g == first) { a.z[p] = best; a.tstar[p] = tb; }
      // softmax cross-entropy of the sample (every segment of its slot, for dz)
      float m = live ? best : -INFINITY;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
      const float ex = live ? expf(best - m) : 0.f;
      float sum = ex;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
      int lab = valid ? a.labels[b] : 0;
      if (lab < 0 || lab >= a.C) { if (g == first && c == 0) atomicOr(a.err, 1); lab = 0; }
      float zl = (live && c == lab) ? best : 0.f;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) zl += __shfl_xor(zl, o);
      const float d = live ? (ex / sum - (c == lab ? 1.f : 0.f)) / (float)a.B : 0.f;
      if (g == first) {
        if (live) a.dz[p] = d;
        if (valid && c == 0) a.loss_b[b] = m + logf(sum) - zl;
      }
      // dJ of the segment, entered in closed form
      const float l2b = log2f(beta_r);
      float hh;
      if (a.integral) {
        const int n = a.T - (ts0 + 16);
        hh = n <= 0 ? 0.f : beta_r == 1.f ? d * (float)n : d * (1.f - exp2f((float)n * l2b)) / (1.f - beta_r);
      } else {
        const int n = tb - (ts0 + 16);
        hh = n > 0 ? d * exp2f((float)n * l2b) : n == 0 ? d : 0.f;
      }
      __syncthreads();                                // Y has been stored
      uint32_t *Ht = (uint32_t *)lds;
#pragma unroll
      for (int k = 15; k >= 0; --k) {
        hh = beta_r * hh + ((a.integral ? ts0 + k < a.T : ts0 + k == tb) ? d : 0.f);
        Ht[(16 * g + k) * JP + c] = NP == 1 ? pack_hl(hh) : __float_as_uint(hh);
      }
      __syncthreads();
      const rsrc_t rdJ = make_rsrc(a.dJ, (unsigned)a.T * a.B * a.ldj * 4u);
#pragma unroll
      for (int k = 0; k < BM / 32; ++k) {
        const int r = 32 * k + (tid >> 3), cc = (tid & 7) * 4, er = pos(r);
        const u32x4 x = *(const u32x4 *)&Ht[r * JP + cc];
        st_b128(rdJ, er >= 0 && cc + 3 < a.ldj ? (er * a.ldj + cc) * 4 : OOB, 0, x);
      }
    }
    // The layer above reads these spikes back from memory.
    if (!last) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
  });
  t0 += SL;
  if (ADAPT) __syncthreads();                         // the next product's stages overwrite the tiles
  } while (ADAPT && t0 < a.T);
}

}  // namespace snn
