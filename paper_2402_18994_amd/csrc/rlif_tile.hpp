// Recurrent LIF layers of up to 256 neurons: V_{t+1} = beta V_t + I_t + S_t R - theta S_t with S_t the
// spikes just emitted from V_t, and the reverse recursion of the same loop.  The whole time loop of a
// direction is one launch; a workgroup owns four samples and all neurons, so nothing of the recurrence
// leaves it.
//
// What bounds a step is its dependent chain on one compute unit: spikes (or g) into LDS, barrier,
// fragments out of LDS, MFMAs, update.  The chain is short when a lane carries few values and when a
// wavefront reads the exchange tile for many neurons:
//   * a wavefront holds 32 neurons (two 16-row tiles of R, in registers for all T steps), so the tile
//     passes through the LDS once per 32 neurons;
//   * four samples instead of the sixteen columns of the MFMA.  Forward: every sample fills four
//     columns, and each of the four lanes that then hold the same sums keeps two neurons.  Reverse: the
//     columns hold the bfloat16 planes of g (hi and lo, twice; hi, mid, lo with fp32 weights), so that one
//     MFMA and one fragment read serve all planes, and a rotation within the row of 16 lanes adds them;
//   * operands and results go straight between registers and memory, PF steps ahead.
// 700-128-128-20, T = 128, B = 256, per layer: forward 55.8 -> 35.2 us (0.28 us per step), reverse 78.4
// -> 48.2 us; sixteen samples and 16 neurons per wavefront, the form before, is the left figure.  (Two such
// layers above each other on rounded weights run as a pair, rlif_pair.hpp.)  Eight
// samples: 38.4 and 54.1 us; 64 neurons per wavefront: 57 and 83 us.  At 256 neurons 67 and 90 us
// where a launch per step took 128 x 4.1 and 128 x 4.8 us and the host's time to launch them.  With no
// memory access at all the steps take 0.27 and 0.29 us.
//
// These kernels are a translation unit of their own because they want MFMA results in ordinary vector
// registers (-amdgpu-mfma-vgpr-form, see build.py): sixteen moves a step less.
#pragma once
#include "surrogate.hpp"

namespace snn {

// x of the lane N columns further in its row of 16 lanes.
template <int N> __device__ __forceinline__ float row_ror(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xF, 0xF, false));
}
// a where mask is all ones, b where it is zero: one v_bfi_b32.  (A choice between elements of an MFMA result
// written with ?: can become an indexed extraction, three selects and their compares.  Reverse kernel, T = 200,
// B = 64, 60 / 128 / 136 / 256 neurons: 49.7 / 70.6 / 107 / 125 us with ?:, 44.0 / 62.7 / 81.4 / 106 so; the forward
// kernel is the same either way.)
__device__ __forceinline__ float pick(uint32_t mask, float a, float b) {
  return __uint_as_float((mask & __float_as_uint(a)) | (~mask & __float_as_uint(b)));
}
// Two values rounded to bfloat16, the first in the low half.
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f2;
  typedef __attribute__((ext_vector_type(2))) __bf16 b2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, b2));
}

// KS: steps of 32 neurons of the contraction (the layer has at most 32 KS), and the most wavefronts.
template <int KS> struct RlifTile {
  static constexpr int CS = 4;                            // samples per workgroup
  static constexpr int XP = KS * 64 + 16;                 // bytes between the samples of an exchange tile
};

// The row tiles of a wavefront (two, or one) of the weight planes [row][k]: lane (c, q) holds row c, k 8q .. 8q+7.
template <int NP, int KS, int RT = 2> struct RlifWeights {
  bf16x8 f[NP][RT][KS];
  __device__ __forceinline__ void load(const uint16_t *Q, int ldq, long long plane, int w, int c, int q) {
    const rsrc_t r = make_rsrc(Q, (unsigned)(NP * plane * 2));
    const int rows = (int)(plane / ldq);
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const int row = 16 * (RT * w + i) + c, k = 32 * ks + 8 * q;
          f[p][i][ks] = __builtin_bit_cast(bf16x8, ld_b128(r, k < ldq && row < rows ? (int)(p * plane + (long long)row * ldq + k) * 2 : OOB, 0));
        }
  }
};

// Of the 32 x 16 sums of a wavefront, a lane (c, q) keeps tile c/8, rows 4q + 2 (c/4 % 2) + {0, 1}.
struct RlifLane {
  int c, q, smp, ti, e0, n;                              // column, row group, sample, tile, first row in the group, neuron
  __device__ __forceinline__ explicit RlifLane(int tid)
      : c(tid & 15), q((tid >> 4) & 3), smp(c & 3), ti(c >> 3), e0(2 * ((c >> 2) & 1)), n(32 * (tid >> 6) + 16 * ti + 4 * q + e0) {}
};

struct RlifLaneMasks : RlifLane {
  uint32_t mt, me;                                        // masks: ti, e0
  __device__ __forceinline__ explicit RlifLaneMasks(int tid) : RlifLane(tid), mt(ti ? ~0u : 0u), me(e0 ? ~0u : 0u) {
    asm("" : "+v"(mt), "+v"(me));                         // (values, not conditions)
  }
};

template <int NP, int KS>
__global__ __launch_bounds__(KS * 64) void rlif_tile_forward_kernel(const float *__restrict__ I, float *__restrict__ V,
                                                                    uint8_t *__restrict__ S, const uint16_t *__restrict__ QRf,
                                                                    int ldqr, long long qr_plane, int T, int B, int ld,
                                                                    const float *__restrict__ beta_v, float theta) {
  typedef RlifTile<KS> G;
  constexpr int PF = 6;                                   // steps of I in flight (4: 38.9 us, 8: 37.3)
  __shared__ __align__(16) char xs[2][G::CS * G::XP];
  const RlifLane L(threadIdx.x);
  const int b = blockIdx.x * G::CS + L.smp, row4 = B * ld * 4;
  const unsigned bytes = (unsigned)T * B * ld * 4u;
  const rsrc_t rI = make_rsrc(I, bytes), rV = make_rsrc(V, bytes), rS = make_rsrc(S, bytes / 4);
  RlifWeights<NP, KS> W;
  W.load(QRf, ldqr, qr_plane, threadIdx.x >> 6, L.c, L.q);
  const bool ok = b < B && L.n < ld;
  const int vo1 = ok ? b * ld + L.n : OOB, vo4 = ok ? vo1 * 4 : OOB;
  const int xo = L.smp * G::XP + L.n * 2, fo = L.smp * G::XP + 16 * L.q;
  float v[2] = {0.f, 0.f}, beta[2];                       // V_0 = 0
#pragma unroll
  for (int e = 0; e < 2; ++e) beta[e] = L.n + e < ld ? beta_v[L.n + e] : 0.f;
  u32x2 cur[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) cur[d] = ld_b64(rI, vo4, min(d, T - 1) * row4);
  for (int i = threadIdx.x; i < 2 * G::CS * G::XP / 4; i += blockDim.x) ((uint32_t *)xs)[i] = 0u;   // neurons beyond the last wavefront
  __syncthreads();

  auto step = [&](u32x2 &in, int t) {
    char *x = xs[t & 1];
    const uint32_t s0 = v[0] > theta ? 1u : 0u, s1 = v[1] > theta ? 1u : 0u;
    *(uint32_t *)(x + xo) = (s0 | (s1 << 16)) * 0x3F80u;
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    lds_barrier();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 sf = *(const bf16x8 *)(x + fo + 64 * ks);
#pragma unroll
      for (int p = NP - 1; p >= 0; --p)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.f[p][i][ks], sf, acc[i], 0, 0, 0);
    }
    st_b64(rV, vo4, t * row4, u32x2{__float_as_uint(v[0]), __float_as_uint(v[1])});
    st_b16(rS, vo1, t * (row4 >> 2), s0 | (s1 << 8));
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float h0 = L.e0 ? acc[0][2 + e] : acc[0][e], h1 = L.e0 ? acc[1][2 + e] : acc[1][e];
      v[e] = beta[e] * v[e] + __uint_as_float(in[e]) + (L.ti ? h1 : h0) - ((e ? s1 : s0) ? theta : 0.f);
    }
    in = ld_b64(rI, vo4, min(t + PF, T - 1) * row4);
  };
  int t = 0;
  for (; t + PF <= T; t += PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) step(cur[d], t + d);
  }
#pragma unroll
  for (int d = 0; d < PF; ++d)
    if (t + d < T) step(cur[d], t + d);
}

// g <- beta g + surr(V_t - theta) (dS_t - theta g + R g), dI_t = g before the update; g enters the product
// as bfloat16 planes, hi + lo with rounded weights (which is also how dI is stored), hi + mid + lo with
// fp32 weights.  db_part (optional): per sample, the sum over t of g_{t+1} V_t.
template <int NP, int SURR, int KS>
__global__ __launch_bounds__(KS * 64) void rlif_tile_reverse_kernel(const float *__restrict__ dS, const float *__restrict__ V,
                                                                    uint32_t *__restrict__ dI, const uint16_t *__restrict__ QRb,
                                                                    int ldqr, long long qr_plane, int T, int B, int ld,
                                                                    const float *__restrict__ beta_v, float theta, float slope,
                                                                    float *__restrict__ db_part) {
  typedef RlifTile<KS> G;
  constexpr int PF = NP == 1 ? 6 : 4;                     // steps of dS and V in flight (one plane: 4: 51.5 us, 8: 47.8)
  constexpr int GP = NP == 1 ? 2 : 3;                     // planes of g; column c holds plane c/8, or c/4 (the fourth: zeros)
  constexpr int XB = G::CS * G::XP;
  // The sigmoid's two exponentials and reciprocals come last in the step where the compiler is free, behind the
  // products; at 129 to 192 neurons they stand under the fragment reads instead (T = 200, B = 64, 130 / 144 / 160 neurons:
  // 76.3 / 76.5 / 83.3 us behind, 77.9 / 78.1 / 78.4 so; 192, six steps of the contraction: 99.4 and 91.6; at 60 and 250
  // neurons behind is faster, 49.5 against 55.2 and 113 against 117).
  constexpr bool EARLY = NP == 1 && SURR == 2 && (KS == 5 || KS == 6);
  __shared__ __align__(16) char xs[2][GP][XB];
  const RlifLaneMasks L(threadIdx.x);
  const int b = blockIdx.x * G::CS + L.smp, row4 = B * ld * 4;
  const unsigned bytes = (unsigned)T * B * ld * 4u;
  const rsrc_t rdS = make_rsrc(dS, bytes), rV = make_rsrc(V, bytes), rdI = make_rsrc(dI, bytes);
  RlifWeights<NP, KS> W;
  W.load(QRb, ldqr, qr_plane, threadIdx.x >> 6, L.c, L.q);
  const bool ok = b < B && L.n < ld;
  const int vo4 = ok ? (b * ld + L.n) * 4 : OOB;
  const int pl = NP == 1 ? L.c >> 3 : L.c >> 2;
  const int xo = L.smp * G::XP + L.n * 2, fo = min(pl, GP - 1) * XB + L.smp * G::XP + 16 * L.q;
  float gv[2] = {0.f, 0.f}, db[2] = {0.f, 0.f}, beta[2];  // g_T = 0
#pragma unroll
  for (int e = 0; e < 2; ++e) beta[e] = L.n + e < ld ? beta_v[L.n + e] : 0.f;
  u32x2 cds[PF], cv[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) {
    cds[d] = ld_b64(rdS, vo4, max(T - 1 - d, 0) * row4);
    cv[d] = ld_b64(rV, vo4, max(T - 1 - d, 0) * row4);
  }
  for (int i = threadIdx.x; i < 2 * GP * XB / 4; i += blockDim.x) ((uint32_t *)xs)[i] = 0u;
  __syncthreads();

  auto step = [&](u32x2 &ds, u32x2 &vv, int t) {
    char *x = (char *)xs[t & 1];
    u32x2 o;
    if (NP == 1) {
      const uint32_t hi = pk_bf16(gv[0], gv[1]);
      const uint32_t lo = pk_bf16(gv[0] - __uint_as_float(hi << 16), gv[1] - __uint_as_float(hi & 0xFFFF0000u));
      *(uint32_t *)(x + xo) = hi;
      *(uint32_t *)(x + XB + xo) = lo;
      o[0] = __builtin_amdgcn_perm(lo, hi, 0x05040100u);
      o[1] = __builtin_amdgcn_perm(lo, hi, 0x07060302u);
    } else {
      o[0] = __float_as_uint(gv[0]);
      o[1] = __float_as_uint(gv[1]);
#pragma unroll
      for (int k = 0; k < GP; ++k) *(uint32_t *)(x + k * XB + xo) = bf16_piece(gv[0], k) | (bf16_piece(gv[1], k) << 16);
    }
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    float sg[2], u[2];
    auto surrogates = [&] {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float vt = __uint_as_float(vv[e]);
        sg[e] = surr_rcp<SURR>(slope, vt - theta);
        u[e] = __uint_as_float(ds[e]) - theta * gv[e];
        db[e] += gv[e] * vt;
      }
    };
    lds_barrier();
    bf16x8 early[EARLY ? KS : 1];
    if constexpr (EARLY) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) early[ks] = *(const bf16x8 *)(x + fo + 64 * ks);
      __builtin_amdgcn_sched_barrier(0);
      surrogates();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 gf = EARLY ? early[EARLY ? ks : 0] : *(const bf16x8 *)(x + fo + 64 * ks);
      if (GP == 3 && pl == 3) gf = bf16x8{};
#pragma unroll
      for (int p = NP - 1; p >= 0; --p)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.f[p][i][ks], gf, acc[i], 0, 0, 0);
    }
    st_b64(rdI, vo4, t * row4, o);
    if (!EARLY) surrogates();
    ds = ld_b64(rdS, vo4, max(t - PF, 0) * row4);
    vv = ld_b64(rV, vo4, max(t - PF, 0) * row4);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      // the sums of the lane's own neuron: its column, and the columns that hold the sample's other planes
      float h0, h1, sum;
      if (NP == 1) {
        h0 = pick(L.me, acc[0][2 + e], acc[0][e]);
        h1 = pick(L.me, acc[1][2 + e], acc[1][e]);
        sum = pick(L.mt, h1, h0) + row_ror<8>(pick(L.mt, h0, h1));
      } else {
        // four planes in columns c, c + 4, c + 8, c + 12: every one of them adds the same four
        auto planes = [](float y) { y += row_ror<8>(y); return y + row_ror<4>(y); };
        const float p0 = planes(acc[0][e]), p1 = planes(acc[0][2 + e]), p2 = planes(acc[1][e]), p3 = planes(acc[1][2 + e]);
        h0 = L.e0 ? p1 : p0;
        h1 = L.e0 ? p3 : p2;
        sum = L.ti ? h1 : h0;
      }
      gv[e] = beta[e] * gv[e] + sg[e] * (u[e] + sum);
    }
  };
  int t = T - 1;
  for (; t - PF + 1 >= 0; t -= PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) step(cds[d], cv[d], t - d);
  }
#pragma unroll
  for (int d = 0; d < PF; ++d)
    if (t - d >= 0) step(cds[d], cv[d], t - d);
  if (db_part && ok) *(u32x2 *)(db_part + (size_t)b * ld + L.n) = u32x2{__float_as_uint(db[0]), __float_as_uint(db[1])};
}

// ---------------------------------------------------------------- sixteen samples
// Batches of many more tiles than compute units: a step's chain is hidden behind other workgroups then, and
// what counts is the instructions of all of them.  Sixteen samples fill the MFMA's columns, a wavefront holds 16
// neurons, a lane four of them: the fragments, the barrier and the bookkeeping of a step serve four
// times the samples.  (Figures at the rule in rlif_tile.hip.)
template <int NP, int KS>
__global__ __launch_bounds__(KS * 128) void rlif_tile16_forward_kernel(const float *__restrict__ I, float *__restrict__ V,
                                                                       uint8_t *__restrict__ S, const uint16_t *__restrict__ QRf,
                                                                       int ldqr, long long qr_plane, int T, int B, int ld,
                                                                       const float *__restrict__ beta_v, float theta) {
  constexpr int XP = RlifTile<KS>::XP, PF = 4;
  constexpr int VP = KS * 32 + 4, SP = KS * 32 + 16;      // V and S leave as the tile lies in memory, one block, through LDS:
  __shared__ __align__(16) char xs[2][16 * XP];           // rows of 64 bytes per sample and wavefront took 80 us instead of 52
  __shared__ __align__(16) float vs[2][16 * VP];          // (128 neurons, B = 8192, T = 32)
  __shared__ __align__(16) uint8_t ss[2][16 * SP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, q = lane >> 4, n = 16 * w + 4 * q;
  const int b = blockIdx.x * 16 + c, row4 = B * ld * 4;
  const unsigned bytes = (unsigned)T * B * ld * 4u;
  const rsrc_t rI = make_rsrc(I, bytes), rV = make_rsrc(V, bytes), rS = make_rsrc(S, bytes / 4);
  RlifWeights<NP, KS, 1> W;
  W.load(QRf, ldqr, qr_plane, w, c, q);
  const bool ok = b < B && n < ld;
  const int vo4 = ok ? (b * ld + n) * 4 : OOB;
  const int xo = c * XP + n * 2, fo = c * XP + 16 * q;
  // piece i of the block: four potentials, or eight spikes, of a sample
  const int vi = 4 * threadIdx.x, vr = vi / ld, si = 8 * threadIdx.x, sr = si / ld, b0 = blockIdx.x * 16;
  const int vso = vr < 16 && b0 + vr < B ? (b0 * ld + vi) * 4 : OOB, sso = sr < 16 && b0 + sr < B ? b0 * ld + si : OOB;
  const int vsl = min(vr, 15) * VP + vi - vr * ld, ssl = min(sr, 15) * SP + si - sr * ld;
  float v[4] = {0.f, 0.f, 0.f, 0.f}, beta[4];             // V_0 = 0
#pragma unroll
  for (int e = 0; e < 4; ++e) beta[e] = n + e < ld ? beta_v[n + e] : 0.f;
  u32x4 cur[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) cur[d] = ld_b128(rI, vo4, min(d, T - 1) * row4);
  for (int i = threadIdx.x; i < 2 * 16 * XP / 4; i += blockDim.x) ((uint32_t *)xs)[i] = 0u;   // neurons beyond the last wavefront
  __syncthreads();

  auto step = [&](u32x4 &in, int t) {
    char *x = xs[t & 1];
    uint32_t s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = v[e] > theta ? 1u : 0u;
    *(u32x2 *)(x + xo) = u32x2{(s[0] | (s[1] << 16)) * 0x3F80u, (s[2] | (s[3] << 16)) * 0x3F80u};
    *(f32x4 *)(vs[t & 1] + c * VP + n) = f32x4{v[0], v[1], v[2], v[3]};
    *(uint32_t *)(ss[t & 1] + c * SP + n) = s[0] | (s[1] << 8) | (s[2] << 16) | (s[3] << 24);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    lds_barrier();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 sf = *(const bf16x8 *)(x + fo + 64 * ks);
#pragma unroll
      for (int p = NP - 1; p >= 0; --p) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.f[p][0][ks], sf, acc, 0, 0, 0);
    }
    st_b128(rV, vso, t * row4, *(const u32x4 *)(vs[t & 1] + vsl));
    st_b64(rS, sso, t * (row4 >> 2), *(const u32x2 *)(ss[t & 1] + ssl));
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = beta[e] * v[e] + __uint_as_float(in[e]) + acc[e] - (s[e] ? theta : 0.f);
    in = ld_b128(rI, vo4, min(t + PF, T - 1) * row4);
  };
  int t = 0;
  for (; t + PF <= T; t += PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) step(cur[d], t + d);
  }
#pragma unroll
  for (int d = 0; d < PF; ++d)
    if (t + d < T) step(cur[d], t + d);
}

template <int NP, int SURR, int KS>
__global__ __launch_bounds__(KS * 128) void rlif_tile16_reverse_kernel(const float *__restrict__ dS, const float *__restrict__ V,
                                                                       uint32_t *__restrict__ dI, const uint16_t *__restrict__ QRb,
                                                                       int ldqr, long long qr_plane, int T, int B, int ld,
                                                                       const float *__restrict__ beta_v, float theta, float slope,
                                                                       float *__restrict__ db_part) {
  constexpr int XP = RlifTile<KS>::XP, PF = 3;
  constexpr int GP = NP == 1 ? 2 : 3, XB = 16 * XP;
  __shared__ __align__(16) char xs[2][GP][XB];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, q = lane >> 4, n = 16 * w + 4 * q;
  const int b = blockIdx.x * 16 + c, row4 = B * ld * 4;
  const unsigned bytes = (unsigned)T * B * ld * 4u;
  const rsrc_t rdS = make_rsrc(dS, bytes), rV = make_rsrc(V, bytes), rdI = make_rsrc(dI, bytes);
  RlifWeights<NP, KS, 1> W;
  W.load(QRb, ldqr, qr_plane, w, c, q);
  const bool ok = b < B && n < ld;
  const int vo4 = ok ? (b * ld + n) * 4 : OOB;
  const int xo = c * XP + n * 2, fo = c * XP + 16 * q;
  float gv[4] = {0.f, 0.f, 0.f, 0.f}, db[4] = {0.f, 0.f, 0.f, 0.f}, beta[4];   // g_T = 0
#pragma unroll
  for (int e = 0; e < 4; ++e) beta[e] = n + e < ld ? beta_v[n + e] : 0.f;
  u32x4 cds[PF], cv[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) {
    cds[d] = ld_b128(rdS, vo4, max(T - 1 - d, 0) * row4);
    cv[d] = ld_b128(rV, vo4, max(T - 1 - d, 0) * row4);
  }
  for (int i = threadIdx.x; i < 2 * GP * XB / 4; i += blockDim.x) ((uint32_t *)xs)[i] = 0u;
  __syncthreads();

  auto step = [&](u32x4 &ds, u32x4 &vv, int t) {
    char *x = (char *)xs[t & 1];
    u32x4 o;
    if (NP == 1) {
      u32x2 hi, lo;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        hi[p] = pk_bf16(gv[2 * p], gv[2 * p + 1]);
        lo[p] = pk_bf16(gv[2 * p] - __uint_as_float(hi[p] << 16), gv[2 * p + 1] - __uint_as_float(hi[p] & 0xFFFF0000u));
        o[2 * p] = __builtin_amdgcn_perm(lo[p], hi[p], 0x05040100u);
        o[2 * p + 1] = __builtin_amdgcn_perm(lo[p], hi[p], 0x07060302u);
      }
      *(u32x2 *)(x + xo) = hi;
      *(u32x2 *)(x + XB + xo) = lo;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(gv[e]);
#pragma unroll
      for (int k = 0; k < GP; ++k)
        *(u32x2 *)(x + k * XB + xo) = u32x2{bf16_piece(gv[0], k) | (bf16_piece(gv[1], k) << 16), bf16_piece(gv[2], k) | (bf16_piece(gv[3], k) << 16)};
    }
    f32x4 acc[GP] = {};                                   // a sum per plane of g
    lds_barrier();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int k = 0; k < GP; ++k) {
        const bf16x8 gf = *(const bf16x8 *)(x + k * XB + fo + 64 * ks);
#pragma unroll
        for (int p = NP - 1; p >= 0; --p) acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.f[p][0][ks], gf, acc[k], 0, 0, 0);
      }
    st_b128(rdI, vo4, t * row4, o);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float vt = __uint_as_float(vv[e]);
      const float sg = surr_rcp<SURR>(slope, vt - theta), u = __uint_as_float(ds[e]) - theta * gv[e];
      const float sum = NP == 1 ? acc[0][e] + acc[1][e] : (acc[0][e] + acc[GP - 1][e]) + acc[1][e];
      db[e] += gv[e] * vt;
      gv[e] = beta[e] * gv[e] + sg * (u + sum);
    }
    ds = ld_b128(rdS, vo4, max(t - PF, 0) * row4);
    vv = ld_b128(rV, vo4, max(t - PF, 0) * row4);
  };
  int t = T - 1;
  for (; t - PF + 1 >= 0; t -= PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) step(cds[d], cv[d], t - d);
  }
#pragma unroll
  for (int d = 0; d < PF; ++d)
    if (t - d >= 0) step(cds[d], cv[d], t - d);
  if (db_part && ok)
    *(u32x4 *)(db_part + (size_t)b * ld + n) = u32x4{__float_as_uint(db[0]), __float_as_uint(db[1]), __float_as_uint(db[2]), __float_as_uint(db[3])};
}

// Whether a recurrent layer's rows fit a workgroup of these kernels.
static bool rlif_tile_fits(int ld) { return ld <= 256; }

hipError_t rlif_tile_forward(hipStream_t st, bool fp32, int T, int B, int ld, const float *I, float *V, uint8_t *S,
                             const uint16_t *QRf, int ldqr, long long qr_plane, const float *beta, float theta);
hipError_t rlif_tile_reverse(hipStream_t st, bool fp32, int T, int B, int ld, const float *dS, const float *V, uint32_t *dI,
                             const uint16_t *QRb, int ldqr, long long qr_plane, const float *beta, float theta, int surrogate,
                             float slope, float *db_part);

}  // namespace snn
