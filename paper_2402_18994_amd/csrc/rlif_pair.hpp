// A recurrent LIF layer and the recurrent layer above it, both of few neurons, in one launch per
// direction: their time loops run side by side on one workgroup of four samples, the upper layer one step
// behind (forward) or ahead (reverse).
//
// A layer's loop alone (rlif_tile.hpp) is a dependent chain per step that leaves most of a compute unit's
// issue slots, and three of four compute units, idle.  Here the workgroup has wavefronts for both layers, one
// barrier serves a step of each, and the product between the layers (I = S W forward, dS = dI W^T in reverse)
// comes from the exchange tile that the one layer writes for its own recurrence: no product launch, no
// currents or spike gradients through memory.  Its MFMAs stand between the barrier and the arrival of the
// layer's own fragments, which that layer would wait for anyway (the fragments between the layers were read
// a step earlier).
//
// Exchange, 32-neuron wavefronts, planes of g in the MFMA's columns: as in rlif_tile.hpp.
#pragma once
#include "rlif_tile.hpp"

namespace snn {

struct RlifPairArgs {
  struct Layer {
    const float *X;        // forward, lower: I [T*B][ld]; reverse, upper: dS
    float *V;
    uint8_t *S;
    uint32_t *dI;
    const uint16_t *R;     // forward [to][from], reverse [from][to]
    int ldr;
    long long r_plane;
    const float *beta_v;
    float *db_part;        // reverse, optional
    int ld;
  } lo, up;
  const uint16_t *W;       // between the layers: forward W^T [upper][lower], reverse W [lower][upper]
  int ldw;
  long long w_plane;
  int T, B;
  float theta, slope;
  int surrogate;
};

// Rounded weights, at most 192 neurons each, eight wavefronts together (the weights of two matrices take up to
// 96 registers of each).
inline bool rlif_pair_fits(int ld_lower, int ld_upper) {
  return ld_lower <= 192 && ld_upper <= 192 && (ld_lower + 31) / 32 + (ld_upper + 31) / 32 <= 8;
}
hipError_t rlif_pair_forward(hipStream_t st, const RlifPairArgs &a);
hipError_t rlif_pair_reverse(hipStream_t st, const RlifPairArgs &a);

template <int KS>
__device__ __forceinline__ void pair_fragments(bf16x8 (&f)[KS], const char *x) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) f[ks] = *(const bf16x8 *)(x + 64 * ks);
}
template <int KS>
__device__ __forceinline__ void pair_product(f32x4 (&acc)[2], const RlifWeights<1, KS> &W, const bf16x8 (&f)[KS]) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.f[0][i][ks], f[ks], acc[i], 0, 0, 0);
}

// K1, K2: steps of 32 neurons of the lower and the upper layer.
template <int K1, int K2>
__global__ __launch_bounds__(512) void rlif_pair_forward_kernel(const RlifPairArgs a) {
  constexpr int X1 = RlifTile<K1>::XP, X2 = RlifTile<K2>::XP, CS = 4;
  __shared__ __align__(16) char xs1[2][CS * X1], xs2[2][CS * X2];
  const int T = a.T, B = a.B, nw1 = (a.lo.ld + 31) / 32;
  for (int i = threadIdx.x; i < 2 * CS * X1 / 4; i += blockDim.x) ((uint32_t *)xs1)[i] = 0u;
  for (int i = threadIdx.x; i < 2 * CS * X2 / 4; i += blockDim.x) ((uint32_t *)xs2)[i] = 0u;
  __syncthreads();
  const bool lower = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) < nw1;   // (a wavefront is one layer's)
  const RlifPairArgs::Layer &y = lower ? a.lo : a.up;
  const RlifLane L(lower ? threadIdx.x : threadIdx.x - 64 * nw1);
  const int w = L.n >> 5, ld = y.ld, b = blockIdx.x * CS + L.smp, row4 = B * ld * 4;
  const unsigned bytes = (unsigned)T * B * ld * 4u;
  const rsrc_t rV = make_rsrc(y.V, bytes), rS = make_rsrc(y.S, bytes / 4);
  const bool ok = b < B && L.n < ld;
  const int vo1 = ok ? b * ld + L.n : OOB, vo4 = ok ? vo1 * 4 : OOB;
  const float theta = a.theta;
  float v[2] = {0.f, 0.f}, beta[2];                       // V_0 = 0
#pragma unroll
  for (int e = 0; e < 2; ++e) beta[e] = L.n + e < ld ? y.beta_v[L.n + e] : 0.f;
  uint32_t s0, s1;
  auto spikes = [&](char *x) {
    s0 = v[0] > theta ? 1u : 0u;
    s1 = v[1] > theta ? 1u : 0u;
    *(uint32_t *)x = (s0 | (s1 << 16)) * 0x3F80u;
  };
  auto store = [&](int t) {
    st_b64(rV, vo4, t * row4, u32x2{__float_as_uint(v[0]), __float_as_uint(v[1])});
    st_b16(rS, vo1, t * (row4 >> 2), s0 | (s1 << 8));
  };
  auto update = [&](const f32x4 (&acc)[2], float i0, float i1) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float h0 = L.e0 ? acc[0][2 + e] : acc[0][e], h1 = L.e0 ? acc[1][2 + e] : acc[1][e];
      v[e] = beta[e] * v[e] + (e ? i1 : i0) + (L.ti ? h1 : h0) - ((e ? s1 : s0) ? theta : 0.f);
    }
  };
  if (lower) {
    constexpr int PF = 6;                                 // steps of I in flight
    const rsrc_t rI = make_rsrc(y.X, bytes);
    RlifWeights<1, K1> R;
    R.load(y.R, y.ldr, y.r_plane, w, L.c, L.q);
    const int xo = L.smp * X1 + L.n * 2, fo = L.smp * X1 + 16 * L.q;
    u32x2 cur[PF];
#pragma unroll
    for (int d = 0; d < PF; ++d) cur[d] = ld_b64(rI, vo4, min(d, T - 1) * row4);
    auto step = [&](u32x2 &in, int t) {
      char *x = xs1[t & 1];
      spikes(x + xo);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K1];
      pair_fragments<K1>(f, x + fo);
      pair_product<K1>(acc, R, f);
      store(t);
      update(acc, __uint_as_float(in[0]), __uint_as_float(in[1]));
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
    lds_barrier();                                        // the upper layer's last step
  } else {
    RlifWeights<1, K1> W;                                 // rows: upper neurons
    W.load(a.W, a.ldw, a.w_plane, w, L.c, L.q);
    RlifWeights<1, K2> R;
    R.load(y.R, y.ldr, y.r_plane, w, L.c, L.q);
    const int xo = L.smp * X2 + L.n * 2, fo = L.smp * X2 + 16 * L.q, f1o = L.smp * X1 + 16 * L.q;
    bf16x8 f1[K1];                                        // the lower layer's spikes of the step
    lds_barrier();                                        // the lower layer's step 0
    pair_fragments<K1>(f1, xs1[0] + f1o);
    auto step = [&](int t) {                              // beside the lower layer's step t + 1
      char *x = xs2[(t + 1) & 1];
      spikes(x + xo);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K2];
      pair_fragments<K2>(f, x + fo);
      __builtin_amdgcn_sched_barrier(0);
      pair_product<K1>(acc, W, f1);
      __builtin_amdgcn_sched_barrier(0);
      pair_fragments<K1>(f1, xs1[(t + 1) & 1] + f1o);     // (after the last step: not used)
      pair_product<K2>(acc, R, f);
      store(t);
      update(acc, 0.f, 0.f);
    };
    int t = 0;
    for (; t + 2 <= T; t += 2) { step(t); step(t + 1); }
    if (t < T) step(t);
  }
}

template <int SURR> __device__ __forceinline__ void pair_surrogate(float (&sg)[2], float slope, float theta, u32x2 vv) {
#pragma unroll
  for (int e = 0; e < 2; ++e) sg[e] = surr_rcp<SURR>(slope, __uint_as_float(vv[e]) - theta);
}

template <int K1, int K2>
__global__ __launch_bounds__(512) void rlif_pair_reverse_kernel(const RlifPairArgs a) {
  constexpr int X1 = RlifTile<K1>::XP, X2 = RlifTile<K2>::XP, CS = 4, B1 = CS * X1, B2 = CS * X2, PF = 6;
  __shared__ __align__(16) char xs1[2][2][B1], xs2[2][2][B2];   // [parity][hi, lo]
  const int T = a.T, B = a.B, nw1 = (a.lo.ld + 31) / 32;
  for (int i = threadIdx.x; i < 4 * B1 / 4; i += blockDim.x) ((uint32_t *)xs1)[i] = 0u;
  for (int i = threadIdx.x; i < 4 * B2 / 4; i += blockDim.x) ((uint32_t *)xs2)[i] = 0u;
  __syncthreads();
  const bool lower = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) < nw1;   // (a wavefront is one layer's)
  const RlifPairArgs::Layer &y = lower ? a.lo : a.up;
  const RlifLane L(lower ? threadIdx.x : threadIdx.x - 64 * nw1);
  const int w = L.n >> 5, ld = y.ld, b = blockIdx.x * CS + L.smp, row4 = B * ld * 4;
  const unsigned bytes = (unsigned)T * B * ld * 4u;
  const rsrc_t rV = make_rsrc(y.V, bytes), rdI = make_rsrc(y.dI, bytes);
  const bool ok = b < B && L.n < ld;
  const int vo4 = ok ? (b * ld + L.n) * 4 : OOB, pl = L.c >> 3;
  const float theta = a.theta, slope = a.slope;
  float gv[2] = {0.f, 0.f}, db[2] = {0.f, 0.f}, beta[2], sg[2];   // g_T = 0
#pragma unroll
  for (int e = 0; e < 2; ++e) beta[e] = L.n + e < ld ? y.beta_v[L.n + e] : 0.f;
  u32x2 o;
  auto planes = [&](char *x, int lo_plane) {              // g into the exchange tile, and as it is stored
    const uint32_t hi = pk_bf16(gv[0], gv[1]);
    const uint32_t lo = pk_bf16(gv[0] - __uint_as_float(hi << 16), gv[1] - __uint_as_float(hi & 0xFFFF0000u));
    *(uint32_t *)x = hi;
    *(uint32_t *)(x + lo_plane) = lo;
    o[0] = __builtin_amdgcn_perm(lo, hi, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(lo, hi, 0x07060302u);
  };
  auto surrogates = [&](u32x2 vv) {                       // (uniform; off the chain of the step)
    switch (a.surrogate) {
      case 0: pair_surrogate<0>(sg, slope, theta, vv); break;
      case 1: pair_surrogate<1>(sg, slope, theta, vv); break;
      case 2: pair_surrogate<2>(sg, slope, theta, vv); break;
      case 3: pair_surrogate<3>(sg, slope, theta, vv); break;
      case 4: pair_surrogate<4>(sg, slope, theta, vv); break;
      default: pair_surrogate<5>(sg, slope, theta, vv); break;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) db[e] += gv[e] * __uint_as_float(vv[e]);
  };
  auto update = [&](const f32x4 (&acc)[2], float d0, float d1) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      // the sums of the lane's own neuron: its column, and the column that holds the sample's other plane
      const float h0 = L.e0 ? acc[0][2 + e] : acc[0][e], h1 = L.e0 ? acc[1][2 + e] : acc[1][e];
      const float sum = (L.ti ? h1 : h0) + row_ror<8>(L.ti ? h0 : h1);
      gv[e] = beta[e] * gv[e] + sg[e] * ((e ? d1 : d0) - theta * gv[e] + sum);
    }
  };
  u32x2 cv[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) cv[d] = ld_b64(rV, vo4, max(T - 1 - d, 0) * row4);
  if (lower) {
    RlifWeights<1, K2> W;                                 // rows: lower neurons
    W.load(a.W, a.ldw, a.w_plane, w, L.c, L.q);
    RlifWeights<1, K1> R;
    R.load(y.R, y.ldr, y.r_plane, w, L.c, L.q);
    const int xo = L.smp * X1 + L.n * 2, fo = pl * B1 + L.smp * X1 + 16 * L.q, f2o = pl * B2 + L.smp * X2 + 16 * L.q;
    bf16x8 f2[K2];                                        // dI of the upper layer at the step
    lds_barrier();                                        // the upper layer's step T - 1
    pair_fragments<K2>(f2, xs2[(T - 1) & 1][0] + f2o);
    auto step = [&](u32x2 &vv, int t) {                   // beside the upper layer's step t - 1
      char *x = (char *)xs1[t & 1];
      planes(x + xo, B1);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K1];
      pair_fragments<K1>(f, x + fo);
      __builtin_amdgcn_sched_barrier(0);
      pair_product<K2>(acc, W, f2);
      __builtin_amdgcn_sched_barrier(0);
      pair_fragments<K2>(f2, xs2[(t + 1) & 1][0] + f2o);  // (of step t - 1; after step 0: not used)
      pair_product<K1>(acc, R, f);
      st_b64(rdI, vo4, t * row4, o);
      surrogates(vv);
      vv = ld_b64(rV, vo4, max(t - PF, 0) * row4);
      update(acc, 0.f, 0.f);
    };
    int t = T - 1;
    for (; t - PF + 1 >= 0; t -= PF) {
#pragma unroll
      for (int d = 0; d < PF; ++d) step(cv[d], t - d);
    }
#pragma unroll
    for (int d = 0; d < PF; ++d)
      if (t - d >= 0) step(cv[d], t - d);
  } else {
    const rsrc_t rdS = make_rsrc(y.X, bytes);
    RlifWeights<1, K2> R;
    R.load(y.R, y.ldr, y.r_plane, w, L.c, L.q);
    const int xo = L.smp * X2 + L.n * 2, fo = pl * B2 + L.smp * X2 + 16 * L.q;
    u32x2 cds[PF];
#pragma unroll
    for (int d = 0; d < PF; ++d) cds[d] = ld_b64(rdS, vo4, max(T - 1 - d, 0) * row4);
    auto step = [&](u32x2 &ds, u32x2 &vv, int t) {
      char *x = (char *)xs2[t & 1];
      planes(x + xo, B2);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K2];
      pair_fragments<K2>(f, x + fo);
      pair_product<K2>(acc, R, f);
      st_b64(rdI, vo4, t * row4, o);
      surrogates(vv);
      const float d0 = __uint_as_float(ds[0]), d1 = __uint_as_float(ds[1]);
      ds = ld_b64(rdS, vo4, max(t - PF, 0) * row4);
      vv = ld_b64(rV, vo4, max(t - PF, 0) * row4);
      update(acc, d0, d1);
    };
    int t = T - 1;
    for (; t - PF + 1 >= 0; t -= PF) {
#pragma unroll
      for (int d = 0; d < PF; ++d) step(cds[d], cv[d], t - d);
    }
#pragma unroll
    for (int d = 0; d < PF; ++d)
      if (t - d >= 0) step(cds[d], cv[d], t - d);
    lds_barrier();                                        // the lower layer's step 0
  }
  if (y.db_part && ok) *(u32x2 *)(y.db_part + (size_t)b * ld + L.n) = u32x2{__float_as_uint(db[0]), __float_as_uint(db[1])};
}

}  // namespace snn
