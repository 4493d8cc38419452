// A recurrent LIF layer and the recurrent layer above it, both of few neurons, in one launch per
// direction: their time loops run side by side on one workgroup of four samples, the upper layer one step
// behind (forward) or ahead (reverse).
//
// A layer's loop alone (rlif_tile.hpp) is a dependent chain per step that leaves most of a compute unit's
// issue slots, and three of four compute units, idle.  Here the workgroup has wavefronts for both layers, one
// barrier serves a step of each, and the product between the layers (I = S W forward, dS = dI W^T in reverse)
// is taken by wavefronts of its own from the exchange tile that the one layer writes for its own recurrence
// and handed to the other through LDS, in time for that layer's same step an iteration later: no product
// launch, no currents or spike gradients through memory, and no step's chain is longer than its own layer's.
// 700-128-128-20, T = 128, B = 256, both layers: forward 69 us in two launches and 6.5 for the product between
// them, 51 so (56 with that product on the upper layer's wavefronts); reverse 96 and 8, 64 so (83).
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

// Rounded weights, at most 192 neurons each, sixteen wavefronts with those between the layers.
inline bool rlif_pair_fits(int ld_lower, int ld_upper) {
  const int lo = (ld_lower + 31) / 32, up = (ld_upper + 31) / 32;
  return ld_lower <= 192 && ld_upper <= 192 && lo + up + (lo > up ? lo : up) <= 16;
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

// Wavefronts of a workgroup, in this order: the lower layer's, those of the product between the layers (one
// per 32 neurons of the layer that receives it), the upper layer's.
struct PairRole {
  int nw1, mid, wave;                                     // wavefronts of the first two kinds; this one
  __device__ __forceinline__ PairRole(int ld_lower, int ld_receiver)
      : nw1((ld_lower + 31) / 32), mid((ld_receiver + 31) / 32), wave(__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) {}
  __device__ __forceinline__ bool lower() const { return wave < nw1; }
  __device__ __forceinline__ bool between() const { return wave >= nw1 && wave < nw1 + mid; }
  __device__ __forceinline__ int thread() const { return threadIdx.x - 64 * (lower() ? 0 : between() ? nw1 : nw1 + mid); }
};

// K1, K2: steps of 32 neurons of the lower and the upper layer.
template <int K1, int K2>
__global__ __launch_bounds__(1024) void rlif_pair_forward_kernel(const RlifPairArgs a) {
  constexpr int X1 = RlifTile<K1>::XP, X2 = RlifTile<K2>::XP, CS = 4, IP = K2 * 32 + 4;
  __shared__ __align__(16) char xs1[2][CS * X1], xs2[2][CS * X2];
  __shared__ __align__(16) float between[2][CS * IP];     // the upper layer's currents, by parity of the step
  const int T = a.T, B = a.B;
  for (int i = threadIdx.x; i < 2 * CS * X1 / 4; i += blockDim.x) ((uint32_t *)xs1)[i] = 0u;
  for (int i = threadIdx.x; i < 2 * CS * X2 / 4; i += blockDim.x) ((uint32_t *)xs2)[i] = 0u;
  __syncthreads();
  const PairRole role(a.lo.ld, a.up.ld);
  const RlifPairArgs::Layer &y = role.lower() ? a.lo : a.up;
  const RlifLaneMasks L(role.thread());
  const int w = L.n >> 5, ld = y.ld, b = blockIdx.x * CS + L.smp, row4 = B * ld * 4;
  const int f1o = L.smp * X1 + 16 * L.q, f2o = L.smp * X2 + 16 * L.q, io = L.smp * IP + L.n;
  auto mine = [&](const f32x4 (&acc)[2], int e) {         // of the sums, those of the lane's own neuron
    return pick(L.mt, pick(L.me, acc[1][2 + e], acc[1][e]), pick(L.me, acc[0][2 + e], acc[0][e]));
  };
  if (role.between()) {
    RlifWeights<1, K1> W;                                 // rows: upper neurons
    W.load(a.W, a.ldw, a.w_plane, w, L.c, L.q);
    for (int t = 0; t < T; ++t) {
      f32x4 acc[2] = {};
      lds_barrier();                                      // the lower layer's spikes of step t
      bf16x8 f[K1];
      pair_fragments<K1>(f, xs1[t & 1] + f1o);
      __builtin_amdgcn_sched_barrier(0);                  // (all reads first)
      pair_product<K1>(acc, W, f);
      *(u32x2 *)(between[t & 1] + io) = u32x2{__float_as_uint(mine(acc, 0)), __float_as_uint(mine(acc, 1))};
    }
    lds_barrier();
    return;
  }
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
    *(uint32_t *)x = (v[0] > theta ? 0x3F80u : 0u) | (v[1] > theta ? 0x3F800000u : 0u);
  };
  auto store = [&](int t) {
    st_b64(rV, vo4, t * row4, u32x2{__float_as_uint(v[0]), __float_as_uint(v[1])});
    st_b16(rS, vo1, t * (row4 >> 2), s0 | (s1 << 8));
  };
  auto update = [&](const f32x4 (&acc)[2], u32x2 in) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
      v[e] = beta[e] * v[e] + __uint_as_float(in[e]) + mine(acc, e) - ((e ? s1 : s0) ? theta : 0.f);
  };
  if (role.lower()) {
    constexpr int PF = 6;                                 // steps of I in flight
    const rsrc_t rI = make_rsrc(y.X, bytes);
    RlifWeights<1, K1> R;
    R.load(y.R, y.ldr, y.r_plane, w, L.c, L.q);
    const int xo = L.smp * X1 + L.n * 2;
    u32x2 cur[PF];
#pragma unroll
    for (int d = 0; d < PF; ++d) cur[d] = ld_b64(rI, vo4, min(d, T - 1) * row4);
    auto step = [&](u32x2 &in, int t) {
      spikes(xs1[t & 1] + xo);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K1];
      pair_fragments<K1>(f, xs1[t & 1] + f1o);
      __builtin_amdgcn_sched_barrier(0);
      pair_product<K1>(acc, R, f);
      store(t);
      update(acc, in);
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
    RlifWeights<1, K2> R;
    R.load(y.R, y.ldr, y.r_plane, w, L.c, L.q);
    const int xo = L.smp * X2 + L.n * 2;
    lds_barrier();                                        // the lower layer's step 0
    auto step = [&](int t) {                              // beside the lower layer's step t + 1
      spikes(xs2[t & 1] + xo);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K2];
      pair_fragments<K2>(f, xs2[t & 1] + f2o);
      const u32x2 in = *(const u32x2 *)(between[t & 1] + io);
      __builtin_amdgcn_sched_barrier(0);
      pair_product<K2>(acc, R, f);
      store(t);
      update(acc, in);
    };
    int t = 0;
    for (; t + 2 <= T; t += 2) { step(t); step(t + 1); }
    if (t < T) step(t);
  }
}

// Columns of the MFMA: the samples' hi planes of g, twice the lo planes' (see RlifLane, rlif_tile_reverse_kernel).
template <int SURR, int K1, int K2>
__global__ __launch_bounds__(1024) void rlif_pair_reverse_kernel(const RlifPairArgs a) {
  constexpr int X1 = RlifTile<K1>::XP, X2 = RlifTile<K2>::XP, CS = 4, B1 = CS * X1, B2 = CS * X2, IP = K1 * 32 + 4;
  constexpr int PF = 6;                                   // steps of V (and dS) in flight
  __shared__ __align__(16) char xs1[2][2][B1], xs2[2][2][B2];   // [parity][hi, lo]
  __shared__ __align__(16) float between[2][CS * IP];     // the lower layer's dS, by parity of the step
  const int T = a.T, B = a.B;
  for (int i = threadIdx.x; i < 4 * B1 / 4; i += blockDim.x) ((uint32_t *)xs1)[i] = 0u;
  for (int i = threadIdx.x; i < 4 * B2 / 4; i += blockDim.x) ((uint32_t *)xs2)[i] = 0u;
  __syncthreads();
  const PairRole role(a.lo.ld, a.lo.ld);
  const RlifPairArgs::Layer &y = role.lower() || role.between() ? a.lo : a.up;
  const RlifLaneMasks L(role.thread());
  const int w = L.n >> 5, ld = y.ld, b = blockIdx.x * CS + L.smp, row4 = B * ld * 4, pl = L.c >> 3;
  const int f1o = pl * B1 + L.smp * X1 + 16 * L.q, f2o = pl * B2 + L.smp * X2 + 16 * L.q, io = L.smp * IP + L.n;
  auto mine = [&](const f32x4 (&acc)[2], int e) {         // the lane's column, and the one that holds the sample's other plane
    const float h0 = pick(L.me, acc[0][2 + e], acc[0][e]), h1 = pick(L.me, acc[1][2 + e], acc[1][e]);
    return pick(L.mt, h1, h0) + row_ror<8>(pick(L.mt, h0, h1));
  };
  if (role.between()) {
    RlifWeights<1, K2> W;                                 // rows: lower neurons
    W.load(a.W, a.ldw, a.w_plane, w, L.c, L.q);
    for (int t = T - 1; t >= 0; --t) {
      f32x4 acc[2] = {};
      lds_barrier();                                      // the upper layer's g of step t
      bf16x8 f[K2];
      pair_fragments<K2>(f, xs2[t & 1][0] + f2o);
      __builtin_amdgcn_sched_barrier(0);
      pair_product<K2>(acc, W, f);
      *(u32x2 *)(between[t & 1] + io) = u32x2{__float_as_uint(mine(acc, 0)), __float_as_uint(mine(acc, 1))};
    }
    lds_barrier();
    return;
  }
  const unsigned bytes = (unsigned)T * B * ld * 4u;
  const rsrc_t rV = make_rsrc(y.V, bytes), rdI = make_rsrc(y.dI, bytes);
  const bool ok = b < B && L.n < ld;
  const int vo4 = ok ? (b * ld + L.n) * 4 : OOB;
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
  auto surrogates = [&](u32x2 vv) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      sg[e] = surr_rcp<SURR>(slope, __uint_as_float(vv[e]) - theta);
      db[e] += gv[e] * __uint_as_float(vv[e]);
    }
  };
  auto update = [&](const f32x4 (&acc)[2], u32x2 ds) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
      gv[e] = beta[e] * gv[e] + sg[e] * (__uint_as_float(ds[e]) - theta * gv[e] + mine(acc, e));
  };
  u32x2 cv[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) cv[d] = ld_b64(rV, vo4, max(T - 1 - d, 0) * row4);
  if (role.lower()) {
    RlifWeights<1, K1> R;
    R.load(y.R, y.ldr, y.r_plane, w, L.c, L.q);
    const int xo = L.smp * X1 + L.n * 2;
    lds_barrier();                                        // the upper layer's step T - 1
    auto step = [&](u32x2 &vv, int t) {                   // beside the upper layer's step t - 1
      planes((char *)xs1[t & 1] + xo, B1);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K1];
      pair_fragments<K1>(f, xs1[t & 1][0] + f1o);
      const u32x2 ds = *(const u32x2 *)(between[t & 1] + io);
      __builtin_amdgcn_sched_barrier(0);
      pair_product<K1>(acc, R, f);
      st_b64(rdI, vo4, t * row4, o);
      surrogates(vv);
      vv = ld_b64(rV, vo4, max(t - PF, 0) * row4);
      update(acc, ds);
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
    const int xo = L.smp * X2 + L.n * 2;
    u32x2 cds[PF];
#pragma unroll
    for (int d = 0; d < PF; ++d) cds[d] = ld_b64(rdS, vo4, max(T - 1 - d, 0) * row4);
    auto step = [&](u32x2 &ds, u32x2 &vv, int t) {
      planes((char *)xs2[t & 1] + xo, B2);
      f32x4 acc[2] = {};
      lds_barrier();
      bf16x8 f[K2];
      pair_fragments<K2>(f, xs2[t & 1][0] + f2o);
      __builtin_amdgcn_sched_barrier(0);
      pair_product<K2>(acc, R, f);
      st_b64(rdI, vo4, t * row4, o);
      surrogates(vv);
      vv = ld_b64(rV, vo4, max(t - PF, 0) * row4);
      update(acc, ds);
      ds = ld_b64(rdS, vo4, max(t - PF, 0) * row4);
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
