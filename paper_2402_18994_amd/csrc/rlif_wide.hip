// Kernels and launches of the recurrent time loops over several workgroups (rlif_wide.hpp).
#include "rlif_wide.hpp"

#include <algorithm>

#include "one_grid.hpp"

namespace snn {

typedef RlifWide G;

__device__ __forceinline__ uint32_t dev_load(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void dev_store(uint32_t *p, uint32_t x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
constexpr int SC1 = 16;                                   // device scope, as the cache policy of a buffer access

// A failed poll: true when waiting has to end (a limit reached here or anywhere).
__device__ __forceinline__ bool give_up(int spins, const RlifWideArgs &a) {
  uint32_t *abort_flag = (uint32_t *)a.space;
  if (spins >= a.max_polls) {
    atomicOr(a.err, 2);
    dev_store(abort_flag, 1u);
    return true;
  }
  return (spins & 15) == 15 && dev_load(abort_flag) != 0;
}

// Orders a wavefront's own LDS writes before its reads.
__device__ __forceinline__ void lds_wave_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ float surr_any(int which, float k, float x) {
  switch (which) {                                        // (the same for every lane)
    case 0: return surr_rcp<0>(k, x);
    case 1: return surr_rcp<1>(k, x);
    case 2: return surr_rcp<2>(k, x);
    case 3: return surr_rcp<3>(k, x);
    case 4: return surr_rcp<4>(k, x);
    default: return surr_rcp<5>(k, x);
  }
}

// Group and member of a workgroup; false: none.
__device__ __forceinline__ bool place(const RlifWideArgs &a, int &grp, int &m) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, gl = slot / a.P;
  m = slot - gl * a.P;
  grp = gl * 8 + xcd;
  return grp < a.groups;
}

// The partial sums of the eight wavefronts: written as the accumulators lie (tile i: neurons 16 i + 4 q .. + 3
// of sample c), read as lane = neuron, samples 2 w and 2 w + 1, added in the order of the wavefronts.
// `red` alternates between two buffers, so one barrier a step is enough.
__device__ __forceinline__ void reduce(const f32x4 (&acc)[4], float *red, int w, int lane, float (&sum)[2]) {
  const int c = lane & 15, q = lane >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) *(f32x4 *)(red + (w * G::SB + c) * G::RP + 16 * i + 4 * q) = acc[i];
  lds_barrier();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += red[(k * G::SB + 2 * w + j) * G::RP + lane];
    sum[j] = s;
  }
}

// The updates, one expression for the loops in one launch and the launches of one step.
__device__ __forceinline__ float next_v(float beta, float v, float cur, float sum, bool spike, float theta) {
  return beta * v + cur + 0.5f * sum - (spike ? theta : 0.f);
}
__device__ __forceinline__ float next_g(float beta, float g, float sg, float u, float sum) { return beta * g + sg * (u + sum); }

// RT tiles of 16 rows of R^T from row r0: rows 16 i + c, columns 32 (NKS w + ks) + 8 q ..
template <int NKS, int RT>
__device__ __forceinline__ void load_forward_rows(const RlifWideArgs &a, int r0, int w, int c, int q, bf16x8 (&wf)[RT][NKS]) {
  const rsrc_t rR = make_rsrc(a.R, (unsigned)((size_t)a.ldr * ((a.ld + 127) / 128 * 128) * 2));
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int r = r0 + 16 * i + c, k = 32 * (NKS * w + ks) + 8 * q;
      wf[i][ks] = __builtin_bit_cast(bf16x8, ld_b128(rR, k < a.ldr && r < a.ld ? (r * a.ldr + k) * 2 : OOB, 0));
    }
}

// RT tiles of 16 rows of R from row r0: rows 16 i + c, columns 32 (8 ks + w) + 4 q .. and 16 further (the
// contraction index of an MFMA step runs over two pieces per lane, so that each load of g covers 64 bytes of
// every sample).  Loaded as 16 bytes a lane, columns 8 q ..: of its groups 2 q and 2 q + 1 of four columns the
// lane hands on what others need for theirs, q and q + 4.
template <int NKS, int RT>
__device__ __forceinline__ void load_reverse_rows(const RlifWideArgs &a, int r0, int w, int c, int q, bf16x8 (&wf)[RT][NKS]) {
  const rsrc_t rR = make_rsrc(a.R, (unsigned)((size_t)a.ldr * ((a.ld + 127) / 128 * 128) * 2));
  u32x4 x[RT][NKS];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int r = r0 + 16 * i + c, k = 32 * (8 * ks + w) + 8 * q;
      x[i][ks] = ld_b128(rR, k < a.ldr && r < a.ld ? (r * a.ldr + k) * 2 : OOB, 0);
    }
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      u32x4 f;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        // lanes q of (x[e], x[2 + e]): (0 2 4 6, 1 3 5 7) -> (0 1 4 5, 2 3 6 7) -> (0 1 2 3, 4 5 6 7)
        const auto s = __builtin_amdgcn_permlane16_swap(x[i][ks][e], x[i][ks][2 + e], false, false);
        const auto d = __builtin_amdgcn_permlane32_swap(s[0], s[1], false, false);
        f[e] = d[0];
        f[2 + e] = d[1];
      }
      wf[i][ks] = __builtin_bit_cast(bf16x8, f);
    }
}

// Products of an MFMA step with the hi/lo words of g (two 16-byte pieces per lane), the lower halves first.
template <int NKS, int RT>
__device__ __forceinline__ void add_words(const bf16x8 (&wf)[RT][NKS], int ks, const u32x4 (&x)[2], f32x4 (&acc)[RT]) {
  u32x4 lo, hi;
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      hi[2 * p + e] = __builtin_amdgcn_perm(x[p][2 * e + 1], x[p][2 * e], 0x05040100u);
      lo[2 * p + e] = __builtin_amdgcn_perm(x[p][2 * e + 1], x[p][2 * e], 0x07060302u);
    }
#pragma unroll
  for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i][ks], __builtin_bit_cast(bf16x8, lo), acc[i], 0, 0, 0);
#pragma unroll
  for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i][ks], __builtin_bit_cast(bf16x8, hi), acc[i], 0, 0, 0);
}

// ---------------------------------------------------------------- all steps in a launch
// NKS: steps of 32 neurons of the contraction per wavefront (the layer has at most 256 NKS, and more than 256).
template <int NKS>
__global__ __launch_bounds__(512) void rlif_wide_forward_kernel(const RlifWideArgs a) {
  constexpr int BP = NKS | 1;                             // dwords between the samples' bits of a wavefront in LDS
  __shared__ __align__(16) float red[2][8 * G::SB * G::RP];
  __shared__ uint32_t bits[8][G::SB * BP];
  __shared__ uint64_t out[2][G::SB];
  int grp, m;
  if (!place(a, grp, m)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, q = lane >> 4;
  const int n = m * G::NB + lane, row = a.B * a.ld;
  const unsigned bytes = (unsigned)((size_t)a.T * row * 4);
  const rsrc_t rI = make_rsrc(a.X, bytes), rV = make_rsrc(a.V, bytes), rS = make_rsrc(a.S, bytes / 4);
  uint64_t *const words = (uint64_t *)(a.space + G::WORDS);

  bf16x8 wf[4][NKS];
  load_forward_rows(a, m * G::NB, w, c, q, wf);
  const float beta = n < a.ld ? a.beta_v[n] : 0.f;
  const int gw = a.P * G::SB * 2;                         // words of a group: [member][sample][2]
  // the words this lane fetches: word i = lane + 64 j of the wavefront's 16 x NKS
  constexpr int WPL = (G::SB * NKS + 63) / 64;
  int at[WPL], to[WPL];
#pragma unroll
  for (int j = 0; j < WPL; ++j) {
    const int i = lane + 64 * j, smp = i / NKS, d = i - smp * NKS, k = NKS * w + d;
    at[j] = smp < G::SB && k < 2 * a.P ? ((k >> 1) * G::SB + smp) * 2 + (k & 1) : -1;
    to[j] = min(smp, G::SB - 1) * BP + d;
  }
  for (int i = lane; i < G::SB * BP; i += 64) bits[w][i] = 0u;   // (members that do not exist stay silent)
  bool aborted = false;
  int vo1[2], vo4[2];
  float v[2], cur[2], nxt[2];
  uint64_t sp[2];                                         // spikes of the wavefront's two samples, one bit per lane
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int b = (a.tile0 + grp) * G::SB + 2 * w + j;
    const bool ok = b < a.B && n < a.ld;
    vo1[j] = ok ? b * a.ld + n : OOB;
    vo4[j] = ok ? vo1[j] * 4 : OOB;
    v[j] = 0.f;                                           // V_0 = 0, S_0 = 0
    st_b32(rV, vo4[j], 0, 0u);
    st_b8(rS, vo1[j], 0, 0u);
    sp[j] = __ballot(v[j] > a.theta);
    cur[j] = __uint_as_float(ld_b32(rI, vo4[j], 0));
  }
  // The accesses that nobody waits for within a step - the stores of V_t and S_t, the fetch of I_{t+1} - are
  // issued as soon as the words of step t are in: a wait for a load is a wait for every older access of
  // the wavefront, so behind the publication they would put a memory round trip into the next poll
  // (4.5 us a step at 2048 neurons against 2.9; 2.5 since one wavefront publishes the member's words as
  // whole lines, where each wavefront stored the 32 bytes of its own samples and polled behind them).
  auto io = [&](int t, bool store) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (store) {
        st_b32(rV, vo4[j], t * row * 4, __float_as_uint(v[j]));
        st_b8(rS, vo1[j], t * row, (uint32_t)(sp[j] >> lane) & 1u);
      }
      nxt[j] = __uint_as_float(ld_b32(rI, vo4[j], min(t + 1, a.T - 1) * row * 4));
    }
  };

  for (int t = 0; t + 1 < a.T; ++t) {
    float sum[2] = {0.f, 0.f};
    if (t > 0) {
      // the bits of s_t
      const uint32_t tag = a.tag0 + t, want = tag + a.tag_bias;
      const uint64_t *src = words + ((size_t)(tag & 1) * a.groups + grp) * gw;
      uint64_t x[WPL] = {};
      bool ok = aborted;
      for (int spins = 0; !ok; ++spins) {
        ok = true;
#pragma unroll
        for (int j = 0; j < WPL; ++j)
          if (at[j] >= 0 && (spins == 0 || (uint32_t)(x[j] >> 32) != want))
            x[j] = __hip_atomic_load(src + at[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < WPL; ++j)
          if (at[j] >= 0 && (uint32_t)(x[j] >> 32) != want) ok = false;
        if (!ok) {
          if (give_up(spins, a)) { aborted = true; break; }
          __builtin_amdgcn_s_sleep(1);                      // (without it the polls delay the stores they wait for)
        }
      }
      io(t, true);
#pragma unroll
      for (int j = 0; j < WPL; ++j)
        if (at[j] >= 0) bits[w][to[j]] = aborted ? 0u : (uint32_t)x[j];
      lds_wave_sync();
      f32x4 acc[4] = {};
      uint32_t d[NKS];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) d[ks] = bits[w][c * BP + ks];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        // eight spikes of sample c as bfloat16 2.0 / 0.0 (the sums are halved below: exact): the byte sits at
        // bits 0..7 and 15..22, so that a shift by 14 - 2 r brings spikes 2 r and 2 r + 1 to bits 14 and 30
        uint32_t z = (d[ks] >> (8 * q)) & 0xFFu;
        z |= z << 15;
        u32x4 f;
        f[0] = (z << 14) & 0x40004000u;
        f[1] = (z << 12) & 0x40004000u;
        f[2] = (z << 10) & 0x40004000u;
        f[3] = (z << 8) & 0x40004000u;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i][ks], __builtin_bit_cast(bf16x8, f), acc[i], 0, 0, 0);
      }
      reduce(acc, red[t & 1], w, lane, sum);
    } else {
      io(t, false);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      v[j] = next_v(beta, v[j], cur[j], sum[j], (sp[j] >> lane) & 1, a.theta);
      sp[j] = __ballot(v[j] > a.theta);
    }
    if (t + 2 < a.T) {                                    // publish s_{t+1}: one wavefront writes the member's 256 bytes
      if (lane == 0) { out[t & 1][2 * w] = sp[0]; out[t & 1][2 * w + 1] = sp[1]; }
      lds_barrier();
      if (tid < 32) {
        const uint32_t tag = a.tag0 + t + 1;
        uint64_t *dst = words + ((size_t)(tag & 1) * a.groups + grp) * gw + m * G::SB * 2 + tid;
        __hip_atomic_store(dst, (uint64_t)((const uint32_t *)out[t & 1])[tid] | ((uint64_t)tag << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) cur[j] = nxt[j];
  }
  if (a.T > 1) io(a.T - 1, true);                         // the last V and S
}

// g <- beta g + surr(V_t - theta) (dS_t - theta g + R g), dI_t = g before the update.
template <int NKS>
__global__ __launch_bounds__(512) void rlif_wide_reverse_kernel(const RlifWideArgs a) {
  __shared__ __align__(16) float red[2][8 * G::SB * G::RP];
  __shared__ __align__(16) uint32_t stage[1024];          // the member's words of g on their way out
  __shared__ int ended;
  int grp, m;
  if (!place(a, grp, m)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, q = lane >> 4;
  const int n = m * G::NB + lane, row = a.B * a.ld;
  const unsigned bytes = (unsigned)((size_t)a.T * row * 4);
  const rsrc_t rdS = make_rsrc(a.X, bytes), rV = make_rsrc(a.V, bytes), rdI = make_rsrc(a.dI, bytes);
  const unsigned gpar = (unsigned)a.groups * a.P * G::SB * G::NB * 4;   // bytes of one parity of the exchanged g
  const rsrc_t rG = make_rsrc(a.space + G::G, 2 * gpar);
  uint32_t *const flags = (uint32_t *)(a.space + G::FLAGS) + grp * G::SLOTS;

  bf16x8 wf[4][NKS];
  load_reverse_rows(a, m * G::NB, w, c, q, wf);
  // The words of a member lie as the readers' fragments want them, [half of the neurons][piece][q][sample][4
  // words]: a load of a wavefront is 1 KB in a row (rows of 64 words per sample: 16 pieces of
  // 64 bytes, the loads and products of a step 3.1 kilocycles instead of 1.8 at 1024 neurons).
  int go[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    const int k = 8 * ks + w, p = k >> 1;
    go[ks] = p < a.P ? (((grp * a.P + p) * 2 + (k & 1)) * 2 * 64 + lane) * 16 : OOB;
  }
  const int gm = (grp * a.P + m) * 4096, gs = ((lane >> 5) * 2 + ((lane >> 4) & 1)) * 1024 + (((lane >> 2) & 3) * 16 + 2 * w) * 16 + (lane & 3) * 4;
  const float beta = n < a.ld ? a.beta_v[n] : 0.f;
  bool aborted = false;
  if (tid == 0) ended = 0;
  int vo4[2];
  float g[2], db[2], ds[2], vt[2], ds_n[2], vt_n[2];
  uint32_t hl[2];                                         // g as the product and dI hold it
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int b = (a.tile0 + grp) * G::SB + 2 * w + j;
    vo4[j] = b < a.B && n < a.ld ? (b * a.ld + n) * 4 : OOB;
    g[j] = db[j] = 0.f;                                   // g_T = 0
    hl[j] = pack_hl(g[j]);
    ds[j] = __uint_as_float(ld_b32(rdS, vo4[j], (a.T - 1) * row * 4));
    vt[j] = __uint_as_float(ld_b32(rV, vo4[j], (a.T - 1) * row * 4));
  }
  __syncthreads();
  // What nobody waits for within a step goes between the products and the sum over the wavefronts: a wait for
  // a load is a wait for every older access of the wavefront, so in front of the loads of g, or among them,
  // these put a memory round trip into the step (8.0 against 4.8 us a step at 2048 neurons).
  auto io = [&](int t) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      st_b32(rdI, vo4[j], t * row * 4, hl[j]);
      ds_n[j] = __uint_as_float(ld_b32(rdS, vo4[j], max(t - 1, 0) * row * 4));
      vt_n[j] = __uint_as_float(ld_b32(rV, vo4[j], max(t - 1, 0) * row * 4));
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  for (int s = 0; s < a.T; ++s) {                         // step s of the reverse pass is time T - 1 - s
    const int t = a.T - 1 - s;
    float sum[2] = {0.f, 0.f}, sg[2], u[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      sg[j] = surr_any(a.surrogate, a.slope, vt[j] - a.theta);
      u[j] = ds[j] - a.theta * g[j];
      db[j] += g[j] * vt[j];
    }
    if (s > 0) {
      const uint32_t tag = a.tag0 + s;
      if (w == 0) {                                       // one wavefront waits for the members' flags
        const uint32_t want = tag + a.tag_bias;
        for (int spins = 0; !aborted; ++spins) {
          const uint32_t f = dev_load(flags + min(lane, a.P - 1));
          if (__all((int)(f - want) >= 0)) break;
          if (__any(give_up(spins, a))) aborted = true;
        }
        if (aborted && lane == 0) ended = 1;
      }
      __syncthreads();
      const int par = (int)((tag & 1) * gpar);
      u32x4 x[NKS][2];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int p = 0; p < 2; ++p)
          x[ks][p] = __builtin_amdgcn_raw_buffer_load_b128(rG, go[ks] == OOB ? OOB : go[ks] + 1024 * p, par, SC1);
      f32x4 acc[4] = {};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) add_words(wf, ks, x[ks], acc);
      io(t);
      reduce(acc, red[s & 1], w, lane, sum);
      if (ended) aborted = true;                          // (written before the barriers of this step)
    } else {
      io(t);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      g[j] = next_g(beta, g[j], sg[j], u[j], sum[j]);
      hl[j] = pack_hl(g[j]);
    }
    if (t > 0) {
      const uint32_t tag = a.tag0 + s + 1;
      // through LDS, so that a wavefront writes whole lines
#pragma unroll
      for (int j = 0; j < 2; ++j) *(uint32_t *)((char *)stage + gs + 16 * j) = hl[j];
      lds_barrier();
      __builtin_amdgcn_raw_buffer_store_b64(*(const u32x2 *)((char *)stage + tid * 8), rG, gm + tid * 8, (int)((tag & 1) * gpar), SC1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // acknowledged: visible to every device-scope load
      __syncthreads();
      if (tid == 0) dev_store(flags + m, tag);
#pragma unroll
      for (int j = 0; j < 2; ++j) { ds[j] = ds_n[j]; vt[j] = vt_n[j]; }
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if (a.db_part && vo4[j] != OOB) a.db_part[vo4[j] / 4] = db[j];   // per sample, the sum over t of g_{t+1} V_t
}

// ---------------------------------------------------------------- a launch per step
// The same sums in the same order, the state through V and gs, the spikes and words through S and dI: nobody
// waits for anybody.  A workgroup takes SN neurons and keeps their rows of R for all its tiles of 16 samples.
// It is bound by the words and by these rows, up to 128 KB a launch: half the neurons of the loops above, so that
// twice the compute units share them where tiles are few (2048 neurons, one sample: 6.0 us forward and 7.0 reverse,
// with 64 neurons 9.6 and 18.7), and always read on one XCD, in whose L2 they lie (workgroup i runs on
// XCD i % 8, blocks of neurons are padded to a multiple of 8).
constexpr int SN = 32;
struct StepPlace {
  int lane, w, c, q, n0, n, grp;                          // first neuron of the block, neuron of the lane
  int half;                                               // of the wavefront's two samples
  bool live;
  static __host__ __device__ int blocks(int ld) { return (ld + SN - 1) / SN; }
  static __host__ __device__ int pitch(int ld) { return blocks(ld) < 8 ? blocks(ld) : (blocks(ld) + 7) / 8 * 8; }
  __device__ __forceinline__ explicit StepPlace(const RlifWideArgs &a) {
    const int m = blockIdx.x % pitch(a.ld);
    grp = blockIdx.x / pitch(a.ld);
    lane = threadIdx.x & 63; w = threadIdx.x >> 6; c = lane & 15; q = lane >> 4; half = lane >> 5;
    n0 = m * SN;
    n = n0 + (lane & 31);
    live = m < blocks(a.ld);
  }
};
// As reduce(), for SN neurons and ST tiles of samples: lane = neuron, its half of the wavefront's samples.
template <int ST>
__device__ __forceinline__ void step_reduce(const f32x4 (&acc)[ST][2], float *red, const StepPlace &p, float (&sum)[ST]) {
  constexpr int RP = SN + 4;
#pragma unroll
  for (int u = 0; u < ST; ++u)
#pragma unroll
    for (int i = 0; i < 2; ++i) *(f32x4 *)(red + ((u * 8 + p.w) * G::SB + p.c) * RP + 16 * i + 4 * p.q) = acc[u][i];
  lds_barrier();
#pragma unroll
  for (int u = 0; u < ST; ++u) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += red[((u * 8 + k) * G::SB + 2 * p.w + p.half) * RP + (p.lane & 31)];
    sum[u] = s;
  }
}

// Step a.step: from V_t, S_t and I_t to V_{t+1} and S_{t+1}; step 0 also writes V_0 and S_0.
template <int NKS, int ST>
__global__ __launch_bounds__(512) void rlif_wide_forward_step_kernel(const RlifWideArgs a) {
  __shared__ __align__(16) float red[2][ST * 8 * G::SB * (SN + 4)];
  const StepPlace p(a);
  if (!p.live) return;
  const int row = a.B * a.ld, t = a.step;
  const unsigned bytes = (unsigned)((size_t)a.T * row * 4);
  const rsrc_t rI = make_rsrc(a.X, bytes), rV = make_rsrc(a.V, bytes), rS = make_rsrc(a.S, bytes / 4);
  bf16x8 wf[2][NKS];
  load_forward_rows(a, p.n0, p.w, p.c, p.q, wf);
  const float beta = p.n < a.ld ? a.beta_v[p.n] : 0.f;
  int par = 0;
  for (int tile = ST * p.grp; tile * G::SB < a.B; tile += ST * a.groups, par ^= 1) {
    int vo1[ST], vo4[ST];
    float v[ST], cur[ST], sum[ST];
    u32x2 x[ST][NKS];
#pragma unroll
    for (int u = 0; u < ST; ++u) {
      const int b = (tile + u) * G::SB + 2 * p.w + p.half, bc = (tile + u) * G::SB + p.c;
      const bool ok = b < a.B && p.n < a.ld;
      vo1[u] = ok ? b * a.ld + p.n : OOB;
      vo4[u] = ok ? vo1[u] * 4 : OOB;
      v[u] = sum[u] = 0.f;                                // V_0 = 0, S_0 = 0
      cur[u] = __uint_as_float(ld_b32(rI, vo4[u], t * row * 4));
      if (t == 0) {
        st_b32(rV, vo4[u], 0, 0u);
        st_b8(rS, vo1[u], 0, 0u);
        continue;
      }
      v[u] = __uint_as_float(ld_b32(rV, vo4[u], t * row * 4));
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int k = 32 * (NKS * p.w + ks) + 8 * p.q;
        x[u][ks] = ld_b64(rS, bc < a.B && k < a.ld ? bc * a.ld + k : OOB, t * row);
      }
    }
    if (t > 0) {
      f32x4 acc[ST][2] = {};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int u = 0; u < ST; ++u) {
          // eight spike bytes as bfloat16 2.0 / 0.0 (the sums are halved in next_v: exact)
          const uint32_t x0 = x[u][ks][0] << 6, x1 = x[u][ks][1] << 6;
          const u32x4 f = {__builtin_amdgcn_perm(0u, x0, 0x010C000Cu), __builtin_amdgcn_perm(0u, x0, 0x030C020Cu),
                           __builtin_amdgcn_perm(0u, x1, 0x010C000Cu), __builtin_amdgcn_perm(0u, x1, 0x030C020Cu)};
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[u][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i][ks], __builtin_bit_cast(bf16x8, f), acc[u][i], 0, 0, 0);
        }
      step_reduce(acc, red[par], p, sum);
    }
    if (t + 1 < a.T) {
#pragma unroll
      for (int u = 0; u < ST; ++u) {
        const float vn = next_v(beta, v[u], cur[u], sum[u], v[u] > a.theta, a.theta);
        st_b32(rV, vo4[u], (t + 1) * row * 4, __float_as_uint(vn));
        st_b8(rS, vo1[u], (t + 1) * row, vn > a.theta ? 1u : 0u);
      }
    }
  }
}

// Step a.step of the reverse pass, time t = T - 1 - step: from g (gs, and dI_t in the product) to g and dI_{t-1}.
template <int NKS, int ST>
__global__ __launch_bounds__(512) void rlif_wide_reverse_step_kernel(const RlifWideArgs a) {
  __shared__ __align__(16) float red[2][ST * 8 * G::SB * (SN + 4)];
  const StepPlace p(a);
  if (!p.live) return;
  const int row = a.B * a.ld, t = a.T - 1 - a.step;
  const unsigned bytes = (unsigned)((size_t)a.T * row * 4);
  const rsrc_t rdS = make_rsrc(a.X, bytes), rV = make_rsrc(a.V, bytes), rdI = make_rsrc(a.dI, bytes);
  bf16x8 wf[2][NKS];
  load_reverse_rows(a, p.n0, p.w, p.c, p.q, wf);
  const float beta = p.n < a.ld ? a.beta_v[p.n] : 0.f;
  int par = 0;
  for (int tile = ST * p.grp; tile * G::SB < a.B; tile += ST * a.groups, par ^= 1) {
    bool ok[ST];
    int vo[ST];
    float g[ST], db[ST], ds[ST], vt[ST], sum[ST];
#pragma unroll
    for (int u = 0; u < ST; ++u) {
      const int b = (tile + u) * G::SB + 2 * p.w + p.half;
      ok[u] = b < a.B && p.n < a.ld;
      vo[u] = ok[u] ? b * a.ld + p.n : 0;
      ds[u] = __uint_as_float(ld_b32(rdS, ok[u] ? vo[u] * 4 : OOB, t * row * 4));
      vt[u] = __uint_as_float(ld_b32(rV, ok[u] ? vo[u] * 4 : OOB, t * row * 4));
      g[u] = db[u] = sum[u] = 0.f;                        // g_T = 0
      if (a.step == 0) {
        st_b32(rdI, ok[u] ? vo[u] * 4 : OOB, t * row * 4, 0u);
        continue;
      }
      g[u] = a.gs[vo[u]];
      if (a.db_part) db[u] = a.db_part[vo[u]];
    }
    if (a.step > 0) {
      f32x4 acc[ST][2] = {};
      constexpr int NX = ST * NKS > 12 ? 4 : NKS;         // steps of words in flight: what the registers hold
#pragma unroll
      for (int k0 = 0; k0 < NKS; k0 += NX) {
        u32x4 x[ST][NX][2];
#pragma unroll
        for (int u = 0; u < ST; ++u)
#pragma unroll
          for (int ks = 0; ks < NX; ++ks)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int bc = (tile + u) * G::SB + p.c, k = 32 * (8 * (k0 + ks) + p.w) + 16 * h + 4 * p.q;
              x[u][ks][h] = ld_b128(rdI, k0 + ks < NKS && bc < a.B && k < a.ld ? (bc * a.ld + k) * 4 : OOB, t * row * 4);
            }
#pragma unroll
        for (int u = 0; u < ST; ++u)
#pragma unroll
          for (int ks = 0; ks < NX; ++ks)
            if (k0 + ks < NKS) add_words(wf, k0 + ks, x[u][ks], acc[u]);
        if (NX < NKS) __builtin_amdgcn_sched_barrier(0);
      }
      step_reduce(acc, red[par], p, sum);
    }
#pragma unroll
    for (int u = 0; u < ST; ++u) {
      const float sg = surr_any(a.surrogate, a.slope, vt[u] - a.theta), w = ds[u] - a.theta * g[u];
      db[u] += g[u] * vt[u];
      g[u] = next_g(beta, g[u], sg, w, sum[u]);
      if (t > 0) st_b32(rdI, ok[u] ? vo[u] * 4 : OOB, (t - 1) * row * 4, pack_hl(g[u]));
      if (ok[u]) {
        a.gs[vo[u]] = g[u];
        if (a.db_part) a.db_part[vo[u]] = db[u];
      }
    }
  }
}

// Zeroes `bytes` (a multiple of 4) of the exchange space.
static __global__ __launch_bounds__(256) void clear_kernel(uint32_t *p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}
static hipError_t clear(hipStream_t st, char *p, size_t bytes) {
  hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((bytes / 4 + 255) / 256)), dim3(256), 0, st, (uint32_t *)p, (int)(bytes / 4));
  return hipGetLastError();
}

// Launches `loop` over all tiles and steps, as many groups at once as fit SLOTS workgroups per XCD, when the
// compute units hold them (persist) and no other such grid can run beside it; else `step` for every step,
// where nobody waits.  The first `cleared` bytes of the exchange space, and the words, start from zero.
template <typename K>
static hipError_t run(hipStream_t st, RlifWideArgs a, int cus, bool persist, size_t cleared, bool words, int steps, K loop, K step1, K step2) {
  a.P = (a.ld + G::NB - 1) / G::NB;
  const int tiles = (a.B + G::SB - 1) / G::SB;
  const dim3 block(512);
  const OneGridAtATime order(st, persist && cus >= 8 * G::SLOTS);
  hipError_t e = hipSuccess;
  if (order.ordered()) {
    if ((e = clear(st, a.space, cleared)) != hipSuccess) return e;
    if (words && (e = clear(st, a.space + G::WORDS, G::WORD_BYTES)) != hipSuccess) return e;
    a.groups = std::min(tiles, 8 * (G::SLOTS / a.P));
    const dim3 grid((unsigned)(8 * a.P * ((a.groups + 7) / 8)));
    int chunk = 0;
    for (a.tile0 = 0; a.tile0 < tiles; a.tile0 += a.groups, ++chunk) {
      a.tag0 = (uint32_t)chunk * (uint32_t)a.T;
      hipLaunchKernelGGL(loop, grid, block, 0, st, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return e;
  }
  // a tile at a time while the compute units take one each, else two, whose loads are in flight together
  const int most = std::max(1, cus / StepPlace::blocks(a.ld)), ST = tiles > most ? 2 : 1;
  a.groups = std::min((tiles + ST - 1) / ST, most);
  const dim3 grid((unsigned)(StepPlace::pitch(a.ld) * a.groups));
  for (a.step = 0; a.step < steps; ++a.step) {
    hipLaunchKernelGGL(ST == 1 ? step1 : step2, grid, block, 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return e;
}

#define SNN_WIDE_CASE(dir, n, ...)                                                           \
  return run(st, a, cus, persist, __VA_ARGS__, rlif_wide_##dir##_kernel<n>, rlif_wide_##dir##_step_kernel<n, 1>, rlif_wide_##dir##_step_kernel<n, 2>)
#define SNN_WIDE(dir, ...)                                                                   \
  switch ((a.ld + 255) / 256) {                                                              \
    case 2: SNN_WIDE_CASE(dir, 2, __VA_ARGS__);                                              \
    case 3: SNN_WIDE_CASE(dir, 3, __VA_ARGS__);                                              \
    case 4: SNN_WIDE_CASE(dir, 4, __VA_ARGS__);                                              \
    case 5: SNN_WIDE_CASE(dir, 5, __VA_ARGS__);                                              \
    case 6: SNN_WIDE_CASE(dir, 6, __VA_ARGS__);                                              \
    case 7: SNN_WIDE_CASE(dir, 7, __VA_ARGS__);                                              \
    default: SNN_WIDE_CASE(dir, 8, __VA_ARGS__);                                             \
  }

hipError_t rlif_wide_forward(hipStream_t st, RlifWideArgs a, int cus, bool persist) {
  SNN_WIDE(forward, G::FLAGS, true, std::max(a.T - 1, 1))
}

hipError_t rlif_wide_reverse(hipStream_t st, RlifWideArgs a, int cus, bool persist) {
  SNN_WIDE(reverse, G::FLAGS + G::FLAG_BYTES, false, a.T)
}
#undef SNN_WIDE
#undef SNN_WIDE_CASE

}  // namespace snn
