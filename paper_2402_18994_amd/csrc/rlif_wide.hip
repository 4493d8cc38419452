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

// NKS: steps of 32 neurons of the contraction per wavefront (the layer has at most 256 NKS).
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
  const rsrc_t rR = make_rsrc(a.R, (unsigned)((size_t)a.ldr * ((a.ld + 127) / 128 * 128) * 2));
  uint64_t *const words = (uint64_t *)(a.space + G::WORDS);

  bf16x8 wf[4][NKS];                                      // rows 16 i + c of the member, columns 32 (NKS w + ks) + 8 q ..
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int r = m * G::NB + 16 * i + c, k = 32 * (NKS * w + ks) + 8 * q;
      wf[i][ks] = __builtin_bit_cast(bf16x8, ld_b128(rR, k < a.ldr && r < a.ld ? (r * a.ldr + k) * 2 : OOB, 0));
    }
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
    if (a.step0 > 0) v[j] = __uint_as_float(ld_b32(rV, vo4[j], a.step0 * row * 4));
    else {
      st_b32(rV, vo4[j], 0, 0u);
      st_b8(rS, vo1[j], 0, 0u);
    }
    sp[j] = __ballot(v[j] > a.theta);
    cur[j] = __uint_as_float(ld_b32(rI, vo4[j], a.step0 * row * 4));
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

  const int t_end = min(a.step0 + a.steps, a.T - 1);
  for (int t = a.step0; t < t_end; ++t) {
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
      io(t, t > a.step0);
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
      v[j] = beta * v[j] + cur[j] + 0.5f * sum[j] - ((sp[j] >> lane) & 1 ? a.theta : 0.f);
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
  if (t_end > a.step0) io(t_end, true);                   // the last V and S
}

// g <- beta g + surr(V_t - theta) (dS_t - theta g + R g), dI_t = g before the update.  The contraction index
// of an MFMA step runs over two 16-byte pieces per lane (words 4 q .. and 16 + 4 q ..), so that each load of
// g covers 64 bytes of every sample.
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
  const rsrc_t rR = make_rsrc(a.R, (unsigned)((size_t)a.ldr * ((a.ld + 127) / 128 * 128) * 2));
  const unsigned gpar = (unsigned)a.groups * a.P * G::SB * G::NB * 4;   // bytes of one parity of the exchanged g
  const rsrc_t rG = make_rsrc(a.space + G::G, 2 * gpar);
  uint32_t *const flags = (uint32_t *)(a.space + G::FLAGS) + grp * G::SLOTS;

  bf16x8 wf[4][NKS];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int r = m * G::NB + 16 * i + c, k = 32 * (8 * ks + w) + 4 * q;
      u32x4 f = {};
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int kp = k + 16 * p;
        const u32x2 x = ld_b64(rR, kp < a.ldr && r < a.ld ? (r * a.ldr + kp) * 2 : OOB, 0);
        f[2 * p] = x[0];
        f[2 * p + 1] = x[1];
      }
      wf[i][ks] = __builtin_bit_cast(bf16x8, f);
    }
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
    const int t = a.T - 1 - a.step0;
    if (a.step0 > 0) {
      if (vo4[j] != OOB) g[j] = a.gs[vo4[j] / 4];
      if (a.db_part && vo4[j] != OOB) db[j] = a.db_part[vo4[j] / 4];
    }
    hl[j] = pack_hl(g[j]);
    ds[j] = __uint_as_float(ld_b32(rdS, vo4[j], t * row * 4));
    vt[j] = __uint_as_float(ld_b32(rV, vo4[j], t * row * 4));
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

  const int s_end = min(a.step0 + a.steps, a.T);
  for (int s = a.step0; s < s_end; ++s) {                 // step s of the reverse pass is time T - 1 - s
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
      for (int ks = 0; ks < NKS; ++ks) {
        u32x4 lo, hi;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            hi[2 * p + e] = __builtin_amdgcn_perm(x[ks][p][2 * e + 1], x[ks][p][2 * e], 0x05040100u);
            lo[2 * p + e] = __builtin_amdgcn_perm(x[ks][p][2 * e + 1], x[ks][p][2 * e], 0x07060302u);
          }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i][ks], __builtin_bit_cast(bf16x8, lo), acc[i], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i][ks], __builtin_bit_cast(bf16x8, hi), acc[i], 0, 0, 0);
      }
      io(t);
      reduce(acc, red[s & 1], w, lane, sum);
      if (ended) aborted = true;                          // (written before the barriers of this step)
    } else {
      io(t);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      g[j] = beta * g[j] + sg[j] * (u[j] + sum[j]);
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
      if (s + 1 == s_end) {                               // (a launch of one step)
#pragma unroll
        for (int j = 0; j < 2; ++j) st_b32(rdI, vo4[j], (t - 1) * row * 4, hl[j]);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) { ds[j] = ds_n[j]; vt[j] = vt_n[j]; }
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if (vo4[j] != OOB) {
      if (a.steps == 1) a.gs[vo4[j] / 4] = g[j];
      if (a.db_part) a.db_part[vo4[j] / 4] = db[j];       // per sample, the sum over t of g_{t+1} V_t
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

// Launches `kernel` over all tiles and steps: as many groups at once as fit SLOTS workgroups per XCD, all steps
// in a launch when the compute units hold them (persist) and no other such grid can run beside it, else a step
// per launch, where nobody waits (700-2048(rec)-20, T = 64, B = 128: 866 and 1345 us instead of 162 and 273).
template <typename K> static hipError_t run(hipStream_t st, RlifWideArgs a, int cus, bool persist, K kernel) {
  a.P = (a.ld + G::NB - 1) / G::NB;
  const int tiles = (a.B + G::SB - 1) / G::SB, most = std::min(8 * (G::SLOTS / a.P), (int)G::GROUPS);
  a.groups = std::min(tiles, most);
  const dim3 grid((unsigned)(8 * a.P * ((a.groups + 7) / 8))), block(512);
  persist = persist && cus >= 8 * G::SLOTS;
  const OneGridAtATime order(st, persist);
  persist = order.ordered();
  hipError_t e = hipSuccess;
  int chunk = 0;
  for (a.tile0 = 0; a.tile0 < tiles; a.tile0 += a.groups, ++chunk) {
    a.tag0 = (uint32_t)chunk * (uint32_t)a.T;
    a.steps = persist ? a.T : 1;
    for (a.step0 = 0; a.step0 < a.T; a.step0 += a.steps) {
      hipLaunchKernelGGL(kernel, grid, block, 0, st, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  return e;
}

#define SNN_WIDE(name)                                                                       \
  switch ((a.ld + 255) / 256) {                                                              \
    case 1: return run(st, a, cus, persist, name<1>);                                        \
    case 2: return run(st, a, cus, persist, name<2>);                                        \
    case 3: return run(st, a, cus, persist, name<3>);                                        \
    case 4: return run(st, a, cus, persist, name<4>);                                        \
    case 5: return run(st, a, cus, persist, name<5>);                                        \
    case 6: return run(st, a, cus, persist, name<6>);                                        \
    case 7: return run(st, a, cus, persist, name<7>);                                        \
    default: return run(st, a, cus, persist, name<8>);                                       \
  }

hipError_t rlif_wide_forward(hipStream_t st, RlifWideArgs a, int cus, bool persist) {
  hipError_t e = clear(st, a.space, G::FLAGS);
  if (e == hipSuccess) e = clear(st, a.space + G::WORDS, G::WORD_BYTES);
  if (e != hipSuccess) return e;
  SNN_WIDE(rlif_wide_forward_kernel)
}

hipError_t rlif_wide_reverse(hipStream_t st, RlifWideArgs a, int cus, bool persist) {
  const hipError_t e = clear(st, a.space, G::FLAGS + G::FLAG_BYTES);
  if (e != hipSuccess) return e;
  SNN_WIDE(rlif_wide_reverse_kernel)
}
#undef SNN_WIDE

}  // namespace snn
