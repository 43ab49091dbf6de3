// Wave64 / workgroup primitives for the gfx950 kernels: ballot-popcount ranks, DPP prefix
// scans, a 256-thread block scan.  Device code only.
#pragma once

#include "rgc_internal.h"

namespace rgc {

// Tensor pointers reach the kernels through descriptor tables in memory, so the compiler sees
// generic ("flat") pointers and would emit flat_load/flat_store, which also tick the LDS
// counter and make every LDS wait a wait for all outstanding global traffic.  Everything the
// library touches through such pointers is global memory: say so.
template <typename T>
using gptr = __attribute__((address_space(1))) T*;

template <typename T>
__device__ __forceinline__ gptr<T> as_global(T* p) {
  return (gptr<T>)p;
}

__device__ __forceinline__ uint32_t lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Number of set bits of `mask` that belong to lanes below the calling lane.
__device__ __forceinline__ uint32_t rank_below(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

__device__ __forceinline__ uint32_t popc64(unsigned long long m) {
  return static_cast<uint32_t>(__popcll(m));
}

template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp_shift_add(uint32_t v) {
  // lanes without a source (shifted in from outside the row, or rows masked off) add 0
  uint32_t t = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      0, static_cast<int>(v), kCtrl, kRowMask, 0xF, false));
  return v + t;
}

// Inclusive prefix sum over the 64 lanes of a wave using DPP row shifts and row broadcasts.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v = dpp_shift_add<0x111, 0xF>(v);  // row_shr:1
  v = dpp_shift_add<0x112, 0xF>(v);  // row_shr:2
  v = dpp_shift_add<0x114, 0xF>(v);  // row_shr:4
  v = dpp_shift_add<0x118, 0xF>(v);  // row_shr:8   -> inclusive scan inside each row of 16
  v = dpp_shift_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_shift_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

__device__ __forceinline__ uint32_t wave_total(uint32_t incl) {
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
}

// Exclusive prefix sum over the threads of a workgroup of kWaves waves.  `lds` holds >= kWaves words.
// Contains barriers: every thread of the workgroup must call it.
template <uint32_t kWaves = kWavesPerBlock>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds, uint32_t& total) {
  const uint32_t incl = wave_incl_scan(v);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 63u) lds[wave] = incl;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (uint32_t w = 0; w < kWaves; ++w) {
    const uint32_t t = lds[w];
    off += (w < wave) ? t : 0u;
    tot += t;
  }
  total = tot;
  return off + incl - v;
}

__device__ __forceinline__ uint32_t ld_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ... at an address that is the same for the whole wave.
__device__ __forceinline__ uint32_t ld_uniform(const uint32_t* p) { return __builtin_amdgcn_readfirstlane(ld_agent(p)); }

__device__ __forceinline__ void st_agent(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// "Last workgroup of the layer" election.  Contract: everything the elected workgroup will
// read from this phase was written with device-scope atomics or st_agent() (both go to the
// device's coherence point, unlike plain stores which may sit in one XCD's L2 until the kernel
// ends), and is read back with ld_agent().  Waiting for the wave's outstanding memory
// operations before the counter increment is then all the ordering needed; a full
// __threadfence() here would force an L2 write-back per workgroup and costs several times the
// streaming pass itself.
// Returns true in every thread of exactly one workgroup per (layer, phase): the one whose
// increment completes the count.  That workgroup also resets the counter.
// The election is two-level: workgroups first count themselves into the counter of their group of
// kElectGroup consecutive workgroups, the last of a group counts the group into the layer's
// counter.  Thousands of workgroups finishing a short phase together otherwise queue up on one
// address (a same-address device atomic takes ~10-25 ns, i.e. ~100 us for 4000 workgroups).
// `again_soon`: the counters are used again before the kernel ends (fallback_kernel): a group's reset has to have arrived before
// the layer's last workgroup can be elected, which lets the next phase begin.
constexpr uint32_t kElectGroup = 32;

__device__ __forceinline__ bool last_block_of_layer(uint32_t* layer_done, uint32_t* group_done, uint32_t wg_in_layer,
                                                    uint32_t wg_count, uint32_t* lds_flag, bool again_soon = false) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t grp = wg_in_layer / kElectGroup;
    const uint32_t groups = (wg_count + kElectGroup - 1u) / kElectGroup;
    const uint32_t in_grp = (grp + 1u == groups) ? wg_count - grp * kElectGroup : kElectGroup;
    bool last = false;
    if (atomicAdd(&group_done[grp], 1u) + 1u == in_grp) {
      st_agent(&group_done[grp], 0u);
      if (again_soon) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (groups == 1u) {
        last = true;                               // (a round trip less for layers of one group)
      } else if (atomicAdd(layer_done, 1u) + 1u == groups) {
        st_agent(layer_done, 0u);
        last = true;
      }
    }
    *lds_flag = last ? 1u : 0u;
  }
  __syncthreads();
  return *lds_flag != 0u;
}

// ---------------------------------------------------------------- shared by every pass over a layer
__device__ __forceinline__ uint32_t fbits(float x) { return __float_as_uint(x); }

// One 16-byte access per lane.  The tensors are only known to be 4-byte aligned (layers packed back to back in one
// flat buffer start anywhere), and gfx950 needs no more for a dwordx4 access: an unaligned tensor costs one more cache
// line per KiB and array.  (24 tensors of odd sizes packed back to back, 8.0 M elements with a velocity: a compression
// call took 80 us when unaligned tensors were read and written a word at a time, 54 us this way.)
typedef float vf4 __attribute__((ext_vector_type(4), aligned(4)));

typedef __attribute__((address_space(1))) vf4* gvf4;
typedef __attribute__((address_space(1))) const vf4* gcvf4;
__device__ __forceinline__ gvf4 as_vec(float* p) { return (gvf4)(p); }
__device__ __forceinline__ gcvf4 as_vec(const float* p) { return (gcvf4)(p); }

// One access of the streaming passes to the residual and the velocity.  kNt: past the memory-side cache, for calls
// whose tensors do not stay in it until the next call anyway (see stream_past_cache() in rgc_api.cpp).
template <bool kNt>
__device__ __forceinline__ vf4 stream_load(gcvf4 p) {
  if constexpr (kNt) return __builtin_nontemporal_load(p); else return *p;
}
template <bool kNt>
__device__ __forceinline__ void stream_store(gvf4 p, vf4 v) {
  if constexpr (kNt) __builtin_nontemporal_store(v, p); else *p = v;
}

// The accumulate of Algorithm 1 and its variants (Sections 2.4, 2.5): every gradient element is
// first multiplied with the clipping coefficient (1 when there is none: an exact product), then
//   plain:                a = V + g
//   momentum correction:  u = fma(m, u, g),   a = V + u
//   its Nesterov form:    u = m * (u + g),    a = (V + u) + g      (every operation rounded)
struct AccumRule {
  float m;       // momentum factor
  float scale;   // clipping coefficient
};

template <bool kMom, bool kNest>
__device__ __forceinline__ void accum4(const float (&g)[4], const float (&v)[4], float (&u)[4],
                                       const AccumRule& r, float (&a)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float gs = __fmul_rn(r.scale, g[j]);
    if constexpr (kMom && kNest) {
      u[j] = __fmul_rn(r.m, __fadd_rn(u[j], gs));
      a[j] = __fadd_rn(__fadd_rn(v[j], u[j]), gs);
    } else if constexpr (kMom) {
      u[j] = __fmaf_rn(r.m, u[j], gs);
      a[j] = __fadd_rn(v[j], u[j]);
    } else {
      a[j] = __fadd_rn(v[j], gs);
    }
  }
}

// The whole groups of 256 elements of a wave's stretch, which begins at the three pointers (`U4` only with a velocity), kAhead groups
// ahead: f(g, v, u, o, next) gets a lane's four elements of a group, which are number 4 o .. 4 o + 3 of the stretch, and calls next(), which asks
// for the group kAhead further on, when it has read them and before it stores anything.  Loads and stores share one counter, in
// order, so a wait for loads that were issued after stores would be a wait for the stores too.  (Four groups' loads, then their work and
// stores, then the next four, against this with kAhead = 1 / 2 / 4, us per call: dense layers, whose lists leave them little room, ResNet-50
// set at 1.5625 % 102.9 / 96.2 / 100.1 / -, VGG16 set at 25 % 913 / 901 / 899 / -, where its runs differ by as much; thresholds reused, LSTM
// set 167.7 / 167.9 / 166.6 / 163.5, searched, 126 M elements at 0.4 % 384 / 386 / 382 / 376; without hints, LSTM set 337 / 349 / 342 / 334.)
template <bool kNt, bool kMom, uint32_t kAhead, typename F>
__device__ __forceinline__ void stream_groups(gcvf4 G4, gvf4 V4, gvf4 U4, uint32_t groups, F&& f) {
  const uint32_t lane = lane_id();
  vf4 g[kAhead], v[kAhead], u[kAhead];
  auto load = [&](uint32_t t, uint32_t at) __attribute__((always_inline)) {
    const uint32_t o = at * kWaveSize + lane;
    g[t] = __builtin_nontemporal_load(&G4[o]);
    v[t] = stream_load<kNt>(V4 + o);
    if constexpr (kMom) u[t] = stream_load<kNt>(U4 + o);
  };
#pragma unroll
  for (uint32_t t = 0; t < kAhead; ++t)
    if (t < groups) load(t, t);
  for (uint32_t g0 = 0; g0 < groups; g0 += kAhead) {
#pragma unroll
    for (uint32_t t = 0; t < kAhead; ++t) {
      const uint32_t at = g0 + t;
      if (at < groups) {
        const float gg[4] = {g[t].x, g[t].y, g[t].z, g[t].w}, vv[4] = {v[t].x, v[t].y, v[t].z, v[t].w};
        float uu[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (kMom) { uu[0] = u[t].x; uu[1] = u[t].y; uu[2] = u[t].z; uu[3] = u[t].w; }
        f(gg, vv, uu, at * kWaveSize + lane, [&]() __attribute__((always_inline)) { if (at + kAhead < groups) load(t, at + kAhead); });
      }
    }
  }
}

// The zeros that mask a sent entry out of the residual (and the velocity) are isolated 4-byte
// writes, one cache line in a thousand.  Left dirty in the caches they are written to DRAM one
// by one while the next streaming pass runs and cost it about a tenth of its bandwidth; stored
// with the streaming hint they leave the caches early and cost half of that.
__device__ __forceinline__ void mask_store(gptr<float> p) { __builtin_nontemporal_store(0.0f, p); }

}  // namespace rgc
