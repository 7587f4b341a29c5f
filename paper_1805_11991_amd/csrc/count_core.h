#pragma once
// Reads shared by the counting kernels: LDS at absolute addresses, uniform
// data through scalar loads.
#include <hip/hip_runtime.h>

#include "plan.h"

namespace hwc {

// LDS reads at absolute LDS byte addresses.  The count and batch kernels
// declare no static LDS, so their dynamic block -- the table image -- starts
// at address 0 (prepare_kernels checks this on the host), and a table step is
// one add and one read with no base to add.
typedef const __attribute__((address_space(3))) uint16_t* lds16_ptr;
typedef const __attribute__((address_space(3))) uint32_t* lds32_ptr;
__device__ __forceinline__ uint32_t lds_u16(uint32_t addr) { return *(lds16_ptr)(size_t)addr; }
__device__ __forceinline__ uint32_t lds_u32(uint32_t addr) { return *(lds32_ptr)(size_t)addr; }
constexpr uint32_t kImageBase = 0;   // LDS address of the dynamic block

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Uniform reads of data no kernel writes while it runs (x lists, tile words):
// through the constant address space they become scalar loads instead of
// vector loads that stall the wave on a full memory round trip.
typedef const __attribute__((address_space(4))) uint32_t* const_u32_ptr;
typedef const __attribute__((address_space(4))) uint64_t* const_u64_ptr;
__device__ __forceinline__ uint32_t sload(const uint32_t* p, uint32_t i) { return ((const_u32_ptr)p)[i]; }
__device__ __forceinline__ uint64_t sload64(const uint64_t* p, uint32_t i) { return ((const_u64_ptr)p)[i]; }
__device__ __forceinline__ LevelDesc load_level(const PlanDesc& P, uint32_t j) {
  static_assert(sizeof(LevelDesc) % 4 == 0, "LevelDesc is copied in dwords");
  LevelDesc L;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(&P.lv[j]);
  uint32_t* dst = reinterpret_cast<uint32_t*>(&L);
#pragma unroll
  for (uint32_t i = 0; i < sizeof(LevelDesc) / 4; ++i) dst[i] = sload(src, i);
  return L;
}

// The plan's norm tables (genus 2), read like a level descriptor.
__device__ __forceinline__ NormDesc load_norm(const PlanDesc& P) {
  static_assert(sizeof(NormDesc) % 4 == 0, "NormDesc is copied in dwords");
  NormDesc D;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(&P.norm);
  uint32_t* dst = reinterpret_cast<uint32_t*>(&D);
#pragma unroll
  for (uint32_t i = 0; i < sizeof(NormDesc) / 4; ++i) dst[i] = sload(src, i);
  return D;
}

// Copies a plan's image to the start of the dynamic LDS block, 16 bytes a lane.
__device__ __forceinline__ void stage_image(uint32_t* lds, const uint32_t* __restrict__ image, uint32_t bytes) {
  const uint4* src = reinterpret_cast<const uint4*>(image);
  uint4* dst = reinterpret_cast<uint4*>(lds);
  for (uint32_t i = threadIdx.x; i < bytes / 16; i += blockDim.x) dst[i] = src[i];
}

// N_k from the per-level counts (Sec. 1.1 decomposition; x = 0 and the
// points at infinity of the model in P(1, g+1, 1) added here).
template <int G>
__device__ __forceinline__ void assemble(const PlanDesc& P, const uint32_t (&lv)[G], uint32_t c0, uint32_t ctop,
                                         uint32_t log0, uint32_t logtop, int32_t* out) {
#pragma unroll
  for (int k = 1; k <= G; ++k) {
    const int chi0 = (k % 2 == 0) ? 1 : ((log0 & 1u) ? -1 : 1);
    const int chit = (k % 2 == 0) ? 1 : ((logtop & 1u) ? -1 : 1);
    int32_t n = (c0 == 0 ? 1 : 1 + chi0) + (ctop == 0 ? 1 : 1 + chit);
    if (P.orbit) {
#pragma unroll
      for (int j = 1; j <= G; ++j) {
        if (k % j) continue;
        const uint32_t z = lv[j - 1] & 0xFFu, ns = lv[j - 1] >> 8;
        const uint32_t s = P.lv[j - 1].nx - z - ns;
        const uint32_t sq = ((k / j) % 2 == 0) ? s + ns : s;
        n += (int32_t)(j * z + 2 * j * sq);
      }
    } else {
      const uint32_t z = lv[k - 1] & 0xFFu, ns = lv[k - 1] >> 8;
      const uint32_t s = P.lv[k - 1].nx - z - ns;
      n += (int32_t)(z + 2 * s);
    }
    out[k - 1] = n;
  }
}

// The end of one tile's (or part's) sweep: with parts (plog > 0) the counts are
// added up in acc and the tile's last part reads the sums back; then N is
// assembled (outN) and the level counts are written (outLv), each if given.
// c0, ctop, log0, logtop: the row's lowest and highest codes and their logs in
// F_q.
template <int G>
__device__ __forceinline__ void finish_tile(const PlanDesc& P, uint32_t c0, uint32_t ctop, uint32_t log0,
                                            uint32_t logtop, uint32_t (&lv)[G], bool live, uint32_t curve, uint32_t lvl_lo,
                                            uint32_t lvl_hi, int32_t* __restrict__ outN, uint32_t* __restrict__ outLv,
                                            uint32_t tile, uint32_t plog, uint32_t* __restrict__ acc,
                                            uint32_t* __restrict__ done) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  if (plog) {
    // packed counts add without carries: a level's zeros stay below 256
    if (live) {
#pragma unroll
      for (int k = 0; k < G; ++k)
        if (lv[k]) atomicAdd(acc + (uint64_t)curve * G + k, lv[k]);
    }
    // Parts of a tile meet through device-scope atomics only (adds above, the
    // loads below), which no L2 holds back, so it is enough that this wave's
    // adds are done before it counts itself: a wait, not a fence, which
    // writes back the L2 for every part (g = 3, q = 13, 2^16 curves: 261 us
    // with the fences, 191 without)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint32_t prior = 0;
    if (lane == 0) prior = atomicAdd(done + tile, 1u);
    if (uniform(prior) != (1u << plog) - 1u) return;
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < G; ++k)
      lv[k] = __hip_atomic_load(acc + (uint64_t)curve * G + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  if (outN) {
    int32_t n[G];
    assemble<G>(P, lv, c0, ctop, log0, logtop, n);
    if (live) {
#pragma unroll
      for (int k = 0; k < G; ++k) outN[(uint64_t)curve * G + k] = n[k];
    }
  }
  if (outLv && live) {
#pragma unroll
    for (int j = 0; j < G; ++j)
      if ((uint32_t)j >= lvl_lo && (uint32_t)j <= lvl_hi) outLv[(uint64_t)curve * G + j] = lv[j];
  }
}

}  // namespace hwc
