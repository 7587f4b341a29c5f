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

// How the waves of a persistent launch take its n entries.  With one queue in
// device memory for all of them every wave pops it once more than it has entries,
// 13 to 20 ns a pop: 8192 waves, 164 us, whatever the entries' work.  So the first
// round, or all of a request of at most two rounds, is each workgroup's own, every
// gridDim-th entry, taken through a word in LDS; the rest is common, and the first
// wave that finds it empty tells its workgroup.  Beyond twelve rounds everything
// is common: the pops of one round matter little, and waves that start apart
// overlap LDS and vector work better (g = 4, q = 13, 2^22 curves 20.39 -> 20.25
// ms).  Three quarters of the rounds as own entries would leave those of the
// workgroups that do not become resident at once for the end (2^24 curves at g =
// 3, q = 13: 7.77 -> 8.31 ms).  Count alone, one queue -> this: 20 000 curves at g =
// 2, q = 101 223 -> 75 us, 80 000 at g = 3, q = 13 209 -> 107.
struct EntryShare {
  uint32_t* taken;        // LDS: own entries taken; the common queue found empty
  uint32_t* queue;        // common entries taken (nullptr: every entry is some workgroup's own)
  uint32_t n, own;        // entries; a workgroup's own share
};

__device__ __forceinline__ EntryShare entry_share(uint32_t* lds, uint32_t* queue, uint32_t n) {
  EntryShare s{lds, queue, n, ~0u};
  const uint32_t wpb = blockDim.x / kWave;
  if (queue && n > 2u * gridDim.x * wpb) s.own = n > 12u * gridDim.x * wpb ? 0u : wpb;
  return s;
}

// The calling wave's next entry, or one past the last.
__device__ __forceinline__ uint32_t next_entry(const EntryShare& s) {
  const bool lead = (threadIdx.x & (kWave - 1)) == 0;
  uint32_t v = 0;
  if (lead) v = atomicAdd(s.taken, 1u);
  v = uniform(v);
  if (v < s.own) return v * gridDim.x + blockIdx.x;
  if (lead) {
    volatile uint32_t* empty = s.taken + 1;
    v = *empty ? s.n : s.own * gridDim.x + atomicAdd(s.queue, 1u);
    if (v >= s.n) *empty = 1u;
  }
  return uniform(v);
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
