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

}  // namespace hwc
