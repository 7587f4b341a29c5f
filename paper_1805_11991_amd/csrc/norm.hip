// The count of one genus 2 request whose plan has norm tables (norm_impl.h): as
// count_kernel, without the code of the other table forms, so that its waves
// keep few registers: 74, or 64 in the build for images of at most 80 KB, where
// two workgroups of 16 waves fit a CU (with four points a pass instead of
// eight; count of 2^18 curves at q = 101 0.87 -> 0.80 ms, 121 1.45 -> 1.20).
#include <hip/hip_runtime.h>

#include "norm_impl.h"
#include "plan.h"

namespace hwc {
namespace {

template <typename CT, int WPE, int PAIR>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(WPE))) void norm_kernel(const PlanDesc* __restrict__ Pd, const CT* __restrict__ codes,
                                                    const uint32_t* __restrict__ perm,
                                                    const uint64_t* __restrict__ tiles,
                                                    const uint32_t* __restrict__ ntiles_p, uint32_t* queue,
                                                    int32_t* __restrict__ outN, uint32_t* __restrict__ outLv,
                                                    uint32_t plog, uint32_t* __restrict__ acc,
                                                    uint32_t* __restrict__ done) {
  const PlanDesc& P = *Pd;
  extern __shared__ uint32_t lds32[];
  uint32_t* taken = lds32 + P.image_bytes / 4;
  stage_image(lds32, P.image, P.image_bytes);
  if (threadIdx.x < 2) taken[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t entries = *ntiles_p << plog;     // tiles, or the 2^plog parts of every tile
  const EntryShare share = entry_share(taken, queue, entries);
  for (;;) {
    const uint32_t t = next_entry(share);
    if (t >= entries) break;
    norm_tile<CT, WPE == 8 ? 4 : 8, PAIR>(P, codes, perm, sload64(tiles, t >> plog), outN, outLv, t >> plog, t & ((1u << plog) - 1u), plog, acc,
                  done);
  }
}

// Images that leave room for a second workgroup on the CU: worth the build of
// 8 waves a SIMD.
bool two_blocks(uint32_t image_bytes) { return image_bytes + 16 <= 80 * 1024; }

}  // namespace

hipError_t launch_norm(const PlanDesc& P, const PlanDesc* dP, int coeff_bytes, const void* codes, const uint32_t* perm,
                       const uint64_t* tiles, const uint32_t* ntiles, uint32_t* queue, int32_t* outN, uint32_t* outLv,
                       uint32_t plog, uint32_t* acc, uint32_t* done, uint32_t grid, uint32_t block, hipStream_t s) {
  if (P.g != 2 || !P.norm.kind || P.image_bytes > kLdsImageLimit) return hipErrorInvalidValue;
#define HWC_NORM(CT, W, PR)                                                                                  \
  hipLaunchKernelGGL((norm_kernel<CT, W, PR>), dim3(grid), dim3(block), P.image_bytes + 16, s, dP,                 \
                     static_cast<const CT*>(codes), perm, tiles, ntiles, queue, outN, outLv, plog, acc, done)
#define HWC_NORM_W(CT, W)               \
  do {                                  \
    if (P.norm.pair) HWC_NORM(CT, W, 1); \
    else HWC_NORM(CT, W, 0);             \
  } while (0)
  if (two_blocks(P.image_bytes)) {
    if (coeff_bytes == 1) HWC_NORM_W(int8_t, 8);
    else HWC_NORM_W(int16_t, 8);
  } else {
    if (coeff_bytes == 1) HWC_NORM_W(int8_t, 4);
    else HWC_NORM_W(int16_t, 4);
  }
#undef HWC_NORM_W
#undef HWC_NORM
  return hipGetLastError();
}

hipError_t occupancy_norm(bool pair, uint32_t block, uint32_t lds_bytes, int* blocks_per_cu) {
  const void* f = two_blocks(lds_bytes) ? (pair ? reinterpret_cast<const void*>(&norm_kernel<int16_t, 8, 1>)
                                                : reinterpret_cast<const void*>(&norm_kernel<int16_t, 8, 0>))
                                        : (pair ? reinterpret_cast<const void*>(&norm_kernel<int16_t, 4, 1>)
                                                : reinterpret_cast<const void*>(&norm_kernel<int16_t, 4, 0>));
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, f, block, lds_bytes + 16);
}

// The whole image budget, and no static LDS (the rows start at LDS address 0).
hipError_t prepare_norm() {
  hipError_t e = hipSuccess;
  for (const void* f : {reinterpret_cast<const void*>(&norm_kernel<int8_t, 4, 0>),
                        reinterpret_cast<const void*>(&norm_kernel<int16_t, 4, 0>),
                        reinterpret_cast<const void*>(&norm_kernel<int8_t, 8, 0>),
                        reinterpret_cast<const void*>(&norm_kernel<int16_t, 8, 0>),
                        reinterpret_cast<const void*>(&norm_kernel<int8_t, 4, 1>),
                        reinterpret_cast<const void*>(&norm_kernel<int16_t, 4, 1>),
                        reinterpret_cast<const void*>(&norm_kernel<int8_t, 8, 1>),
                        reinterpret_cast<const void*>(&norm_kernel<int16_t, 8, 1>)}) {
    if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsImageLimit + 16);
    hipFuncAttributes a{};
    if (e == hipSuccess) e = hipFuncGetAttributes(&a, f);
    if (e == hipSuccess && a.sharedSizeBytes != 0) e = hipErrorInvalidKernelFile;
  }
  return e;
}

}  // namespace hwc
