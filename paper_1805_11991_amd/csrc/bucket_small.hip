// The bucketing of a small request in one workgroup: dense translates,
// patterns, the tile list and the permutation (what shift_kernel,
// classify_kernel, bucket_scan_kernel, tile_fill_kernel and scatter_kernel do
// in five or six launches of 4-10 us), and the part counters cleared, one
// launch for any number of requests.
//
// Latency bounds it (one workgroup per request, a few barriers): 9 us
// at 500 rows (146 -> 140 us a call), 110 us for 71 requests of 8192 rows at once
// (their 355 launches took about 1.6 ms of 7.2).  Past 8192 rows a request has work for many workgroups a pass.
#include <hip/hip_runtime.h>

#include "plan.h"
#include "rows.h"

namespace hwc {
namespace {

constexpr int kThreads = 1024;
constexpr uint32_t kPatterns = 1u << kMaxCoef;   // 2048

struct Shared {
  uint32_t cnt[kPatterns];        // rows per pattern; later the pattern's next place
  uint32_t start[kPatterns + 1];  // first row | first tile << 16, exclusive
  uint32_t wsum[kThreads / kWave];
  uint16_t pid[kBucketSmallMax];
  uint32_t step[(27 * 27 * 27 + 15) / 16 * 4];   // prime powers up to 27: step[t][a][b] = a + t b
};
static_assert(kBucketSmallMax <= 8192, "row and tile counts are packed in 16 bits each");

template <int NC, typename CT, int MODE>   // MODE 0: rows as given; 1: translates, prime q; 2: by the step table
__device__ __forceinline__ void bucket_rows(const BucketJob& J, Shared& sh, uint32_t& bad) {
  const CT* __restrict__ in = static_cast<const CT*>(J.codes);
  CT* __restrict__ out = static_cast<CT*>(J.out);
  const uint32_t* __restrict__ tmat = MODE == 1 ? J.step + shift_tmat_offset_words(J.q) : nullptr;
  const uint32_t qm = ((1u << 20) + J.q - 1) / J.q;
  for (uint32_t base = 0; base < J.n; base += kThreads) {   // uniform: the row steps have ballots
    const uint32_t r = base + threadIdx.x;
    const bool live = r < J.n;
    CT raw[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) raw[i] = live ? in[(uint64_t)r * NC + i] : (CT)0;
    int o[NC];
    if constexpr (MODE) {
      uint32_t w[NC];
      const bool done = translate_row<NC, CT, MODE == 1>(raw, live, J.q, qm, tmat,
                                                         reinterpret_cast<const uint8_t*>(sh.step), w);
#pragma unroll
      for (int i = 0; i < NC; ++i) o[i] = done ? (int)w[i] : (int)raw[i];
      if (live) {
#pragma unroll
        for (int i = 0; i < NC; ++i) out[(uint64_t)r * NC + i] = (CT)o[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < NC; ++i) o[i] = (int)raw[i];
    }
    const uint32_t pat = row_pattern<NC>(o, J.q, live, bad);
    if (live) sh.pid[r] = (uint16_t)pat;
    wave_count(sh.cnt, pat, live);
  }
}

template <int NC, typename CT>
__device__ __forceinline__ void bucket_mode(const BucketJob& J, Shared& sh, uint32_t& bad) {
  if (J.mode == 1) bucket_rows<NC, CT, 1>(J, sh, bad);
  else if (J.mode == 2) bucket_rows<NC, CT, 2>(J, sh, bad);
  else bucket_rows<NC, CT, 0>(J, sh, bad);
}

__device__ void bucket_one(const BucketJob& J, Shared& sh, uint32_t* __restrict__ err) {
  const uint32_t t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  for (uint32_t i = t; i < kPatterns; i += kThreads) sh.cnt[i] = 0;
  if (J.mode == 2)
    for (uint32_t i = t; i < (J.q * J.q * J.q + 3) / 4; i += kThreads) sh.step[i] = J.step[i];
  for (uint32_t i = t; i < J.acc_words; i += kThreads) J.acc[i] = 0;
  __syncthreads();
  uint32_t bad = 0;
#define HWC_ROWS(GG)                                                   \
  case GG:                                                             \
    if (J.cb == 1) bucket_mode<2 * GG + 3, int8_t>(J, sh, bad);        \
    else bucket_mode<2 * GG + 3, int16_t>(J, sh, bad);                 \
    break;
  switch (J.g) {
    HWC_ROWS(1) HWC_ROWS(2) HWC_ROWS(3) HWC_ROWS(4)
    default: break;
  }
#undef HWC_ROWS
  if (bad) atomicOr(err, bad);
  __syncthreads();
  // exclusive scan of (rows, tiles) over the patterns, two to a thread
  const uint32_t c0 = sh.cnt[2 * t], c1 = sh.cnt[2 * t + 1];
  const uint32_t v0 = c0 | ((c0 + kWave - 1) / kWave) << 16, v1 = c1 | ((c1 + kWave - 1) / kWave) << 16;
  uint32_t incl = v0 + v1;
#pragma unroll
  for (uint32_t off = 1; off < kWave; off <<= 1) {
    const uint32_t a = (uint32_t)__shfl_up((int)incl, off);
    incl += lane >= off ? a : 0u;
  }
  if (lane == kWave - 1) sh.wsum[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t w = 0; w < wave; ++w) before += sh.wsum[w];
  const uint32_t s0 = before + incl - v0 - v1;
  sh.start[2 * t] = s0;
  sh.start[2 * t + 1] = s0 + v0;
  if (t == kThreads - 1) sh.start[kPatterns] = s0 + v0 + v1;
  sh.cnt[2 * t] = s0 & 0xFFFFu;
  sh.cnt[2 * t + 1] = (s0 + v0) & 0xFFFFu;
  __syncthreads();
  const uint32_t nt = sh.start[kPatterns] >> 16;
  for (uint32_t i = t; i < nt; i += kThreads) {
    uint32_t lo = 0, hi = kPatterns;   // the last pattern whose first tile is at most i: the one that holds it
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if ((sh.start[mid] >> 16) <= i) lo = mid; else hi = mid;
    }
    const uint32_t first = (sh.start[lo] & 0xFFFFu) + (i - (sh.start[lo] >> 16)) * kWave;
    const uint32_t left = (sh.start[lo + 1] & 0xFFFFu) - first;
    J.tiles[i] = tile_pack(lo, first, left < (uint32_t)kWave ? left : (uint32_t)kWave);
  }
  if (t == 0) {
    *J.ntiles = nt;
    *J.queue = 0;
  }
  // places: one LDS add per distinct pattern of a wave
  for (uint32_t base = wave * kWave; base < J.n; base += kThreads) {
    const uint32_t r = base + lane;
    const bool live = r < J.n;
    const uint32_t pat = live ? sh.pid[r] : 0u;
    uint64_t left = __ballot(live);
    while (left) {
      const uint32_t head = (uint32_t)__builtin_ctzll(left);
      const uint32_t leader = uniform((uint32_t)__builtin_amdgcn_readlane((int)pat, (int)head));
      const uint64_t same = __ballot(live && pat == leader);
      uint32_t at = 0;
      if (lane == head) at = atomicAdd(&sh.cnt[leader], (uint32_t)__popcll(same));
      at = (uint32_t)__builtin_amdgcn_readlane((int)at, (int)head);
      if (live && pat == leader)
        J.perm[at + (uint32_t)__popcll(same & (lane == 0 ? 0ull : (~0ull >> (kWave - lane))))] = r;
      left &= ~same;
    }
  }
}

extern __shared__ uint32_t bucket_lds[];

__global__ __launch_bounds__(kThreads) void bucket_small_kernel(BucketJob J, uint32_t* __restrict__ err) {
  bucket_one(J, *reinterpret_cast<Shared*>(bucket_lds), err);
}

__global__ __launch_bounds__(kThreads) void bucket_small_batch_kernel(const BucketJob* __restrict__ jobs,
                                                                      uint32_t* __restrict__ err) {
  bucket_one(jobs[blockIdx.x], *reinterpret_cast<Shared*>(bucket_lds), err);
}

hipError_t check(const BucketJob& J) {
  const bool ok = J.n <= kBucketSmallMax && J.g >= 1 && J.g <= (uint32_t)kMaxG && (J.cb == 1 || J.cb == 2) &&
                  (J.mode == 0 || (J.out && J.step && J.q <= (J.mode == 1 ? kShiftMaxQ : 27u)));
  return ok ? hipSuccess : hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_bucket_small(const BucketJob& J, uint32_t* err, hipStream_t s) {
  if (check(J) != hipSuccess) return hipErrorInvalidValue;
  hipLaunchKernelGGL(bucket_small_kernel, dim3(1), dim3(kThreads), sizeof(Shared), s, J, err);
  return hipGetLastError();
}

// hjobs: host copies of the njobs device descriptors
hipError_t launch_bucket_small_batch(const BucketJob* hjobs, const BucketJob* jobs, uint32_t njobs, uint32_t* err,
                                     hipStream_t s) {
  if (njobs == 0) return hipSuccess;
  for (uint32_t k = 0; k < njobs; ++k)
    if (check(hjobs[k]) != hipSuccess) return hipErrorInvalidValue;
  hipLaunchKernelGGL(bucket_small_batch_kernel, dim3(njobs), dim3(kThreads), sizeof(Shared), s, jobs, err);
  return hipGetLastError();
}

hipError_t prepare_bucket_small() {
  hipError_t e = hipSuccess;
  for (const void* f : {reinterpret_cast<const void*>(&bucket_small_kernel),
                        reinterpret_cast<const void*>(&bucket_small_batch_kernel)})
    if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(Shared));
  return e;
}

}  // namespace hwc
