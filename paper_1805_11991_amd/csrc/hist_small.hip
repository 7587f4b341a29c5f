// Histogram of a small request in one workgroup: keys, radix sort, run
// lengths and decoding in LDS, one launch for any number of requests (one
// workgroup each), where hist.hip's passes take about 17 launches a request.
//
// What bounds it is latency: the chain of barriers and LDS round trips of one
// workgroup, about 1 us a digit.  A request of 500 curves (g = 3, q = 13) went
// from 17 launches (199 us for the whole call) to one of 9 us (146 us); the
// histograms of 71 requests of 8192 curves from 1180 launches (12.0 ms for the
// whole batch) to one of 38 us (7.2 ms).  Past 8192 rows, where a workgroup's
// LDS ends, many workgroups a pass win again.
//
// The key packs the columns into bit fields (N_1 most significant), so that
// decoding is shifts: sum over k of the bits of 2 q^k + 2, plus the
// partition's rank, must be at most 64, which the callers check.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan.h"

namespace hwc {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr uint32_t kBins = 256;            // 8-bit digits
constexpr int kMaxItems = kHistSmallMax / kThreads;

struct Shared {
  uint64_t key[kHistSmallMax];
  uint32_t run[kWaves][kBins];             // a wave's count per digit, then its start; after the sort, run starts
  uint32_t wsum[kWaves];
  uint32_t total;
};
static_assert(sizeof(uint16_t) * kHistSmallMax <= sizeof(Shared::run), "run starts fit the digit counters");

__device__ __forceinline__ uint32_t wave_inclusive(uint32_t v) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (uint32_t off = 1; off < kWave; off <<= 1) {
    const uint32_t a = (uint32_t)__shfl_up((int)v, off);
    v += lane >= off ? a : 0u;
  }
  return v;
}

// lanes of the wave with the same digit (the valid ones)
__device__ __forceinline__ uint64_t same_digit(bool valid, uint32_t dig) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const uint64_t ones = __ballot(((dig >> b) & 1u) != 0);
    peers &= ((dig >> b) & 1u) ? ones : ~ones;
  }
  return peers;
}

// Bits of the field of column k: N_k takes values 0 .. 2 q^k + 2.
__device__ __forceinline__ uint32_t field_bits(uint32_t top) { return 32u - (uint32_t)__builtin_clz(top); }

// I keys per thread: wave w holds keys w 64 I .. in rounds of 64, so index
// order is wave, round, lane and the ranking below keeps the sort stable.
template <int I, bool LAM>
__device__ void hist_one(const HistJob& J, const LamCodes* __restrict__ lc, Shared& sh, uint32_t* __restrict__ err) {
  const uint32_t t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  const uint32_t n = J.n, g = J.g, width = g + (LAM ? 1u : 0u);
  uint32_t top[4], bits[4], nbits = 0;
  uint32_t qk = 1;
  for (uint32_t k = 0; k < 4; ++k) {
    qk = k < g ? qk * J.q : qk;
    top[k] = 2u * qk + 2u;
    bits[k] = k < g ? field_bits(top[k]) : 0u;
    nbits += bits[k];
  }
  const uint32_t lbits = LAM ? field_bits(lc->n) : 0u;
  nbits += lbits;
  const uint32_t first = wave * (kWave * I) + lane;
  uint64_t key[I];
  bool bad = false;
#pragma unroll
  for (int r = 0; r < I; ++r) {
    const uint32_t i = first + r * kWave;
    uint64_t k64 = 0;
    if (i < n) {
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        if (k >= g) break;
        int32_t v = J.N[(uint64_t)i * g + k];
        if (v < 0 || (uint32_t)v > top[k]) { bad = true; v = 0; }
        k64 = (k64 << bits[k]) | (uint32_t)v;
      }
      if (LAM) {
        const uint32_t v = J.lam[i];
        uint32_t rk = lc->slot[(v * lc->mul) >> 24];          // rank + 1 of the code in v's slot
        if (rk == 0 || lc->code[rk - 1] != v) { bad = true; rk = 1; }
        k64 = (k64 << lbits) | (rk - 1);
      }
    }
    key[r] = k64;
  }
  if (bad) atomicOr(err, 4u);
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  for (uint32_t shift = 0; shift < nbits; shift += 8) {
    for (uint32_t d = t; d < kWaves * kBins; d += kThreads) (&sh.run[0][0])[d] = 0;
    __syncthreads();
    uint32_t rank[I];
#pragma unroll
    for (int r = 0; r < I; ++r) {
      const bool valid = first + r * kWave < n;
      const uint32_t dig = (uint32_t)(key[r] >> shift) & (kBins - 1);
      const uint64_t peers = same_digit(valid, dig);
      // every lane reads the wave's count before its leader adds the round's
      // keys (one wave: LDS operations complete in issue order)
      const uint32_t before = valid ? sh.run[wave][dig] : 0u;
      const uint32_t below = (uint32_t)__popcll(peers & lt);
      __builtin_amdgcn_wave_barrier();
      if (valid && below == 0) sh.run[wave][dig] = before + (uint32_t)__popcll(peers);
      __builtin_amdgcn_wave_barrier();
      rank[r] = before + below;
    }
    __syncthreads();
    // starts: digits in order, the waves of a digit in order
    uint32_t c[kWaves], sum = 0;
    if (t < kBins) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        c[w] = sh.run[w][t];
        sum += c[w];
      }
    }
    const uint32_t incl = wave_inclusive(sum);
    if (t < kBins && lane == kWave - 1) sh.wsum[wave] = incl;
    __syncthreads();
    if (t < kBins) {
      uint32_t at = incl - sum;
      for (uint32_t w = 0; w < wave; ++w) at += sh.wsum[w];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        sh.run[w][t] = at;
        at += c[w];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < I; ++r)
      if (first + r * kWave < n) sh.key[sh.run[wave][(uint32_t)(key[r] >> shift) & (kBins - 1)] + rank[r]] = key[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < I; ++r)
      if (first + r * kWave < n) key[r] = sh.key[first + r * kWave];
  }
  // run heads in index order: a wave's rounds in turn, ballots within one
  uint64_t heads[I];
  uint32_t mine = 0;
#pragma unroll
  for (int r = 0; r < I; ++r) {
    const uint32_t i = first + r * kWave;
    heads[r] = __ballot(i < n && (i == 0 || sh.key[i - 1] != key[r]));
    mine += (uint32_t)__popcll(heads[r]);
  }
  if (lane == 0) sh.wsum[wave] = mine;
  __syncthreads();
  uint32_t at = 0, runs = 0;
  for (uint32_t w = 0; w < kWaves; ++w) {
    const uint32_t s = sh.wsum[w];
    at += w < wave ? s : 0u;
    runs += s;
  }
  uint16_t* start = reinterpret_cast<uint16_t*>(&sh.run[0][0]);
#pragma unroll
  for (int r = 0; r < I; ++r) {
    if ((heads[r] >> lane) & 1ull) start[at + (uint32_t)__popcll(heads[r] & lt)] = (uint16_t)(first + r * kWave);
    at += (uint32_t)__popcll(heads[r]);
  }
  __syncthreads();
  for (uint32_t j = t; j < runs && j < J.cap; j += kThreads) {
    const uint32_t i = start[j], end = j + 1 < runs ? start[j + 1] : n;
    J.counts[j] = end - i;
    uint64_t k64 = sh.key[i];
    if (LAM) {
      J.keys[(uint64_t)j * width + g] = (int32_t)lc->code[(uint32_t)k64 & ((1u << lbits) - 1u)];
      k64 >>= lbits;
    }
#pragma unroll
    for (int k = 3; k >= 0; --k) {
      if ((uint32_t)k >= g) continue;
      J.keys[(uint64_t)j * width + k] = (int32_t)((uint32_t)k64 & (uint32_t)((1ull << bits[k]) - 1ull));
      k64 >>= bits[k];
    }
  }
  if (t == 0 && J.len) *J.len = runs;
}

template <bool LAM>
__device__ __forceinline__ void hist_any(const HistJob& J, const LamCodes* lc, Shared& sh, uint32_t* err) {
  if (J.n <= kThreads) hist_one<1, LAM>(J, lc, sh, err);
  else if (J.n <= 2 * kThreads) hist_one<2, LAM>(J, lc, sh, err);
  else if (J.n <= 4 * kThreads) hist_one<4, LAM>(J, lc, sh, err);
  else hist_one<kMaxItems, LAM>(J, lc, sh, err);
}

extern __shared__ uint64_t hist_lds[];

__global__ __launch_bounds__(kThreads) void hist_small_kernel(HistJob J, uint32_t* __restrict__ err) {
  hist_any<false>(J, nullptr, *reinterpret_cast<Shared*>(hist_lds), err);
}

__global__ __launch_bounds__(kThreads) void hist_small_lambda_kernel(HistJob J, LamCodes lc, uint32_t* __restrict__ err) {
  hist_any<true>(J, &lc, *reinterpret_cast<Shared*>(hist_lds), err);
}

__global__ __launch_bounds__(kThreads) void hist_small_batch_kernel(const HistJob* __restrict__ jobs,
                                                                    uint32_t* __restrict__ err) {
  hist_any<false>(jobs[blockIdx.x], nullptr, *reinterpret_cast<Shared*>(hist_lds), err);
}

}  // namespace

// Whether a request's histogram is taken by one workgroup: at most
// kHistSmallMax rows and a key of bit fields within 64 bits, for a key space that
// hist_run accepts (2^63 keys: at q = 61, g = 4 the fields fit, the space does not).
bool hist_is_small(uint64_t n, uint32_t g, uint32_t q, bool lam) {
  if (n == 0 || n > kHistSmallMax) return false;
  const uint32_t codes = lam ? lam_code_list(g, nullptr) : 0u;
  uint32_t bits = lam ? 32u - (uint32_t)__builtin_clz(codes) : 0u;
  unsigned __int128 space = lam ? codes : 1u;
  uint64_t qk = 1;
  for (uint32_t k = 0; k < g; ++k) {
    qk *= q;
    if (qk > (1u << 24)) return false;
    bits += 32u - (uint32_t)__builtin_clz((uint32_t)(2 * qk + 2));
    space *= 2 * qk + 3;
  }
  return bits <= 64 && space <= (unsigned __int128)1 << 63;
}

hipError_t launch_hist_small(const HistJob& J, const LamCodes* lc, uint32_t* err, hipStream_t s) {
  if (J.n == 0 || J.n > kHistSmallMax) return hipErrorInvalidValue;
  if (lc) hipLaunchKernelGGL(hist_small_lambda_kernel, dim3(1), dim3(kThreads), sizeof(Shared), s, J, *lc, err);
  else hipLaunchKernelGGL(hist_small_kernel, dim3(1), dim3(kThreads), sizeof(Shared), s, J, err);
  return hipGetLastError();
}

// One workgroup per job (device descriptors, each as hist_is_small accepts).
hipError_t launch_hist_small_batch(const HistJob* jobs, uint32_t njobs, uint32_t* err, hipStream_t s) {
  if (njobs == 0) return hipSuccess;
  hipLaunchKernelGGL(hist_small_batch_kernel, dim3(njobs), dim3(kThreads), sizeof(Shared), s, jobs, err);
  return hipGetLastError();
}

hipError_t prepare_hist_small() {
  hipError_t e = hipSuccess;
  for (const void* f : {reinterpret_cast<const void*>(&hist_small_kernel),
                        reinterpret_cast<const void*>(&hist_small_lambda_kernel),
                        reinterpret_cast<const void*>(&hist_small_batch_kernel)})
    if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(Shared));
  return e;
}

}  // namespace hwc
