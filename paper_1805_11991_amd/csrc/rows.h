#pragma once
// Row steps shared by the bucketing kernels: the dense translate of a row
// (shift_kernel in kernels.hip says which and why), its pattern, and counts
// per pattern.
#include <hip/hip_runtime.h>

#include "count_core.h"
#include "plan.h"

namespace hwc {

// hist[pat] += 1 for every active lane, one LDS atomic per distinct pattern in
// the wave (rows of a wave mostly share one or two patterns, so per-lane
// atomics would serialize on the same address).
__device__ __forceinline__ void wave_count(uint32_t* hist, uint32_t pat, bool active) {
  uint64_t left = __ballot(active);
  while (left) {
    const uint32_t leader = uniform((uint32_t)__builtin_amdgcn_readlane((int)pat, (int)__builtin_ctzll(left)));
    const uint64_t same = __ballot(active && pat == leader);
    if ((threadIdx.x & (kWave - 1)) == (uint32_t)__builtin_ctzll(left)) atomicAdd(&hist[leader], (uint32_t)__popcll(same));
    left &= ~same;
  }
}

// The pattern of a row (plan.h) and its error bits: 1 for a code outside
// [0, q), 2 for a degree below 2g + 1.
template <int NC>
__device__ __forceinline__ uint32_t row_pattern(const int (&o)[NC], uint32_t q, bool live, uint32_t& bad) {
  uint32_t mask = 0;
  const uint32_t d = o[NC - 1] ? NC - 1 : NC - 2;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    if (live && (o[i] < 0 || o[i] >= (int)q)) bad |= 1u;
    if ((uint32_t)i < d && o[i] != 0) mask |= 1u << i;
  }
  if (live && o[NC - 1] == 0 && o[NC - 2] == 0) bad |= 2u;
  return (o[NC - 1] ? (1u << (NC - 1)) : 0u) | mask;
}

// The row's dense translate into w, when it has one and needs one (returned);
// every lane of a wave takes part (ballots).  tmat: the packed matrix rows
// (DOT, prime q); tab: the step table in LDS.
template <int NC, typename CT, bool DOT>
__device__ __forceinline__ bool translate_row(const CT (&raw)[NC], bool live, uint32_t q, uint32_t qm,
                                              const uint32_t* __restrict__ tmat, const uint8_t* tab,
                                              uint32_t (&w)[NC]) {
  constexpr uint32_t NW = shift_tmat_row_words(NC);
  const uint32_t qq = q * q;
  uint32_t c[NC];
  bool valid = live;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int v = (int)raw[i];
    valid = valid && v >= 0 && v < (int)q;
    c[i] = (v >= 0 && v < (int)q) ? (uint32_t)v : 0u;
  }
  const uint32_t d = c[NC - 1] ? NC - 1 : NC - 2;
  bool need = false;
#pragma unroll
  for (int i = 0; i < NC - 1; ++i) need = need || ((uint32_t)i < d && c[i] == 0);
  need = need && valid && c[d] != 0;
  bool done = false;
#pragma unroll
  for (int i = 0; i < NC; ++i) w[i] = c[i];
  uint32_t cp[NW];
  if constexpr (DOT) {
#pragma unroll
    for (uint32_t x = 0; x < NW; ++x) {
      uint32_t word = 0;
#pragma unroll
      for (uint32_t b = 0; b < 4; ++b)
        if (4 * x + b < (uint32_t)NC) word |= c[4 * x + b] << (8 * b);
      cp[x] = word;
    }
  }
  for (uint32_t t = 1; t < q && t <= kShiftTries; ++t) {
    if (!__ballot(need && !done)) break;
    uint32_t v[NC];
    if constexpr (DOT) {
      const uint32_t* Tt = tmat + t * shift_tmat_words(NC);
#pragma unroll
      for (int i = 0; i < NC - 1; ++i) {
        uint32_t acc = 0;
#pragma unroll
        for (uint32_t x = (uint32_t)i / 4; x < NW; ++x)
          acc = __builtin_amdgcn_udot4(Tt[i * NW + x], cp[x], acc, false);
        v[i] = acc - __umul24(q, __umul24(acc, qm) >> 20);   // 24-bit products, full rate
      }
      v[NC - 1] = c[NC - 1];
    } else {
      const uint32_t base = t * qq;
#pragma unroll
      for (int i = 0; i < NC; ++i) v[i] = c[i];
#pragma unroll
      for (int k = 0; k < NC - 1; ++k) {
#pragma unroll
        for (int i = NC - 2; i >= k; --i) v[i] = tab[base + v[i] * q + v[i + 1]];
      }
    }
    bool dense = true;
#pragma unroll
    for (int i = 0; i < NC - 1; ++i) dense = dense && ((uint32_t)i >= d || v[i] != 0);
    if (need && !done && dense) {
#pragma unroll
      for (int i = 0; i < NC; ++i) w[i] = v[i];
      done = true;
    }
  }
  return done;
}

}  // namespace hwc
