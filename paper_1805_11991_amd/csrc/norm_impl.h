#pragma once
// Genus 2, level 2 by norms: the quadratic character of F_{q^2} read in F_q.
//
// Let delta be a nonsquare of F_q and F_{q^2} = F_q(sqrt delta).  Every
// Frobenius orbit of size 2 is {t + s sqrt delta, t - s sqrt delta}, so the
// orbits are the pairs (t, v) with t in F_q and v = s^2 delta a nonsquare of
// F_q.  With f(t + y) = sum_i b_i y^i,
//   f(t + s sqrt delta) = E + s sqrt delta O,
//   E = b_0 + b_2 v + b_4 v^2 + b_6 v^3,   O = b_1 + b_3 v + b_5 v^2,
// and chi(z) over F_{q^2} is chi of the norm N z = E^2 - v O^2 over F_q
// (z^((q^2-1)/2) = (z^(q+1))^((q-1)/2)).  So one point costs six Zech steps in
// F_q (three for E, two for O, one for the norm) instead of about three in
// F_{q^2}; but F_q's table has q - 1 entries instead of q^2 - 1, so each lane
// gets a copy of its own in its own LDS bank, and a read takes the 2 CU-clocks
// of a conflict-free one, not the 6.3 of a random gather, with no folding of
// half tables.  Count kernel on 2^18 curves against the level's own table:
// q = 293 (85 848 elements) 19.2 -> 5.7 ms, 241 5.7 -> 3.4, 169 3.2 -> 2.0,
// 101 1.31 -> 0.80, 37 0.24 -> 0.21.  Bound at q = 241: LDS 16.3 CU-clocks a
// point (five conflict-free reads and one of the byte table), 13.5 vector
// instructions, 17.7 measured; with the extra subtraction (q = 293) 17
// instructions and 19.9.
//
// One lane holds one curve, as everywhere in the count; t and v are uniform.
// Rows of the image (kNormRow bytes: one u32 per bank, all alike; M = q - 1):
//   0 .. Z - 1   128 Z(r mod M), or the marker S where 1 + gamma^r = 0
//   Z            0 (a vanished partial sum restarts from the next coefficient)
//   Z + 1 ..     2M rows that return their own index mod M (128 (r mod M)),
//                the last one the marker: the step of a zero coefficient,
//                which only multiplies by v
// (S: a power of two, at least 4M rows) with Z = 3M, or Z = 2M where 3M does not fit (fold: one more subtraction per
// step).  A step is a + delta + L, clamped to the row that a marker must
// reach (Z for a Zech step, the last row for a multiplication), and one read.
// A step's delta, clamp and fold are per lane, so the zero coefficients that
// some lane of nearly every translate has cost nothing.
//
// For primes q = 1 mod 4, v and -v are both nonsquares and share most of the
// work (norm_pairs): the norm itself is a polynomial of degree 6 in v,
//   N(v) = E^2 - v O^2 = sum_i n_i v^i = A(v^2) + v B(v^2),
//   A = n_0 + n_2 y + n_4 y^2 + n_6 y^3,   B = n_1 + n_3 y + n_5 y^2,
// so a pair costs three steps for A, two for B and one read of a byte table for
// both N(v) and N(-v): six reads for two points in place of six for one.  The
// n_i are integers, some 50 more vector instructions a translate.  A pair is 16
// vector instructions and 16.3 clocks of LDS; with the translates 22.4 and 17.1 at
// q = 293, in 21.6 CU-clocks: vector issue bounds it (1.04 instructions per CU and
// clock, LDS active 79 %).  Single points -> pairs, count with its bucketing: q =
// 293, 2^18 curves 5.83 -> 3.46 ms; 101, 500 001 curves 1.41 -> 1.01; 37, 2^18
// curves 250 -> 236 us.
//
// The last step of the other fields needs the parity of log(1 - v O^2 / E^2) only:
// w = log(-v) + 2 (log O - log E) mod M, so the sum d of the halves counts mod
// M / 2.  As it is taken, -M < d < 5M / 2, or past 3M when O = 0 (N = E^2, a
// square), or below -3M / 2 when E = 0 (N = -v O^2, of -v's parity): a byte
// table over -S <= d < S + 2M holds the answer for each.  Both zero is a root,
// found by a comparison.
#include <type_traits>

#include "count_core.h"

namespace hwc {

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t lds_u8(uint32_t addr) {
  return *(const __attribute__((address_space(3))) uint8_t*)(size_t)addr;
}

// floor(v m / 2^32) on 24-bit operands (v_mul_hi_u32_u24)
__device__ __forceinline__ uint32_t norm_mulhi24(uint32_t v, uint32_t m) {
  return (uint32_t)(((uint64_t)(v & 0xFFFFFFu) * (m & 0xFFFFFFu)) >> 32);
}

// One step's per-lane constants.
struct NormStep {
  uint32_t del, cap, fold;
};

// Links coefficient b (log, M = zero) below the chain whose last nonzero
// coefficient has log beta: the step's constants (rows scaled to bytes, the
// lane's bank included), and beta for the next one.
__device__ __forceinline__ NormStep norm_link(uint32_t& beta, uint32_t b, uint32_t M, uint32_t zrow, uint32_t lane4) {
  const bool z = b == M;
  const uint32_t d = beta >= b ? beta - b : beta + M - b;
  NormStep s;
  s.del = (z ? zrow + 1u : d) * kNormRow + lane4;
  s.cap = (z ? zrow + 2u * M : zrow) * kNormRow + lane4;
  s.fold = z ? 0u : M * kNormRow;
  beta = z ? beta : b;
  return s;
}

template <bool FOLD>
__device__ __forceinline__ uint32_t norm_step(uint32_t a, const NormStep& s, uint32_t L) {
  const uint32_t v = a + s.del + L;
  return lds_u32(FOLD ? min(min(v, v - s.fold), s.cap) : min(v, s.cap));
}

// U consecutive nonsquares v (logs L, L + 2, ..) at one t: odd logs of the
// norms into odd, roots into z.  kl: the lane's and the first v's terms of the
// last index, with the byte table's offset.
template <bool FOLD, bool TOP, int U>
__device__ __forceinline__ void norm_group(uint32_t L, uint32_t kl, const NormStep& e4, const NormStep& e2,
                                           const NormStep& e0, const NormStep& o3, const NormStep& o1, uint32_t S,
                                           uint32_t& odd, uint32_t& z) {
  uint32_t aE[U], aO[U], r[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t Lu = L + 2u * kNormRow * u;
    // the leading b_6 (degree 6) never vanishes, so its step cannot meet a
    // marker; the chains that start at b_5 or b_4 carry a vanished start in
    // their first delta
    if (TOP) aE[u] = norm_step<FOLD>(lds_u32(e4.del + Lu), e2, Lu);
    else aE[u] = lds_u32(min(e2.del + Lu, e2.cap));
    aO[u] = lds_u32(min(o3.del + Lu, o3.cap));
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t Lu = L + 2u * kNormRow * u;
    aE[u] = norm_step<FOLD>(aE[u], e0, Lu);
    aO[u] = norm_step<FOLD>(aO[u], o1, Lu);
  }
  uint32_t both = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    uint32_t x = aO[u] - aE[u] + kl;
    asm("" : "+v"(x));                 // one shift of the sum, not one per term
    r[u] = lds_u8(x / kNormRow + u);   // log(-v) / 2 grows by one per v
    odd += r[u];
    both |= aE[u] & aO[u];             // the marker is one bit above every row
  }
  if (__ballot(both >= S)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool root = (aE[u] & aO[u]) >= S;
      z += root;
      odd -= root ? r[u] : 0u;
    }
  }
}

// Every nonsquare v at one t: the chains of the translate's coefficients
// b[0..6] (logs, M = zero; b[6] = M in degree 5).
// U: nonsquares per pass of the inner loop.
template <bool FOLD, bool TOP, int U>
__device__ __forceinline__ void norm_sweep_v(const uint32_t (&b)[7], const NormDesc& D, uint32_t lane4,
                                             uint32_t& odd, uint32_t& z) {
  const uint32_t M = D.M, H = M / 2, S = D.srow * kNormRow, zrow = FOLD ? 2u * M : 3u * M;
  NormStep e4{}, e2, e0, o3, o1;
  uint32_t bE, bO;
  if (TOP) {
    bE = b[6];
    e4 = norm_link(bE, b[4], M, zrow, lane4);
    e2 = norm_link(bE, b[2], M, zrow, lane4);
  } else {
    bE = b[4] == M ? 0u : b[4];
    e2 = norm_link(bE, b[2], M, zrow, lane4);
    e2.del += b[4] == M ? S : 0u;
  }
  e0 = norm_link(bE, b[0], M, zrow, lane4);
  bO = b[5] == M ? 0u : b[5];
  o3 = norm_link(bO, b[3], M, zrow, lane4);
  o3.del += b[5] == M ? S : 0u;
  o1 = norm_link(bO, b[1], M, zrow, lane4);
  // v = gamma^(2k+1), k < H: log(-v) = H + 2k + 1, halved (its parity is
  // fixed); with log O - log E of the chains' bases, mod H
  uint32_t K = bO >= bE ? bO - bE : bO + M - bE;
  K = K >= H ? K - H : K;
  uint32_t L = kNormRow, kl = (K + (H + 1u) / 2u + D.fin_off + D.srow) * kNormRow, k = 0;
  for (; k + (uint32_t)U <= H; k += (uint32_t)U) {
    norm_group<FOLD, TOP, U>(L, kl, e4, e2, e0, o3, o1, S, odd, z);
    L += 2u * (uint32_t)U * kNormRow;
    kl += (uint32_t)U * kNormRow;
  }
  const uint32_t rest = H - k;
  if (U > 4 && (rest & 4u)) {
    norm_group<FOLD, TOP, 4>(L, kl, e4, e2, e0, o3, o1, S, odd, z);
    L += 8u * kNormRow;
    kl += 4u * kNormRow;
  }
  if (rest & 2u) {
    norm_group<FOLD, TOP, 2>(L, kl, e4, e2, e0, o3, o1, S, odd, z);
    L += 4u * kNormRow;
    kl += 2u * kNormRow;
  }
  if (rest & 1u) norm_group<FOLD, TOP, 1>(L, kl, e4, e2, e0, o3, o1, S, odd, z);
}

// U consecutive pairs v, -v at one t (y = v^2, logs L, L + 4, ..): the byte
// table's sums into acc (254 a zero), pairs with A = B = 0 into both.
template <bool FOLD, bool TOP, int U>
__device__ __forceinline__ void norm_pair_group(uint32_t L, uint32_t kl, const NormStep& e4, const NormStep& e2,
                                                const NormStep& e0, const NormStep& o3, const NormStep& o1, uint32_t S,
                                                uint32_t& acc, uint32_t& nboth) {
  uint32_t aA[U], aB[U], r[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t Lu = L + 4u * kNormRow * u;
    if (TOP) aA[u] = norm_step<FOLD>(lds_u32(e4.del + Lu), e2, Lu);
    else aA[u] = lds_u32(min(e2.del + Lu, e2.cap));
    aB[u] = lds_u32(min(o3.del + Lu, o3.cap));
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t Lu = L + 4u * kNormRow * u;
    aA[u] = norm_step<FOLD>(aA[u], e0, Lu);
    aB[u] = norm_step<FOLD>(aB[u], o1, Lu);
  }
  uint32_t both = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    uint32_t x = aB[u] - aA[u] + kl;
    asm("" : "+v"(x));                               // one shift of the sum
    r[u] = lds_u8((x / (kNormRow / 2) | (aA[u] / kNormRow & 1u)) + 4u * u);   // log v grows by two per pair
    acc += r[u];
    both |= aA[u] & aB[u];
  }
  if (__ballot(both >= S)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool root = (aA[u] & aB[u]) >= S;
      nboth += root;
      acc -= root ? r[u] : 0u;
    }
  }
}

// Every pair v, -v of nonsquares at one t (q = 1 mod 4), from the logs of
// n[0..6] (n[6] = M in degree 5).  The byte table is indexed by
// d = log(v B) - log A, counted as in norm_sweep_v, and by log A's parity in the
// rows, entry 2 (d + srow) + parity: the odd logs among A + vB and A - vB, plus
// 254 where one of the two vanishes.
template <bool FOLD, bool TOP, int U>
__device__ __forceinline__ void norm_sweep_pairs(const uint32_t (&n)[7], const NormDesc& D, uint32_t lane4,
                                                 uint32_t& odd, uint32_t& z) {
  const uint32_t M = D.M, S = D.srow * kNormRow, zrow = FOLD ? 2u * M : 3u * M;
  NormStep e4{}, e2, e0, o3, o1;
  uint32_t bA, bB;
  if (TOP) {
    bA = n[6];
    e4 = norm_link(bA, n[4], M, zrow, lane4);
    e2 = norm_link(bA, n[2], M, zrow, lane4);
  } else {
    bA = n[4] == M ? 0u : n[4];
    e2 = norm_link(bA, n[2], M, zrow, lane4);
    e2.del += n[4] == M ? S : 0u;
  }
  e0 = norm_link(bA, n[0], M, zrow, lane4);
  bB = n[5] == M ? 0u : n[5];
  o3 = norm_link(bB, n[3], M, zrow, lane4);
  o3.del += n[5] == M ? S : 0u;
  o1 = norm_link(bB, n[1], M, zrow, lane4);
  // v = gamma^(2k+1), k < M / 4; -v has the log M / 2 + 2k + 1
  const uint32_t K = bB >= bA ? bB - bA : bB + M - bA, P = M / 4;
  uint32_t L = 2u * kNormRow, kl = (K + 1u + D.srow) * kNormRow + D.fin_off * (kNormRow / 2), k = 0;
  uint32_t acc = 0, nboth = 0;
  for (; k + (uint32_t)U <= P; k += (uint32_t)U) {
    norm_pair_group<FOLD, TOP, U>(L, kl, e4, e2, e0, o3, o1, S, acc, nboth);
    L += 4u * (uint32_t)U * kNormRow;
    kl += 2u * (uint32_t)U * kNormRow;
  }
  const uint32_t rest = P - k;
  if (U > 4 && (rest & 4u)) {
    norm_pair_group<FOLD, TOP, 4>(L, kl, e4, e2, e0, o3, o1, S, acc, nboth);
    L += 16u * kNormRow;
    kl += 8u * kNormRow;
  }
  if (rest & 2u) {
    norm_pair_group<FOLD, TOP, 2>(L, kl, e4, e2, e0, o3, o1, S, acc, nboth);
    L += 8u * kNormRow;
    kl += 4u * kNormRow;
  }
  if (rest & 1u) norm_pair_group<FOLD, TOP, 1>(L, kl, e4, e2, e0, o3, o1, S, acc, nboth);
  // acc = odd + 254 zeros with odd <= M / 2 < 254 and at most 6 zeros (degree 6)
  const uint32_t z1 = __umul24(acc, 259u) >> 16, o = acc - 254u * z1, zt = z1 + 2u * nboth;
  odd += bA & 1u ? M / 2 - zt - o : o;    // the table counts from log A's rows: its base turns odd to even
  z += zt;
}

// Sum of two elements of F_q given as logs (M = zero), by the Zech rows; no
// branches, so the reads of one translate overlap.
__device__ __forceinline__ uint32_t norm_add(uint32_t M, uint32_t S, uint32_t lane4, uint32_t a, uint32_t b) {
  const bool az = a == M, bz = b == M;
  uint32_t d = b >= a ? b - a : b + M - a;
  d = (az || bz) ? 0u : d;
  const uint32_t v = lds_u32(d * kNormRow + lane4);
  uint32_t s = a + v / kNormRow;
  s = s >= M ? s - M : s;
  s = v == S ? M : s;
  return az ? b : (bz ? a : s);
}

// The counts of level 1 over the nonzero x = gamma^L, L in share `part` of
// 2^plog: f by one chain of the same steps as level 2's.
template <bool FOLD>
__device__ __forceinline__ uint32_t norm_level1(const NormDesc& D, const uint32_t (&w)[7], uint32_t lane4,
                                                uint32_t part, uint32_t plog) {
  const uint32_t M = D.M, S = D.srow * kNormRow, zrow = FOLD ? 2u * M : 3u * M;
  uint32_t beta = w[6] == M ? 0u : w[6];
  const uint32_t a0 = w[6] == M ? S : 0u;
  NormStep st[6];
#pragma unroll
  for (int i = 5; i >= 0; --i) st[i] = norm_link(beta, w[i], M, zrow, lane4);
  uint32_t odd = 0, z = 0;
  const uint32_t l1 = part_begin(M, part + 1u, plog);
  for (uint32_t l = part_begin(M, part, plog); l < l1; ++l) {
    const uint32_t L = l * kNormRow;
    uint32_t a = a0;
#pragma unroll
    for (int i = 5; i >= 0; --i) a = norm_step<FOLD>(a, st[i], L);
    const bool root = a >= S;
    z += root;
    odd += root ? 0u : ((a / kNormRow + beta) & 1u);
  }
  return z | (odd << 8);
}

// The counts of level 2 over the orbits (t, v), t in part `part` of 2^plog
// shares of F_q: roots | nonsquares << 8, as count_level returns them.
template <bool FOLD, bool TOP, bool PAIR, int U>
__device__ __forceinline__ uint32_t norm_level2(const NormDesc& D, const uint32_t (&code)[7], const uint32_t (&w)[7],
                                                uint32_t lane4, uint32_t part, uint32_t plog) {
  const uint32_t M = D.M, q = M + 1u;
  const uint32_t t0 = part_begin(q, part, plog), t1 = part_begin(q, part + 1u, plog);
  uint32_t odd = 0, z = 0;
  uint32_t pk[4];   // coefficient pairs for the integer translates
#pragma unroll
  for (int k = 0; k < 4; ++k) pk[k] = code[2 * k] | (k < 3 ? code[2 * k + 1 < 7 ? 2 * k + 1 : 6] << 16 : 0u);
#pragma unroll 1
  for (uint32_t t = t0; t < t1; ++t) {
    uint32_t b[7];
    b[6] = w[6];
    if (PAIR) {
      // the residues c_i of the translate (times 2^esh: s), as below, then the n_i
      // in the same scale, -c kept as q - c: each is at most 7 q M 2^esh
      uint32_t s[7], c[7], at = t * kNormTmatWords;
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        uint32_t acc = 0;
#pragma unroll
        for (int k = i / 2; k < 4; ++k)
          acc = __builtin_amdgcn_udot2(__builtin_bit_cast(ushort2_t, sload(D.tmat, at++)), __builtin_bit_cast(ushort2_t, pk[k]),
                                       acc, false);
        s[i] = acc - __umul24(norm_mulhi24(acc, D.qm), q << D.esh);
        c[i] = s[i] >> D.esh;
      }
      c[6] = code[6];
      s[6] = c[6] << D.esh;
      const uint32_t m1 = q - c[1], m3 = q - c[3], m5 = q - c[5];
      uint32_t n[6];
      n[0] = __umul24(s[0], c[0]);
      n[1] = __umul24(2u * s[0], c[2]) + __umul24(s[1], m1);
      n[2] = __umul24(2u * s[0], c[4]) + __umul24(2u * s[1], m3) + __umul24(s[2], c[2]);
      n[3] = __umul24(2u * s[0], c[6]) + __umul24(2u * s[2], c[4]) + __umul24(2u * s[1], m5) + __umul24(s[3], m3);
      n[4] = __umul24(2u * s[2], c[6]) + __umul24(2u * s[3], m5) + __umul24(s[4], c[4]);
      n[5] = __umul24(2u * s[4], c[6]) + __umul24(s[5], m5);
#pragma unroll
      for (int i = 0; i < 6; ++i) b[i] = lds_u32(D.emb_off + n[i] - __umul24(norm_mulhi24(n[i], D.qm), q << D.esh));
      b[6] = w[6] == M ? M : (2u * w[6] >= M ? 2u * w[6] - M : 2u * w[6]);   // n_6 = c_6^2
      norm_sweep_pairs<FOLD, TOP, U>(b, D, lane4, odd, z);
      continue;
    }
    if (D.tmat) {
      // prime q: b_i = sum_j binom(j, i) t^(j-i) c_j mod q by 2 x 16-bit dot
      // products with the uniform rows of t, whose entries come times the
      // bytes of a log's slot, so the scaled residue is its offset
      uint32_t at = t * kNormTmatWords;
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        uint32_t acc = 0;
#pragma unroll
        for (int k = i / 2; k < 4; ++k)
          acc = __builtin_amdgcn_udot2(__builtin_bit_cast(ushort2_t, sload(D.tmat, at++)), __builtin_bit_cast(ushort2_t, pk[k]),
                                       acc, false);
        b[i] = lds_u32(D.emb_off + acc - __umul24(norm_mulhi24(acc, D.qm), q << D.esh));
      }
    } else {
      // prime powers: repeated synthetic division by X - t in logs; t runs
      // over 0, 1, gamma, gamma^2, ..
#pragma unroll
      for (int i = 0; i < 6; ++i) b[i] = w[i];
      if (t) {
        const uint32_t lt = t - 1u;
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
          for (int i = 5; i >= k; --i) {
            uint32_t m = b[i + 1] + lt;
            m = m >= M ? m - M : m;
            b[i] = norm_add(M, D.srow * kNormRow, lane4, b[i], b[i + 1] == M ? M : m);
          }
      }
    }
    norm_sweep_v<FOLD, TOP, U>(b, D, lane4, odd, z);
  }
  return z | (odd << 8);
}

// One tile, or part `part` of 2^plog of it, as process_tile for a plan with
// norm tables.  PAIR: whether they are those of pairs (1, 0), or read from the
// plan (2).
template <typename CT, int U, int PAIR>
__device__ __forceinline__ void norm_tile(const PlanDesc& P, const CT* __restrict__ codes,
                                          const uint32_t* __restrict__ perm, uint64_t w, int32_t* __restrict__ outN,
                                          uint32_t* __restrict__ outLv, uint32_t tile, uint32_t part, uint32_t plog,
                                          uint32_t* __restrict__ acc, uint32_t* __restrict__ done) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t cnt = uniform((uint32_t)((w >> 16) & 0xFFFFu) + 1u);
  const uint32_t start = uniform((uint32_t)(w >> 32));
  const bool live = lane < cnt;                     // lanes past the end shadow the last curve
  const uint32_t curve = perm[start + (live ? lane : cnt - 1)];
  const NormDesc D = load_norm(P);
  uint32_t code[7], lg[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    int v = (int)codes[(uint64_t)curve * 7 + i];
    v = v < 0 ? 0 : (v > (int)D.M ? (int)D.M : v);  // keeps reads in bounds on bad input
    code[i] = (uint32_t)v;
  }
#pragma unroll
  for (int i = 0; i < 7; ++i) lg[i] = lds_u32(D.emb_off + (code[i] << D.esh));
  const bool top = uniform((uint32_t)(w & 0xFFFFu)) >> 6;   // the pattern's bit of degree 6
  const uint32_t lane4 = (lane & 31u) * 4u;
  const bool fold = D.kind == kNormFold;
  uint32_t lv[2] = {0, 0};
  // level 1 is shared out over the last 2^slog parts (part 0 of a whole tile)
  const uint32_t pts = D.M / kPartPoints, last = (1u << plog) - 1u;
  const uint32_t slog = pts < 2u ? 0u : min(plog, 31u - (uint32_t)__builtin_clz(pts));
  if (((last - part) >> slog) == 0)
    lv[0] = fold ? norm_level1<true>(D, lg, lane4, last - part, slog) : norm_level1<false>(D, lg, lane4, last - part, slog);
  const auto level2 = [&](auto fold_c, auto pair_c) {
    constexpr bool F = decltype(fold_c)::value, PR = decltype(pair_c)::value;
    return top ? norm_level2<F, true, PR, U>(D, code, lg, lane4, part, plog)
               : norm_level2<F, false, PR, U>(D, code, lg, lane4, part, plog);
  };
  if (PAIR == 1 || (PAIR == 2 && D.pair))
    lv[1] = fold ? level2(std::true_type{}, std::true_type{}) : level2(std::false_type{}, std::true_type{});
  if (PAIR == 0 || (PAIR == 2 && !D.pair))
    lv[1] = fold ? level2(std::true_type{}, std::false_type{}) : level2(std::false_type{}, std::false_type{});
  finish_tile<2>(P, code[0], code[6], lg[0], lg[6], lv, live, curve, 0, 1, outN, outLv, tile, plog, acc, done);
}

}  // namespace hwc
