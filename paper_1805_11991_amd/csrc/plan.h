// Device-side description of one (q, g) counting plan, shared by the HIP
// kernels and the host code that builds it.
//
// A plan covers the fields F_{q^j}, j = 1..g (one "level" per field).  All
// of its lookup tables are packed into one image that every workgroup copies
// into LDS before it starts counting:
//
//   form A  (M <= 10922)  "byte units":  5M u16 entries.  Entry i < 3M holds
//           2*Z(i mod M), or the zero marker 6M when 1 + gamma^(i mod M) = 0;
//           entries 3M..5M-1 hold 0.  One Horner step is one add and one read.
//   form C  (M <= 32767)  "element units": 2M u16 entries.  Entry i holds
//           Z(i mod M), or M as the zero marker.  One Horner step is add,
//           fold into [0, 2M), scale to bytes, read, and a marker test.
//   form E  (M <= 65534)  "element units, one period": M u16 entries, entry
//           i holds Z(i), or M as the zero marker.  A step folds its index
//           into the period once more than form C and doubles the entry it
//           reads, so it shares form C's code; twice the field size of form C
//           fits in LDS.
//   form F  (M <= 131070)  "half table": Z(k) for k = 0..M/2 only, entry
//           i = M/2 - k, as u16 low halves; the 17th bit of entry i is bit
//           i >> 12 of word i mod 4096 of a plane of kFormFPlane bytes before
//           them.  The other half follows from Z(-k) = Z(k) - k
//           (1 + g^-k = g^-k (1 + g^k)), so Z(k) = Z(M - k) + k mod M for
//           k > M/2: both halves read entry |k - M/2|.  Two reads per lookup.
//   form D  (any M)  the form C layout with u32 entries, kept in device
//           memory (L2/MALL-resident) when the level does not fit in LDS.
//   emb     q u32 entries: log of the F_q code c in F_{q^j}, or M for c = 0.
//
// Logs are taken to the primitive element gamma of each F_{q^j}; Z is the
// Zech logarithm Z(k) = log(1 + gamma^k) (eq. 2.1, table (3.2)).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "parts.h"

namespace hwc {

constexpr int kMaxG = 4;                 // genus handled by the kernels
constexpr int kMaxCoef = 2 * kMaxG + 3;  // a_0 .. a_{2g+2}
constexpr uint32_t kFormA = 0, kFormC = 1, kFormD = 2, kFormE = 3, kFormF = 4, kFormG = 5;
constexpr uint32_t kFormAMaxM = 10922;   // 6M must fit in u16
constexpr uint32_t kFormCMaxM = 32767;   // M must fit in 15 bits
constexpr uint32_t kFormEMaxM = 65534;   // M (the zero marker) must fit in u16
constexpr uint32_t kFormFMaxM = 131070;  // M must fit in 17 bits, M/2 + 1 entries in the half table
constexpr uint32_t kFormFPlane = 8192;   // 4096 u16 words: 16 bits each reach the largest M / 2
// Form G: the half table of form F as u32 entries in byte units (one read, no
// bit plane), used where its 4 (M/2 + 1) bytes fit the LDS image
constexpr int kWave = 64;
// LDS of one CU is 160 KiB; 256 bytes stay free for the kernels' own variables
constexpr uint32_t kLdsImageLimit = 160 * 1024 - 256;
// Dense translates (rows replaced by f(x + t), see shift_kernel): fields with
// q <= kShiftMaxQ, whose q^3-byte step table fits LDS, at most kShiftTries t.
constexpr uint32_t kShiftMaxQ = 32;
constexpr uint32_t kShiftTries = 8;
// For prime q the translate is also an integer matrix product: after the
// step table (q^3 bytes, padded to 16) the shift buffer holds, for t = 0 ..
// kShiftTries, the rows i = 0 .. NC-2 of binom(j, i) t^(j-i) mod q (j >= i,
// zero below), bytes packed four to a word: shift_tmat_words(NC) words per t.
inline constexpr uint32_t shift_tmat_offset_words(uint32_t q) { return (q * q * q + 15) / 16 * 4; }
inline constexpr uint32_t shift_tmat_row_words(uint32_t nc) { return (nc + 3) / 4; }
inline constexpr uint32_t shift_tmat_words(uint32_t nc) { return (nc - 1) * shift_tmat_row_words(nc); }

struct LevelDesc {
  uint32_t M;         // |F_{q^j}^x|
  uint32_t form;      // kFormA, kFormC, kFormD, kFormE, kFormF or kFormG
  uint32_t tab_off;   // byte offset of the level's table in the image
  uint32_t emb_off;   // byte offset of the level's emb table in the image
  uint32_t nx;        // number of x logs swept at this level
  uint32_t weight;    // points of F_{q^j} each swept x stands for (orbit size, or 1)
  const uint32_t* xs; // x logs (device), nullptr: x runs over 0..M-1
  const uint32_t* gtab;  // form D: 2M entries in device memory
  // split evaluation over mu_m cosets (m = 4, 3 or 2; forms C/D: 4 or 2): nt tuple
  // representatives (points L + s M/m, s < m) and ns single points; together
  // they are the same nx points.  msplit = 0 turns it off.
  uint32_t msplit, nt, ns;
  const uint32_t* xs_t;  // nullptr: representatives 0..M/m-1 (full sweep)
  const uint32_t* xs_s;
};

// Genus 2 with the norm tables (norm_impl.h) in place of level 2's Zech table.
// Image: the rows at offset 0, the codes' logs, the byte table of the last step.
constexpr uint32_t kNormRow = 128;         // bytes of a row: one u32 per LDS bank
constexpr uint32_t kNormTmatWords = 18;    // words per t of the translates of degree 6
constexpr uint32_t kNormPlain = 1, kNormFold = 2;
struct NormDesc {
  uint32_t kind;          // 0: none, kNormPlain, kNormFold
  uint32_t M;             // q - 1
  uint32_t srow;          // row a vanished sum reads as: a power of two, at least 4M
  uint32_t emb_off, esh;  // logs of the codes in F_q: u32 every 2^esh bytes
  uint32_t fin_off;       // byte table of the last step
  uint32_t pair;          // prime q = 1 mod 4: v and -v together (its byte table has two entries an index)
  uint32_t qm;            // floor(v / (q << esh)) = (v * qm) >> 32 for the integer translates
  const uint32_t* tmat;   // prime q: [q][kNormTmatWords] translate rows; nullptr: log arithmetic
};

struct PlanDesc {
  uint32_t q, p, g, ncoef;   // q = p^e; ncoef = 2g+3
  uint32_t orbit;         // 1: level j sweeps primitive Frobenius orbits of F_{q^j}
  uint32_t image_bytes;   // LDS image size (multiple of 16)
  const uint32_t* image;  // device copy of the image (dwords)
  LevelDesc lv[kMaxG];
  NormDesc norm;          // kind != 0: level 2 is counted by norms
};

// Factorization partition code (eq. 1.2): the multiplicity of part j
// (j = 1..10, i.e. 2g+2 <= 10) sits in bits [lam_shift(j), lam_shift(j) + w_j)
// with widths w = 4, 3, 2, 2, 2, 1, 1, 1, 1, 1 -- enough for every partition
// of 10 -- so a code fits in kLamBits bits.
constexpr uint32_t kLamBits = 18;
constexpr uint32_t kLamInvalid = 0xFFFFFFFFu;   // root counts inconsistent with a square-free row
__host__ __device__ constexpr uint32_t lam_shift(uint32_t j) {
  return j == 1 ? 0u : j == 2 ? 4u : j == 3 ? 7u : j == 4 ? 9u : j == 5 ? 11u : 7u + j;
}

// The partition codes a histogram column can hold for genus g: 0 (the mark of
// a row with a square factor) and the code of every partition of 2g+2, in
// ascending order, so a code's rank there is a dense digit (at most 43 values,
// p(10) = 42) that sorts like the code. Writes them to out (room for
// kLamCodesMax, or nullptr) and returns how many there are.
constexpr uint32_t kLamCodesMax = 48;
inline uint32_t lam_code_list(uint32_t g, uint32_t* out) {
  uint32_t buf[kLamCodesMax];
  uint32_t n = 0;
  buf[n++] = 0;
  // parts in non-increasing order: stack of (remaining degree, largest part, code)
  struct Frame { uint32_t rem, maxp, code; };
  Frame st[64];                          // pending siblings along one path: <= 10 + 9 + .. + 1
  uint32_t top = 0;
  st[top++] = {2 * g + 2, 2 * g + 2, 0};
  while (top) {
    const Frame f = st[--top];
    if (f.rem == 0) {
      if (n < kLamCodesMax) buf[n++] = f.code;
      continue;
    }
    for (uint32_t j = 1; j <= f.maxp && j <= f.rem; ++j) st[top++] = {f.rem - j, j, f.code + (1u << lam_shift(j))};
  }
  for (uint32_t i = 1; i < n; ++i)   // insertion sort (n <= 43)
    for (uint32_t k = i; k > 0 && buf[k - 1] > buf[k]; --k) {
      const uint32_t t = buf[k];
      buf[k] = buf[k - 1];
      buf[k - 1] = t;
    }
  if (out)
    for (uint32_t i = 0; i < n; ++i) out[i] = buf[i];
  return n;
}

// The partition codes as histogram digits: a code's rank, found through a
// multiplicative hash with a slot per code.
struct LamCodes {
  uint32_t n;                       // codes (ascending)
  uint32_t code[kLamCodesMax];
  uint32_t mul;                     // slot (c * mul) >> 24 is distinct for every code c
  uint8_t slot[256];                // rank + 1 of the code in that slot, 0 for none
};

// One request of the one-workgroup histogram (hist_small.hip).
constexpr uint32_t kHistSmallMax = 8192;
struct HistJob {
  const int32_t* N;        // [n][g]
  const uint32_t* lam;     // [n] partition codes, or nullptr
  int32_t* keys;           // [cap][g, or g + 1 with lam]
  uint64_t* counts;        // [cap]
  uint64_t* len;           // number of distinct tuples, or nullptr
  uint64_t cap;
  uint32_t n, g, q, pad;
};

// One request of the one-workgroup bucketing (bucket_small.hip).
constexpr uint32_t kBucketSmallMax = 8192;
struct BucketJob {
  const void* codes;       // [n][2g+3] int8 or int16
  void* out;               // dense translates of the rows (mode 1, 2)
  const uint32_t* step;    // the plan's shift buffer (mode 1, 2)
  uint32_t* perm;          // [n]
  uint64_t* tiles;
  uint32_t* ntiles;
  uint32_t* queue;
  uint32_t* acc;           // words to clear for tile parts
  uint32_t acc_words;
  uint32_t n, q, g, cb;
  uint32_t mode;           // 0: rows as given; 1: translates, prime q; 2: translates by the step table
};

// One curve for the lane-per-x kernel: coefficient logs in F_{q^k} (M where
// the coefficient is zero), degree d, M = q^k - 1.
constexpr uint32_t kSingleThreads = 512;
struct SingleDesc {
  uint32_t lc[2 * kMaxG + 3];
  uint32_t d, M;
};

// Counting by F_p-linear algebra (prime q = p): with F_{p^j} = F_p[t]/(P) and
// x^i = sum_d a_{i,d} t^d, f(x) = sum_i c_i x^i has coordinates
// D_d = sum_i c_i a_{i,d} mod p, i.e. the codes times a Vandermonde matrix of
// coordinates -- an int8 matrix product for the matrix cores.  The image holds,
// per level, the swept points in blocks of 32 as the A operand of
// v_mfma_i32_32x32x16_i8 ([block][d][row][16 bytes]; coordinate 0 times 4, so
// its residue mod 4p is four times the residue mod p), then a u32 table of the
// quadratic character over packed elements (byte offset 4 sum_d r_d p^d):
// 0 square, 1 nonsquare, kVZero for zero.  Needs 4(p-1) <= 127: p <= 31.
// When a level's blocks do not fit one image, its points are split over
// several images (passes) that add their counts per curve; such a level may
// use a u16 table (byte offset 2 sum_d r_d p^d, coordinate 0 doubled).
// The K slots past the coefficients hold 127 on the curve side and, in the
// coordinate-0 rows, values summing to to / 127, so the product adds the
// table's byte offset (a multiple of 508) to coordinate 0 by itself.
constexpr uint32_t kVSlotUnit = 127;
constexpr uint32_t kVZero = 1u << 15;
constexpr uint32_t kVMaxP = 31;
struct VLevel {
  uint32_t pts, nblk;     // swept points in the image and their 32-point blocks
  uint32_t pad;           // padding rows of the blocks (zero points, subtracted)
  uint32_t vo, to;        // byte offsets of the blocks and of the character table
  uint32_t m0, s0;        // floor(v / 4p) = (v * m0) >> s0 for every value coordinate 0 reaches
  uint32_t nbm0;          // -to * m0 mod 2^32: coordinate 0 arrives with the table offset added
  uint32_t m1, s1;        // floor(v / p) = (v * m1) >> s1 for the other coordinates
};
// Fractional form (p <= 13): the points' coordinates come as fractions of
// 2^kFracBits, a -> a 2^12 / p rounded (two int8 parts, matched by the codes
// times `frac` and the codes on the curve side, 22 of 32 slots), so the
// product is D_d 2^12 / p up to a small error and, modulo 2^12, the fraction of
// D_d / p: no division by p.  Its top four bits are one of 16 cells, and no two
// residues share a cell (16 / p - 2 err 2^-8 >= 1, checked for the points of
// every level); coordinates 1 .. k - 1 give a word's index, coordinate 0's top
// five bits rotate the word, whose two low bits then say square (00),
// nonsquare (11) or zero (01 or 10).  Words: [cell_1 | cell_2 << 4][64 lanes],
// or for four coordinates [cell_1 << 8 | cell_2 << 12 | cell_3 << 4][4 copies].
constexpr uint32_t kFracBits = 12, kFracMaxP = 13;
struct VPlanDesc {
  uint32_t p, g, ncoef, orbit;
  uint32_t frac;          // fractional form: the curve side's weight floor(127 / ((p - 1) / 2)), else 0
  uint32_t nsmask;        // fractional form: bit c set where the code c is a nonsquare of F_p
  uint32_t image_bytes;
  const uint32_t* image;
  VLevel lv[kMaxG];
};

// One request of a multi-plan launch (device memory).
struct JobDesc {
  const PlanDesc* plan;   // device copy of the job's plan
  const void* codes;      // [n][2g+3] int8 or int16
  const uint32_t* perm;   // bucketed order of the job's rows
  const uint64_t* tiles;  // the job's tile words
  const uint32_t* ntiles; // number of tile words (written by the bucketing)
  uint32_t* queue;        // the job's tile queue (set to 0 by the bucketing)
  int32_t* outN;          // [n][g]
  uint32_t cb, g;         // code bytes, genus
  // Every tile's sweep cut into 2^plog parts (queue entry u: tile u >> plog,
  // part u & (2^plog - 1)) when a job has few tiles for the waves in flight:
  // the parts add their level counts into acc and the last part of a tile
  // (counted in done) assembles N.  plog = 0: whole tiles.
  uint32_t plog;
  uint32_t norm;          // the plan has norm tables
  float cost;             // work of one queue entry
  uint32_t chunk;         // entries a workgroup takes at once, at least (at most one for each of its waves)
  uint32_t* acc;          // [n][g] packed level counts (zero before the launch)
  uint32_t* done;         // [tiles] parts finished (zero before the launch)
};

// A tile is up to 64 curves that share degree and zero pattern.
// word = pattern | (count-1) << 16 | start << 32
__host__ __device__ inline uint64_t tile_pack(uint32_t pattern, uint32_t start, uint32_t count) {
  return (uint64_t)pattern | ((uint64_t)(count - 1) << 16) | ((uint64_t)start << 32);
}

// Pattern of a row: bit 2g+2 set when deg f = 2g+2; bits 0..d-1 mark the
// nonzero a_i below the leading term.
__host__ __device__ inline uint32_t pattern_count(uint32_t g) { return 1u << (2 * g + 3); }

}  // namespace hwc
