#pragma once
// Tile parts: into how many parts a tile's sweep is cut and which points each
// part takes.  Plain C++ (constexpr functions serve the host and the kernels
// alike), so that the rule and the bounds can be checked without a GPU.
//
// A request whose top level sweeps at least kPartMinPoints points by orbits has
// every tile cut into 2^kPartLog parts, so that the last tiles of a launch do
// not hold a few waves long after the rest of the GPU has run dry (one
// 2^20-curve request at q = 293, g = 2: 80 -> 72 ms).  A request (or batch) of
// fewer entries than the waves in flight want is cut further, down to
// kPartPoints top-level points a part: there a wave's serial sweep is the time
// (500 curves at g = 3, q = 13: 8 tiles of 112 us, now 128 parts in 37 us).
#include <cstdint>

namespace hwc {

constexpr uint32_t kPartMinPoints = 8192;
constexpr uint32_t kPartLog = 3;
constexpr uint32_t kPartMaxLog = 8;
// Least points of a part's share of a level, and the distance between the first
// parts of neighbouring levels (odd: no two start alike).
constexpr uint32_t kPartPoints = 48;
constexpr uint32_t kPartStep = 5;

// First of a list's n points that part `part` of 2^plog takes; it ends where the
// next one begins.  In 32 bits: a list is shorter than 2^23 (the orbits of
// F_{q^g}, g >= 2, at most 2^24 elements) and part <= 2^kPartMaxLog.
constexpr uint32_t kPartMaxList = 1u << 23;
static_assert(((uint64_t)kPartMaxList << kPartMaxLog) <= 0xFFFFFFFFull, "n * part stays in 32 bits");
constexpr uint32_t part_begin(uint32_t n, uint32_t part, uint32_t plog) { return (n * part) >> plog; }

// log2 of the parts of a tile whose top level sweeps nx points by orbits, when an
// entry costing `cost` should cost at most `target`.
constexpr uint32_t part_log(uint32_t nx, double cost, double target) {
  uint32_t pl = nx >= kPartMinPoints ? kPartLog : 0;
  while (pl < kPartMaxLog && (nx >> pl) >= 2 * kPartPoints && cost > target * (double)(1u << pl)) ++pl;
  return pl;
}

// ... of a single request of `tiles` tiles: one entry for each of the `waves`
// resident waves, two where the top level sweeps thousands of points and a
// part's setup is small beside its share (count kernel, one against two entries
// a wave: g = 4, q = 13, 7098 points, 2^16 curves 1015 / 627 us; g = 3, q = 13,
// 728 points, 2^17 curves 164 / 186 us).
constexpr uint32_t part_log_single(uint32_t nx, double tiles, double waves, bool norm) {
  uint32_t pl = part_log(nx, 1.0, tiles / (nx >= 6000 ? 2.0 * waves : waves));
  // below eight rounds of the resident waves the last one is a large part of the
  // time: finer while a part keeps 512 points (count kernel: g = 4, q = 13, 2^19
  // curves 3.67 -> 2.72 ms; g = 3, q = 25, 2^17 1.01 -> 0.54)
  if (!norm && nx >= kPartMinPoints / 2)
    while (pl < kPartMaxLog && tiles * (double)(1u << pl) < 8.0 * waves && (nx >> pl) >= 1024) ++pl;
  return pl;
}

}  // namespace hwc
