"""Tile parts (csrc/parts.h) without a GPU: for every admitted field and every
size of request the number of parts stays within its limit, and the parts'
ranges are those of whole-number arithmetic -- in order and covering each list
exactly, so that no part reads outside it."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_11991_amd", "csrc")

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include <set>
#include "parts.h"

static bool odd_prime_power(uint32_t q) {
  for (uint32_t p = 3; p * p <= q; p += 2)
    if (q % p == 0) {
      while (q % p == 0) q /= p;
      return q == 1;
    }
  return q >= 3;
}

// the parts of a list of n points
static bool covers(uint32_t n, uint32_t plog) {
  for (uint64_t part = 0; part <= (1ull << plog); ++part)
    if (hwc::part_begin(n, (uint32_t)part, plog) != ((uint64_t)n * part) >> plog) return false;
  return true;
}

int main() {
  uint32_t fields = 0;
  for (uint32_t g = 1; g <= 4; ++g)
    for (uint32_t q = 3; q <= 20448; q += 2) {
      uint64_t Q = 1;
      for (uint32_t k = 0; k < g; ++k) Q *= q;
      if (Q > (1u << 24)) break;
      if (!odd_prime_power(q)) continue;
      ++fields;
      // Frobenius orbits of length g
      const uint64_t below = g == 1 ? 1 : g == 4 ? (uint64_t)q * q : q;
      const uint32_t nx = (uint32_t)((Q - below) / g);
      std::set<uint32_t> logs;
      for (uint32_t waves : {256u, 1024u, 4096u, 6144u, 8192u})
        for (uint32_t tiles = 1; tiles <= (1u << 18); tiles += tiles < 64 ? 1 : tiles / 3) {
          for (bool norm : {false, true}) logs.insert(hwc::part_log_single(nx, tiles, waves, norm));
          logs.insert(hwc::part_log(nx, 1.0, tiles / (double)waves));   // a job of a batch
        }
      for (uint32_t pl : logs) {
        if (pl > hwc::kPartMaxLog) {
          printf("g=%u q=%u: 2^%u parts\n", g, q, pl);
          return 1;
        }
        // whole lists, the tuples of the split evaluation and their singles
        for (uint32_t n : {nx, nx / 2, nx / 4, nx / 3, nx % 4, nx % 97})
          if (!covers(n, pl)) {
            printf("g=%u q=%u: %u points in 2^%u parts\n", g, q, n, pl);
            return 1;
          }
      }
    }
  printf("%u fields\n", fields);
  return fields > 2000 ? 0 : 1;
}
"""


def test_parts_cover_every_list(tmp_path):
    src, exe = tmp_path / "parts.cpp", tmp_path / "parts"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
