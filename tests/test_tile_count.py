"""The counting of the tile form, replayed on the host: sums of decisions t and of
t^2 over a block of tiles in the kernel's order and arithmetic, the comparison that
finds an undecided point, and the total. t is 1 for an inlier and 0 for an outlier;
one t just off 0 or 1 (or up to three) can leave both sums equal, and then counts as
what it is next to, at every place in the block."""
import os
import subprocess

import pytest

from paper_2402_18008_amd import build

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include <vector>
#include "ransac_dev.hpp"

static long replayed = 0, agreed = 0;

// One lane over blocks of TB tiles: the count, and whether any block was listed.
static bool replay(const std::vector<float> &t, int TB, unsigned &count) {
  float total = hg::kTotalZero;
  for (size_t b = 0; b < t.size(); b += TB) {
    volatile float s = 0.0f, q = 0.0f;
    for (size_t i = b; i < b + TB && i < t.size(); ++i) {
      s = s + t[i];
      q = fmaf(t[i], t[i], q);
    }
    if (s != q) return false;
    total = hg::block_total(total, s);
  }
  count = hg::total_count(total);
  return true;
}

static bool check(const std::vector<float> &t, int TB) {
  unsigned want = 0, got = 0;
  for (float x : t) want += x >= 0.5f;
  ++replayed;
  if (!replay(t, TB, got)) return true;   // listed: counted in float64
  ++agreed;
  if (got != want) printf("TB %d, %zu tiles: %u counted, not %u\n", TB, t.size(), got, want);
  return got == want;
}

int main() {
  const float ulp = 0x1p-24f;
  long odd = 0;
  for (int TB : {16, 32})
    for (int tiles : {1, 5, TB, 2 * TB, 3 * TB + 7})
      for (int ones = 0; ones <= tiles; ++ones)
        for (int at = 0; at < tiles; ++at)
          for (int j = 1; j <= 40; ++j)
            for (float off : {1.0f - j * ulp, j * ulp * ulp, j * ulp}) {
              std::vector<float> t(tiles, 0.0f);
              for (int i = 0; i < ones; ++i) t[(at + 1 + i) % tiles] = 1.0f;
              t[at] = off;
              const long before = agreed;
              if (!check(t, TB)) return 1;
              odd += agreed > before && off > 0.5f;
              if (tiles > 2 && j % 7 == 0) {   // more of them
                t[(at + 2) % tiles] = off;
                t[(at + tiles / 2) % tiles] = 1.0f - ulp;
                if (!check(t, TB)) return 1;
              }
            }
  // long pairs: totals where a float no longer holds halves
  unsigned c = 0;
  if (!replay(std::vector<float>((1u << 21) + 3, 1.0f), 16, c) || c != (1u << 21) + 3) return 1;
  printf("%ld replayed, %ld with equal sums, %ld of them with one t just below 1\n", replayed,
         agreed, odd);
  return odd > 0 ? 0 : 1;
}
"""


def test_count_of_equal_sums(tmp_path):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    src = tmp_path / "count_check.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "count_check"
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", build.CSRC,
                        str(src), "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, (r.stdout, r.stderr)
