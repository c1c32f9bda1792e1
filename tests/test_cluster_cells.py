"""The cells that candidates are bucketed by (no GPU): every candidate of the
range is in one of the cells that are cleared and scanned, and linked ones are
in the same or neighbouring cells, up to the largest tolerances and ranges."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2512_00398_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include "sps_cluster_cells.h"
using namespace sps;

int main() {
  const int64_t lo = INT_MIN, hi = INT_MAX;
  const int32_t tols[] = {0, 1, 31, 4095, (1 << 30) - 1, 1 << 30, INT_MAX - 1, INT_MAX};
  const int64_t samples[][2] = {{0, 0}, {-5, 100000}, {0, hi}, {lo, 0}, {lo, hi}, {lo, -1}, {-1, hi}, {lo + 1, hi - 1}};
  const int64_t trials[][2] = {{0, 0}, {0, 7}, {3, 1023}, {0, (1 << 27) - 1}};
  std::mt19937_64 rng(7);
  long checked = 0;
  for (int32_t tt : tols)
    for (int32_t dt : tols)
      for (auto& sr : samples)
        for (auto& dr : trials) {
          int32_t geo[8] = {(int32_t)sr[0], (int32_t)sr[1], 0, 0, (int32_t)dr[0], (int32_t)dr[1], 0, 0};
          cluster_cells(tt, dt, geo);
          const int64_t cells = (int64_t)geo[7] * geo[3];
          bool ok = geo[2] > 0 && geo[3] > 0 && geo[6] != 0 && geo[7] > 0 && cells <= kClusterCells;
          auto pick = [&](const int64_t* r) {
            return r[0] + (int64_t)(rng() % (uint64_t)(r[1] - r[0] + 1));
          };
          for (int k = 0; ok && k < 60; ++k) {
            // the ends of the ranges, values a tolerance from them, and any others
            const int64_t s0 = k % 4 == 0 ? sr[0] : k % 4 == 1 ? sr[1] : pick(sr);
            const int64_t d0 = k % 3 == 0 ? dr[0] : k % 3 == 1 ? dr[1] : pick(dr);
            int64_t s1 = s0 + (k & 8 ? tt : -(int64_t)tt), d1 = d0 + (k & 16 ? dt : -(int64_t)dt);
            if (k & 1) s1 = s0 + (int64_t)(rng() % ((uint64_t)tt + 1));
            s1 = s1 < sr[0] ? sr[0] : s1 > sr[1] ? sr[1] : s1;
            d1 = d1 < dr[0] ? dr[0] : d1 > dr[1] ? dr[1] : d1;
            int t0, c0, t1, c1;
            const uint32_t a = cluster_cell(geo, (int32_t)s0, (uint32_t)d0, t0, c0);
            const uint32_t b = cluster_cell(geo, (int32_t)s1, (uint32_t)d1, t1, c1);
            ok = ok && a < cells && b < cells && t0 >= 0 && t0 < geo[7] && t1 >= 0 && t1 < geo[7];
            ok = ok && c0 >= 0 && c0 < geo[3] && c1 >= 0 && c1 < geo[3];
            ok = ok && abs(t1 - t0) <= 1 && abs(c1 - c0) <= 1;
            ++checked;
          }
          if (!ok) {
            std::printf("tol %d %d samples %lld..%lld trials %lld..%lld: width %d rows %d DM cells %d\n", tt, dt,
                        (long long)sr[0], (long long)sr[1], (long long)dr[0], (long long)dr[1], geo[2], geo[7], geo[3]);
            return 1;
          }
        }
  std::printf("checked %ld\n", checked);
  return 0;
}
"""


def test_cells_hold_every_candidate(tmp_path):
    src, exe = tmp_path / "cells.cpp", tmp_path / "cells"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert r.stdout.startswith("checked")


@pytest.mark.gpu
@pytest.mark.parametrize("tt", [2**31 - 2, 2**31 - 1])
@pytest.mark.parametrize("dms", [4, 40, 700])
def test_largest_time_tolerance(tt, dms):
    import numpy as np
    from oracle import CAND_DTYPE
    from test_gpu_cluster import check
    rng = np.random.default_rng(dms)
    ends = np.array([-2**31, -2**31 + 1, -1, 0, 1, 2**31 - 2, 2**31 - 1])
    # the ends of the range on every trial, then others; trials 3 apart, so linked in time alone
    s = np.concatenate([np.repeat(ends, dms), rng.integers(-2**31, 2**31, size=300)])
    d = np.concatenate([np.tile(np.arange(dms) * 3, ends.size), rng.integers(0, dms, size=300) * 3])
    c = np.empty(s.size, dtype=CAND_DTYPE)
    c["sample"], c["dm_idx"], c["width"] = s, d, 1
    c["snr"] = rng.permutation(s.size).astype(np.float32) + 6
    check(c[rng.permutation(c.size)], tt, 0, 0, "largest-tolerance")
    check(c[rng.permutation(c.size)][:900], tt, 3, 0, "largest-tolerance-trials")
