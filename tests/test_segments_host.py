"""The rules that cut rows into detection segments and baseline chains (no GPU):
segments of lengths that the kernel takes, never more of them than the scratch
was ever sized for, chosen quickly however long the row; no more chains than the
chip holds at once with the histograms asked for."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2512_00398_amd", "csrc")

PROGRAM = r"""
#include <chrono>
#include <cstdio>
#include <random>
#include "sps_segments.h"
using namespace sps;

int main() {
  std::mt19937_64 rng(3);
  for (int k = 0; k < 20000; ++k) {
    const int64_t npos = k < 200 ? 1 + k * 37 : 1 + (int64_t)(rng() % (1ull << (1 + rng() % 31)));
    const int64_t ndm = 1 + (int64_t)(rng() % (1ull << (rng() % 14))), w = 1ll << (rng() % 13);
    const int64_t s = detect_segment(ndm, npos, w), nmax = (npos + 1023) / 1024 * 1024;
    // as many segments as the shortest give, or fewer
    const int64_t least = std::min(nmax, (std::max(std::min(ndm * npos / 8192, kLongSegment), 4 * w) + 1023) / 1024 * 1024);
    const int64_t most = (npos + std::max<int64_t>(least, 1024) - 1) / std::max<int64_t>(least, 1024);
    if (s % kDetectStep || s < kDetectStep || s > nmax || (npos + s - 1) / s > most || s > (int64_t)INT32_MAX) {
      std::printf("ndm %lld npos %lld width %lld: %lld\n", (long long)ndm, (long long)npos, (long long)w, (long long)s);
      return 1;
    }
  }
  const auto t0 = std::chrono::steady_clock::now();
  int64_t sum = 0;
  for (int k = 0; k < 20000; ++k) sum += detect_segment(1, (int64_t)INT32_MAX - 8192 - k, 1);
  const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  std::printf("%.3f %lld\n", s, (long long)sum);
  return s < 2.0 ? 0 : 2;  // 100 us a call; one turn for every possible count takes over 300
}
"""


CHAINS = r"""
#include <cstdio>
#include <random>
#include "sps_segments.h"
using namespace sps;

int main() {
  std::mt19937_64 rng(5);
  for (int k = 0; k < 40000; ++k) {
    const int bins = k % 2 ? 16384 : 4096;
    const int64_t slots = bins == 16384 ? 256 * 2 * 2 : 256 * 4 * 4;  // waves that 160 KB of LDS per CU hold
    const int64_t nb = 1 + (int64_t)(rng() % (1ull << (1 + rng() % 24)));
    const int64_t ndm = 1 + (int64_t)(rng() % (1ull << (rng() % 14))), window = 1 + (int64_t)(rng() % 65535);
    const int64_t seg = chain_blocks(ndm, nb, window, bins), chains = ndm * ((nb + seg - 1) / seg);
    // no more chains than slots, unless there is at least one per row anyway
    if (seg < 1 || seg > nb || chains > std::max(slots, ndm)) {
      std::printf("bins %d: %lld rows of %lld blocks: %lld a chain, %lld chains\n", bins, (long long)ndm, (long long)nb,
                  (long long)seg, (long long)chains);
      return 1;
    }
    const int64_t total = ndm * nb + (int64_t)(rng() % 100000), one = chain_blocks_shared(nb, window, total, bins);
    if (one < 1 || one > nb) return 2;
  }
  return 0;
}
"""


def run(tmp_path, program):
    src, exe = tmp_path / "program.cpp", tmp_path / "program"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_detection_segments(tmp_path):
    run(tmp_path, PROGRAM)


def test_chains_fit_the_chip(tmp_path):
    run(tmp_path, CHAINS)
