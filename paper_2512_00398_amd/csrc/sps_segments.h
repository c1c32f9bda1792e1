// sps_segments.h - how rows are cut into baseline chains and detection
// segments (tuning only; results do not depend on it). Host code without HIP.
#pragma once

#include <algorithm>
#include <cstdint>

namespace sps {

constexpr int kCus = 256;
constexpr int kDetectStep = 1024;

// Chains (waves) of the statistics kernel in a workgroup, and workgroups that a
// CU holds: by their histograms, 32 KB for four chains of 4096 bins, 64 KB for
// two of 16384.
inline int64_t chain_waves(int bins) { return bins == 16384 ? 2 : 4; }
inline int64_t chain_groups(int bins) { return bins == 16384 ? 2 : 4; }

// Blocks per baseline chain for `ndm` rows of `nb` blocks: one workgroup per CU
// up to as many as it holds, whichever is modelled fastest. More, shorter
// chains hide each other's latency (a block takes about 1 us in a lone chain;
// with four workgroups of four on a CU each runs at 1 / 1.54 of its speed,
// measured on 256 x 131072) but each recounts its first window, about as long as
// `window` / 128 blocks. More chains than the chip holds only add recounts.
// Measured (us, statistics alone; with chains of at least four windows, then
// this): 64 x 16384, window 4096: 2437, 66; 16 x 500000, window 3000: 2185, 173;
// 256 x 65536, window 4096: 332, 161; 2048 x 65536, window 16384: 2078, 1001.
// 16384 bins, whole calls (with that, with chains for the 4096 slots of 4096
// bins, with their own 1024): 1024 x 2^18, window 16384: 3847, 2855, 2599; 32 x
// 2^20, window 30000: 1479, 506, 391; 2000 x 5000, window 1000: 1919, 422, 339;
// 64 x 16384, window 4096: 522, 61, 61.
inline int64_t chain_blocks(int64_t ndm, int64_t nb, int64_t window, int bins) {
  const double recount = 10.0 + (double)window / 128.0;
  const double slower = bins == 16384 ? 0.02 : 0.18;  // (four chains of 16384 bins are one wave per SIMD)
  int64_t best = nb;
  double best_t = 0.0;
  for (int64_t k = 1; k <= chain_groups(bins); ++k) {
    const int64_t per_row = std::max<int64_t>(1, kCus * chain_waves(bins) * k / ndm);
    const int64_t seg = std::max<int64_t>(std::min<int64_t>(nb, 4), (nb + per_row - 1) / per_row);
    const double t = (recount + (double)seg) * (1.0 + slower * (double)(k - 1));
    if (k == 1 || t < best_t) {
      best = seg;
      best_t = t;
    }
  }
  return std::max<int64_t>(1, best);
}

// The same for one of several blocks in a launch with `total_blocks` in all:
// chains of about the launch's share of a resident wave, even within a row,
// each longer than its window's recount.
inline int64_t chain_blocks_shared(int64_t nb, int64_t window, int64_t total_blocks, int bins) {
  const int64_t slots = kCus * chain_waves(bins) * chain_groups(bins);
  const int64_t want = std::max<int64_t>((total_blocks + slots - 1) / slots, 16 + window / 128);
  const int64_t per_row = (nb + want - 1) / want;
  return std::max<int64_t>(1, (nb + per_row - 1) / std::max<int64_t>(per_row, 1));
}

// Shortest detection segments are at most this long: short ones even out rows of unlike cost.
constexpr int64_t kLongSegment = 65536;

// Positions per detection segment for `ndm` rows of `npos` positions. At least
// 4 max_width (each segment repeats that much of its neighbour) and about
// 8192 segments in all; from there on the length whose modelled time is least:
//   a segment takes its own steps and its halo's;
//   up to four workgroups per CU are one round, somewhat shorter with fewer;
//   more take rounds that are partly filled, partly made up as some end early;
//   many workgroups even out segments of unlike cost;
//   a row's segments are stitched one after another, each a seventh of a step.
// Five workgroups fit a CU, but share its issue slots: with a round of five the
// model does 2 % better on average and up to 17 % worse on single shapes.
// Fitted on 32 shapes of 1 x 2^20 to 5000 x 2048, widths to 1 .. 4096, with and
// without drift and at low thresholds, 5 to 30 lengths each: 6.5 % above the
// best of each on average, 11.3 % without the stitching and with whole rounds
// (us, the whole search of a quiet and of a drifting block, that rule and this
// one: 1 x 2^20, widths to 64, 312 and 494, 101 and 191; 40 x 2^20, to 32, 398
// and 802, 364 and 704; 128 x 2^18, to 256, 304 and 786, 299 and 731; 1100 x
// 30000, to 128, 443 and 1024, 434 and 983; 256 x 131072, 333 x 100003, 64 x
// 16384 and gulps of 2048 x 65536 the same; 40 x 2^20 at a threshold of 2.5, with
// a candidate in every 15 samples, 856, 891).
inline int64_t detect_segment(int64_t ndm, int64_t npos, int64_t max_width) {
  int64_t seg = std::max<int64_t>(std::min<int64_t>(ndm * npos / 8192, kLongSegment), 4 * max_width);
  const int64_t nmax = (npos + kDetectStep - 1) / kDetectStep * kDetectStep;
  seg = std::max<int64_t>(kDetectStep, std::min(nmax, (seg + kDetectStep - 1) / kDetectStep * kDetectStep));
  int64_t best = seg;
  double best_t = 0.0;
  // (all counts up to 16, from there on every sixteenth part: a row may be cut into thousands)
  for (int64_t per_row = (npos + seg - 1) / seg; per_row >= 1; per_row -= std::max<int64_t>(1, per_row / 16)) {
    const int64_t s = ((npos + per_row - 1) / per_row + kDetectStep - 1) / kDetectStep * kDetectStep;
    const int64_t nseg = (npos + s - 1) / s;
    const double per_cu = (double)((ndm * nseg + kCus - 1) / kCus);
    const double steps = (double)(s / kDetectStep + (max_width + 64 + kDetectStep - 1) / kDetectStep);
    const double full = (double)((ndm * nseg + 4 * kCus - 1) / (4 * kCus));
    const double rounds = per_cu <= 4.0 ? 0.7 + 0.075 * per_cu : 0.6 * full + 0.4 * (0.25 * per_cu + 0.2);
    const double t = steps * rounds * (1.0 + 0.9 / per_cu) + (nseg > 1 ? 0.15 * (double)nseg : 0.0);
    if (best_t == 0.0 || t < best_t) {
      best_t = t;
      best = s;
    }
  }
  return best;
}

}  // namespace sps
