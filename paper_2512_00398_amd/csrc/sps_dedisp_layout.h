// sps_dedisp_layout.h - host side of the dedispersion kernel: the patterns
// that a delay table's subbands take in each trial group, laid out as the
// kernel's records, and the choice of the subband and tile sizes.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "sps_internal.h"

namespace sps {

struct DedispShape {
  int32_t gch, nsub, tile, trials, ngroups, rec_words, lds_blocks;
};

// A run of subband samples built once for the trials of a group that share
// the subband's pattern of relative delays: samples lo .. hi + tile - 1 of
// the subband's first channel.
struct DedispSegment {
  int32_t lo, hi;
  int32_t rel[kDedispMaxGch];
};

// Segments of (trials d0 .. d0 + nd - 1, channels f0 .. f0 + nf - 1); which[j]
// is trial j's. A trial joins a segment of its pattern when that costs no
// more samples than a segment of its own, so a group never needs more than
// nd * tile samples. Returns the segments' blocks in all.
template <int NF>
inline int dedisp_segments_of(const int32_t* delays, int32_t nchan, int32_t ndm, int32_t d0, int32_t nd, int32_t f0,
                              int32_t tile, DedispSegment* seg, int32_t* which, int& nseg) {
  nseg = 0;
  for (int32_t j = 0; j < nd; ++j) {
    const int32_t* p = delays + (int64_t)std::min(d0 + j, ndm - 1) * nchan + f0;
    int32_t rel[NF];
    for (int32_t i = 0; i < NF; ++i) rel[i] = p[i] - p[0];
    int at = 0;
    for (; at < nseg; ++at) {
      DedispSegment& s = seg[at];
      bool same = true;
      for (int32_t i = 1; i < NF; ++i) same = same && s.rel[i] == rel[i];
      if (!same) continue;
      const int32_t lo = std::min(s.lo, p[0]), hi = std::max(s.hi, p[0]);
      if ((hi - lo) - (s.hi - s.lo) <= tile) {
        s.lo = lo;
        s.hi = hi;
        break;
      }
    }
    if (at == nseg) {
      seg[nseg].lo = seg[nseg].hi = p[0];
      for (int32_t i = 1; i < NF; ++i) seg[nseg].rel[i] = rel[i];
      ++nseg;
    }
    which[j] = at;
  }
  int blocks = 0;
  for (int v = 0; v < nseg; ++v) blocks += (seg[v].hi - seg[v].lo + tile + kDedispBlock - 1) / kDedispBlock;
  return blocks;
}

inline int dedisp_segments(const int32_t* delays, int32_t nchan, int32_t ndm, int32_t d0, int32_t nd, int32_t f0,
                           int32_t nf, int32_t tile, DedispSegment* seg, int32_t* which, int& nseg) {
  static_assert(kDedispMaxGch == 4, "one case for each subband size");
  switch (nf) {
    case 1: return dedisp_segments_of<1>(delays, nchan, ndm, d0, nd, f0, tile, seg, which, nseg);
    case 2: return dedisp_segments_of<2>(delays, nchan, ndm, d0, nd, f0, tile, seg, which, nseg);
    case 3: return dedisp_segments_of<3>(delays, nchan, ndm, d0, nd, f0, tile, seg, which, nseg);
    default: return dedisp_segments_of<4>(delays, nchan, ndm, d0, nd, f0, tile, seg, which, nseg);
  }
}

// Mean and largest block count of the records of a shape, over about
// `sample` of them (0: all).
inline void dedisp_blocks(int32_t nchan, int32_t ndm, const int32_t* delays, const DedispShape& sh, int sample,
                          double& mean, int32_t& most) {
  DedispSegment seg[kDedispMaxTrials];
  int32_t which[kDedispMaxTrials];
  int nseg = 0;
  const int32_t gs = sample ? std::max(1, sh.ngroups / 8) : 1, ss = sample ? std::max(1, sh.nsub * 8 / sample) : 1;
  double sum = 0.0, seen = 0.0;
  most = 0;
  for (int32_t q = 0; q < sh.ngroups; q += gs)
    for (int32_t s = 0; s < sh.nsub; s += ss) {
      const int n = dedisp_segments(delays, nchan, ndm, q * sh.trials, sh.trials, s * sh.gch,
                                    std::min(sh.gch, nchan - s * sh.gch), sh.tile, seg, which, nseg);
      sum += n;
      seen += 1.0;
      most = std::max(most, n);
    }
  mean = sum / seen;
}

// A shape of g channels per subband and the q-th tile size, its block counts
// filled in; false if its subband sums need more than 64 KB of LDS. The last
// tile size always fits (2 blocks x 8 trials).
constexpr int kDedispTiles[4][2] = {{4, 32}, {4, 16}, {2, 16}, {2, 8}};  // blocks x trials

inline bool dedisp_shape(int32_t nchan, int32_t ndm, const int32_t* delays, int q, int32_t g, int sample,
                         DedispShape& sh, double& mean) {
  sh.gch = g;
  sh.nsub = (nchan + g - 1) / g;
  sh.tile = kDedispTiles[q][0] * kDedispBlock;
  sh.trials = kDedispTiles[q][1];
  sh.ngroups = (ndm + sh.trials - 1) / sh.trials;
  dedisp_blocks(nchan, ndm, delays, sh, sample, mean, sh.lds_blocks);
  return 4 * dedisp_copy_bytes(sh.lds_blocks) <= 65536;
}

// Modelled cycles of a shape with `mean` blocks per record. Each resident
// workgroup needs about 900 cycles a subband for its sums and the barrier and,
// for every block that a wave builds, 400 + 100 per channel; the vector units
// need 11 cycles per trial and 1008 samples, 15 to 40 per block and 25 per
// wave. Fitted on 64 to 1024 channels x 24 to 1024 trials, all shapes. For
// example (us; blocks x trials x channels): 1024 x 1024 x 2^18: 4x32x2 7766,
// 4x16x2 8526, 2x16x2 9402, 4x32x1 12373; 256 x 128 x 40001: 2x8x2 145,
// 2x8x4 157, 2x16x1 169, 4x32x1 181; 64 x 24 x 5000: 2x8x4 25, 2x8x1 34,
// 4x32x1 49; 64 x 1024 x 100000: 4x16x1 353, 4x32x1 382, 2x8x1 578.
inline double dedisp_cost(const DedispShape& sh, double mean, int64_t nsamp_out) {
  static const double kBuild[kDedispMaxGch + 1] = {0.0, 15.0, 19.0, 32.0, 40.0};
  const int waves = sh.trials == 32 ? 8 : 4;
  const double tiles = (double)((nsamp_out + sh.tile - 1) / sh.tile);
  const double per_cu = std::ceil(tiles * sh.ngroups / 256.0);
  const double resident = std::min(sh.trials == 32 ? 2.0 : sh.tile == 4 * kDedispBlock ? 5.0 : 6.0,
                                   std::floor(163840.0 / (4.0 * dedisp_copy_bytes(sh.lds_blocks))));
  const double issue = sh.trials * (sh.tile / 1008.0) * 11.0 + mean * kBuild[sh.gch] + 25.0 * waves;
  const double latency = 900.0 + std::max(1.0, mean / waves) * (400.0 + 100.0 * sh.gch);
  return sh.nsub * std::max(1.35 * issue * per_cu, latency * std::ceil(per_cu / resident));
}

inline DedispShape dedisp_choose(int32_t nchan, int32_t ndm, int64_t nsamp_out, const int32_t* delays) {
  // every shape on a sample of the records, then the cheapest that fits on all
  // of them (64 records choose as 256 did on 296 of 300 random tables, the
  // others within 3 % of its modelled cost, in a third of the time)
  struct Option {
    double cost;
    int q;
    int32_t g;
  };
  std::vector<Option> options;
  DedispShape sh;
  double mean;
  for (int q = 0; q < 4; ++q)
    for (int32_t g = 1; g <= std::min<int32_t>(kDedispMaxGch, nchan); ++g)
      if (dedisp_shape(nchan, ndm, delays, q, g, 64, sh, mean))
        options.push_back({dedisp_cost(sh, mean, nsamp_out), q, g});
  std::sort(options.begin(), options.end(), [](const Option& x, const Option& y) { return x.cost < y.cost; });
  for (const Option& o : options)
    if (dedisp_shape(nchan, ndm, delays, o.q, o.g, 0, sh, mean)) break;
  return sh;  // (the last tile size is among the options and always fits)
}

// The records of a shape ([ngroups][nsub][rec_words]) for a delay table [ndm][nchan].
inline void dedisp_records(int32_t nchan, int32_t ndm, int64_t nsamp_in, const int32_t* delays, DedispShape& sh,
                           std::vector<int32_t>& rec) {
  const int32_t g = sh.gch;
  sh.rec_words = kDedispHead + std::max(sh.lds_blocks, kDedispAhead) * g;
  rec.assign((size_t)sh.ngroups * sh.nsub * sh.rec_words, 0);
  DedispSegment seg[kDedispMaxTrials];
  int32_t which[kDedispMaxTrials];
  int nseg = 0;
  for (int32_t q = 0; q < sh.ngroups; ++q)
    for (int32_t s = 0; s < sh.nsub; ++s) {
      const int32_t f0 = s * g, nf = std::min(g, nchan - f0);
      int32_t* r = &rec[((size_t)q * sh.nsub + s) * sh.rec_words];
      r[0] = dedisp_segments(delays, nchan, ndm, q * sh.trials, sh.trials, f0, nf, sh.tile, seg, which, nseg);
      int32_t first[kDedispMaxTrials];
      int32_t at = 0;
      for (int v = 0; v < nseg; ++v) {
        first[v] = at * kDedispBlock;
        const int n = (seg[v].hi - seg[v].lo + sh.tile + kDedispBlock - 1) / kDedispBlock;
        for (int k = 0; k < n; ++k, ++at)
          for (int32_t i = 0; i < g; ++i) {
            const bool have = i < nf;
            const int64_t row = (int64_t)(f0 + (have ? i : 0)) * nsamp_in;
            const int64_t from = row + seg[v].lo + k * kDedispBlock + (have && i > 0 ? seg[v].rel[i] : 0);
            r[kDedispHead + g * at + i] =
                (int32_t)((uint32_t)((from >> 2) - (row >> 2)) | ((uint32_t)(from & 3) << 30));
          }
      }
      for (; at < kDedispAhead; ++at)
        for (int32_t i = 0; i < g; ++i) r[kDedispHead + g * at + i] = r[kDedispHead + g * (at - 1) + i];
      for (int32_t j = 0; j < sh.trials; ++j) {
        const int32_t d = std::min(q * sh.trials + j, ndm - 1);
        const int32_t e = first[which[j]] + delays[(int64_t)d * nchan + f0] - seg[which[j]].lo;
        const uint32_t byte = (e & 1) ? dedisp_copy_bytes(sh.lds_blocks) + 2 * (e - 1) : 2 * e;
        r[1 + j / 2] |= (int32_t)(byte << (16 * (j & 1)));  // below 2^15: two copies of at most 16 KB
      }
    }
}

}  // namespace sps
