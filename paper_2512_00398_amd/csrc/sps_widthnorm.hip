// sps_widthnorm.hip - per-width re-normalisation (Heimdall++ Section II-B,
// the normalisation stage read as one robust noise scale for every
// boxcar-filtered series): for every row and width w = 2^j, over the
// filtered series T_w = {S_w(i) : 0 <= i <= N - w}, S_w(i) = sum of r over
// [i, i + w), r_t = x_t - m_{floor(t/64)}, the lower median c_w (rank
// floor((n - 1) / 2) of n = N - w + 1 values) and MAD_w, the lower median of
// |S_w(i) - c_w|. Exact.
//
// Design (gfx950): one 1024-thread workgroup per row. The row is streamed in
// steps of 4096 samples; the prefix sums P of the residual of two steps live
// in an LDS ring, so every boxcar sum of every width is one difference
// P[E] - P[E - w] (uint32, wrapping; exact for |S| < 2^31). Each pass over
// the row evaluates all widths at once.
//
// Bound by vector instructions per key and, before the sampling, by the LDS
// atomics of a histogram of every key (1024 rows x 2^20: 40 ms, 28 of them
// atomics). So the row is first sampled (every 4th position, for widths from
// 64 on every 16th; more of a short row): a pass for the sampled range, one
// for a 2048-bin histogram, from which median and MAD are estimated. The
// exact pass then counts, in registers, the keys below a window of values
// about the median c and the keys closer to its estimate than a window of
// distances about the MAD, and histograms only the keys inside these windows
// (a few per cent). With that #{S < x} is known at every bin edge of the
// first window, which gives c, and #{|S - c| <= d} at every bin edge of the
// second, whose smallest d above the rank is the MAD. Bins wider than one
// value (few samples, wide ranges) narrow the windows for another pass, with
// bounds in place of values. Where one value holds much of a series (a row
// blanked, padded or constant), its keys would all be added to the same bins:
// a sample of one value needs no histogram, and the exact pass counts the keys
// at the estimate with ballots and equal neighbours together (sps_width_stats of
// 256 x 131072, constant rows: 3.60 ms without, 1.55 with full histograms, now
// 0.74; rows blanked for two thirds: 2.91, 2.18 and 2.00). A width whose
// windows miss (data unlike their sample) is left to the general selection: its full range, then levels of
// 11-bit digits of the key's distance from the current lower bound (one
// 2048-bin LDS histogram per width): a level histograms the keys inside the
// current range, one wave per width finds the bin holding the wanted rank,
// and the range shrinks to that bin. A range of R values takes
// ceil(log2(R) / 11) levels (at most three), so the median takes one to three
// passes and the MAD as many again. Keys are S with the sign bit flipped
// (unsigned order = signed order); MAD keys are |S - c_w| as uint32.
// 256 x 131072, widths to 4096: 1.19 -> 0.59 ms; the whole of sps_width_stats (its
// block statistics became faster too): 64 x 2^19 5.28 -> 2.10 ms; 2000 x 5000,
// widths to 1024, 1.27 -> 0.66 ms; where the windows miss, 256 x 131072 with every
// 4th sample unlike the rest, 1.62 -> 1.45 ms.
#include <climits>
#include <type_traits>

#include "sps_internal.h"
#include "sps_wave.h"

namespace sps {

namespace {

constexpr int kWT = 1024;           // threads per workgroup
constexpr int kWaves = kWT / 64;
constexpr int kWStep = 4 * kWT;     // samples per step (4 per thread)
constexpr int kWRing = 2 * kWStep;  // prefix sums of two steps
constexpr int kWBits = 11;
constexpr int kWBins = 1 << kWBits; // histogram bins per width and level

__device__ __forceinline__ uint32_t absdiff_u(int a, int b) {
  return a >= b ? (uint32_t)a - (uint32_t)b : (uint32_t)b - (uint32_t)a;
}

__device__ __forceinline__ int bits_of(uint32_t r) { return r == 0u ? 0 : 32 - __clz((int)r); }

constexpr int kWMid = 512, kWSide = 768;  // bins of the three windows (512 + 2 x 768 = kWBins)
static_assert(kWMid + 2 * kWSide == kWBins, "the windows fill a width's histogram");
// A width is dense when more than one in so many sampled keys is in the median's
// bin, and that is no wider than so many bits (a wider one holds that many keys
// of any series with a few far values): many of these keys have one value, and
// would all be added to the same bins.
constexpr uint32_t kDenseShare = 8;
constexpr int kDenseShift = 6;

// Windows of the exact pass, on keys: the median's, [mlo, mlo + lim[0]), and
// that of the distances from the key cen, [dlo, dlo + lim[1]), keys below cen
// and keys from cen on in histograms of their own; bin shifts.
struct __align__(16) WidthWindows {
  uint32_t mlo, cen, dlo;
  uint32_t lim[2];
  int32_t sh[2];
  int32_t dense;  // much of the series is expected to equal cen
};

struct WidthShared {
  uint32_t ring[kWRing];
  uint32_t hist[kMaxWidths][kWBins];
  uint32_t wtot[2][kWaves];
  int32_t mn[kMaxWidths], mx[kMaxWidths];
  // selection state per width: lower bound of the key range, bucket shift of
  // the level (-1: finished or no positions), rank sought, result key
  uint32_t lo[kMaxWidths];
  int32_t sh[kMaxWidths];
  uint32_t rank[kMaxWidths];
  uint32_t res[kMaxWidths];
  int32_t cen[kMaxWidths];  // the median c_w
  WidthWindows win[kMaxWidths];
  uint32_t below[kMaxWidths][2];  // keys below the first window, distances below the second
  // 1 while the width is sought by windows (2: they are set, no histogram of
  // the sample), 0 when its cen and res are final, -1 when it is left to the
  // general selection
  int32_t live[kMaxWidths];
};

// Streams the row once; for every step and width with its bit in `active`
// calls f(j, key, clean, v) with the keys S[q] ^ 0x80000000 of the boxcar sums
// of the thread's first QN window ends E = E0 + q (position E - w). v[q]:
// w <= E <= N; clean: true for all of the workgroup, v is not to be read.
// Otherwise the keys with v[q] false are replaced by kNoKey.
constexpr uint32_t kNoKey = 0xFFFFFFFFu;

template <int NW, int QN, class F>
__device__ __forceinline__ void stream_row(const WidthStatsArgs& A, const int row, WidthShared& sm, const int nw,
                                           const uint32_t active, F&& f) {
  const int tid = threadIdx.x, lane = lane_id(), wave = readfirst(tid >> 6);
  const float* xr = A.x + (int64_t)row * A.ld;
  const int32_t* mr = A.med + (int64_t)row * A.nblocks;
  const int N = A.N;
  const int nsteps = N / kWStep + 1;  // window ends 0 .. N
  const bool vec = (reinterpret_cast<uintptr_t>(xr) & 15u) == 0;
  // The next step's samples are loaded before this one is evaluated: the one
  // workgroup of a CU waits for its loads together.
  float f0, f1, f2, f3;
  int m;
  auto fetch = [&](int c) {
    const int t0 = c * kWStep + 4 * tid;
    m = mr[min(t0, N - 1) >> 6];  // the four samples share one 64-sample block
    if (vec && (c + 1) * kWStep <= N) {
      const float4 v = *reinterpret_cast<const float4*>(xr + t0);
      f0 = v.x; f1 = v.y; f2 = v.z; f3 = v.w;
    } else {
      f0 = xr[min(t0, N - 1)];
      f1 = xr[min(t0 + 1, N - 1)];
      f2 = xr[min(t0 + 2, N - 1)];
      f3 = xr[min(t0 + 3, N - 1)];
    }
  };
  fetch(0);
  uint32_t carry = 0;
  for (int c = 0; c < nsteps; ++c) {
    const int t0 = c * kWStep + 4 * tid;
    const int r0 = t0 < N ? (int)f0 - m : 0, r1 = t0 + 1 < N ? (int)f1 - m : 0;
    const int r2 = t0 + 2 < N ? (int)f2 - m : 0, r3 = t0 + 3 < N ? (int)f3 - m : 0;
    const uint32_t p0 = (uint32_t)r0, p1 = p0 + (uint32_t)r1, p2 = p1 + (uint32_t)r2, p3 = p2 + (uint32_t)r3;
    const uint32_t incl = (uint32_t)wave_scan_incl((int)p3);
    if (lane == 63) sm.wtot[c & 1][wave] = incl;
    if (c + 1 < nsteps) fetch(c + 1);
    __syncthreads();  // also: every wave is done with the ring half written below
    uint32_t woff = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      const uint32_t v = sm.wtot[c & 1][k];
      woff += k < wave ? v : 0u;
      tot += v;
    }
    // P[E0 + q] = sum of r over the row's first E0 + q samples
    const uint32_t pb = carry + woff + incl - p3;
    const uint4 pe = make_uint4(pb, pb + p0, pb + p1, pb + p2);
    const int E0 = c * kWStep + 4 * tid;
    *reinterpret_cast<uint4*>(&sm.ring[E0 & (kWRing - 1)]) = pe;
    carry += tot;
    const uint32_t kx = pe.x ^ 0x80000000u, ky = pe.y ^ 0x80000000u, kz = pe.z ^ 0x80000000u, kw = pe.w ^ 0x80000000u;
    const bool clean = c > 0 && (c + 1) * kWStep - 1 <= N;  // (widths are at most one step)
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      if (!((active >> j) & 1u)) continue;  // (no bits from nw on)
      const int w = 1 << j;
      uint4 ps;
      if (w >= 4 || QN == 1) {
        // E0 - w is a multiple of 4 for QN = 4; when it is negative every end is invalid
        if (QN == 1) ps.x = sm.ring[(E0 - w) & (kWRing - 1)];
        else ps = *reinterpret_cast<const uint4*>(&sm.ring[(E0 - w) & (kWRing - 1)]);
      } else {
        ps.x = sm.ring[(E0 - w) & (kWRing - 1)];
        ps.y = sm.ring[(E0 + 1 - w) & (kWRing - 1)];
        ps.z = sm.ring[(E0 + 2 - w) & (kWRing - 1)];
        ps.w = sm.ring[(E0 + 3 - w) & (kWRing - 1)];
      }
      uint32_t key[QN];
      bool v[QN];
#pragma unroll
      for (int q = 0; q < QN; ++q) {
        key[q] = q == 0 ? kx - ps.x : q == 1 ? ky - ps.y : q == 2 ? kz - ps.z : kw - ps.w;
        v[q] = E0 + q >= w && E0 + q <= N;
      }
      if (!clean) {
#pragma unroll
        for (int q = 0; q < QN; ++q) key[q] = v[q] ? key[q] : kNoKey;
      }
      f(j, key, clean, v);
    }
  }
  __syncthreads();
}

// The thread's four keys are one (long runs of one value: a row blanked or padded).
__device__ __forceinline__ bool all_equal(const uint32_t (&key)[4]) {
  return (key[0] == key[1]) & (key[1] == key[2]) & (key[2] == key[3]);
}

// Adds the thread's keys in range to width j's histogram (equal neighbouring
// buckets merged into one atomic).
__device__ __forceinline__ void hist_keys(uint32_t* h, const uint32_t (&key)[4], const bool (&v)[4], uint32_t lo,
                                          int sh) {
  uint32_t prev = 0xFFFFFFFFu, cnt = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t d = key[q] - lo;
    const bool in = v[q] && key[q] >= lo && (d >> sh) < (uint32_t)kWBins;
    const uint32_t b = d >> sh;
    if (in) {
      if (b == prev) {
        ++cnt;
      } else {
        if (cnt) atomicAdd(&h[prev], cnt);
        prev = b;
        cnt = 1;
      }
    }
  }
  if (cnt) atomicAdd(&h[prev], cnt);
}

// One wave per active width: the bin of the histogram holding the wanted
// rank; the range shrinks to it (or the key is found), the histogram is
// cleared for the next level.
__device__ __forceinline__ void resolve_level(WidthShared& sm, const int nw) {
  const int wave = threadIdx.x >> 6, lane = lane_id();
  for (int j = wave; j < nw; j += kWaves) {
    const int sh = sm.sh[j];
    uint32_t* h = sm.hist[j];
    if (sh >= 0) {
      uint32_t b32[32];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint4 v = *reinterpret_cast<const uint4*>(&h[32 * lane + 4 * k]);
        b32[4 * k] = v.x; b32[4 * k + 1] = v.y; b32[4 * k + 2] = v.z; b32[4 * k + 3] = v.w;
      }
      uint32_t s = 0;
#pragma unroll
      for (int k = 0; k < 32; ++k) s += b32[k];
      const uint32_t incl = (uint32_t)wave_scan_incl((int)s);  // at most 2^31 keys per row
      const uint32_t rank = sm.rank[j];
      const uint64_t mk = ballot(incl > rank);  // the range holds more than rank keys
      const int L = mk ? ctz(mk) : 63;
      uint32_t r = rank - ((uint32_t)readlane((int)incl, L) - (uint32_t)readlane((int)s, L));
      // within lane L's 32 bins (evaluated in every lane, used from lane L)
      int bin = 31;
      bool found = false;
#pragma unroll
      for (int k = 0; k < 32; ++k) {
        const bool here = !found && r < b32[k];
        bin = here ? k : bin;
        found = found || here;
        r = (found || here) ? r : r - b32[k];
      }
      const int B = 32 * L + readlane(bin, L);
      const uint32_t rr = (uint32_t)readlane((int)r, L);
      if (lane == 0) {
        const uint32_t lo = sm.lo[j] + ((uint32_t)B << sh);
        if (sh == 0) {
          sm.res[j] = lo;
          sm.sh[j] = -1;
        } else {
          sm.lo[j] = lo;
          sm.rank[j] = rr;
          sm.sh[j] = sh > kWBits ? sh - kWBits : 0;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) *reinterpret_cast<uint4*>(&h[32 * lane + 4 * k]) = make_uint4(0u, 0u, 0u, 0u);
  }
}

// Exclusive prefix sums of a width's histogram in place, by one wave; returns the total.
__device__ __forceinline__ uint32_t prefix_bins(uint32_t* h, const int lane) {
  uint32_t b32[32];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint4 v = *reinterpret_cast<const uint4*>(&h[32 * lane + 4 * k]);
    b32[4 * k] = v.x; b32[4 * k + 1] = v.y; b32[4 * k + 2] = v.z; b32[4 * k + 3] = v.w;
  }
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < 32; ++k) s += b32[k];
  const uint32_t incl = (uint32_t)wave_scan_incl((int)s);
  uint32_t run = incl - s;
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const uint32_t v = b32[k];
    b32[k] = run;
    run += v;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k)
    *reinterpret_cast<uint4*>(&h[32 * lane + 4 * k]) = make_uint4(b32[4 * k], b32[4 * k + 1], b32[4 * k + 2], b32[4 * k + 3]);
  wave_lds_fence();
  return (uint32_t)readlane((int)incl, 63);
}

__device__ __forceinline__ void clear_bins(uint32_t* h, const int lane) {
  wave_lds_fence();
#pragma unroll
  for (int k = 0; k < 8; ++k) *reinterpret_cast<uint4*>(&h[32 * lane + 4 * k]) = make_uint4(0u, 0u, 0u, 0u);
}

// The smallest shift with (bins << shift) >= span (at most 2^32 values).
__device__ __forceinline__ int window_shift(int64_t span, int bins) {
  int g = 0;
  while (g < 31 && ((int64_t)bins << g) < span) ++g;
  return g;
}

// Windows of width j about the median key c (in [c - em, c + em]) and the MAD
// d (in [d - ed, d + ed]), or live -1 where they would leave the keys' range.
// One lane.
__device__ __forceinline__ void set_windows(WidthShared& sm, const int j, const int64_t m0, const int64_t mspan,
                                            const int64_t cen, const int64_t d0, const int64_t dspan,
                                            const bool dense) {
  WidthWindows& w = sm.win[j];
  const int gm = window_shift(mspan, kWMid), gd = window_shift(dspan, kWSide);
  const int64_t dlo = d0 > 0 ? d0 : 0;
  const int64_t lm = ((mspan >> gm) + 1) << gm, ld = ((dspan >> gd) + 1) << gd;  // whole bins
  const int64_t lim0 = lm < ((int64_t)kWMid << gm) ? lm : (int64_t)kWMid << gm;
  const int64_t lim1 = ld < ((int64_t)kWSide << gd) ? ld : (int64_t)kWSide << gd;
  const bool ok = gm <= 20 && gd <= 20 && m0 >= 0 && m0 + lim0 < (int64_t)kNoKey && cen >= 0 &&
                  cen + dlo + lim1 < (int64_t)kNoKey;
  w.mlo = (uint32_t)m0;
  w.cen = (uint32_t)cen;
  w.dlo = (uint32_t)dlo;
  w.lim[0] = (uint32_t)lim0;
  w.lim[1] = (uint32_t)lim1;
  w.sh[0] = gm;
  w.sh[1] = gd;
  w.dense = dense;
  sm.below[j][0] = sm.below[j][1] = 0u;
  sm.live[j] = ok ? 1 : -1;
}

// The smallest of x .. y for which the monotone f holds (it does for y), by one
// wave, 64 candidates at a time: the search waits for one read of LDS a round,
// two or three rounds for a window's bins.
template <class F>
__device__ __forceinline__ int first_of(int x, int y, const int lane, F&& f) {
  while (x < y) {
    const int step = (int)(((uint32_t)(y - x) + 63u) >> 6);
    const uint64_t mk = ballot(f((int)min((int64_t)x + (int64_t)lane * step, (int64_t)y)));
    if (!mk) {
      x += 63 * step + 1;  // at most y, for which it holds
    } else {
      const int k = ctz(mk);
      y = min(x + k * step, y);
      if (k) x += (k - 1) * step + 1;
    }
  }
  return y;
}

// First windows of width j from the histogram of its samples (lo, sh), by one
// wave: median and MAD by linear interpolation in the bins. `whole`: the
// samples are the whole series.
__device__ __forceinline__ void aim_windows(WidthShared& sm, const int j, const int lane, const bool whole,
                                            const double spread) {
  uint32_t* h = sm.hist[j];
  const int sh = sm.sh[j];
  const uint32_t tot = prefix_bins(h, lane);
  const double bin = (double)(1u << sh);
  if (tot == 0u || sh > 20) {
    if (lane == 0) sm.live[j] = -1;
  } else {
    auto pre = [&](int k) { return k >= kWBins ? tot : h[k]; };
    // interpolated #{key < lo + x}
    auto F = [&](double x) -> double {
      if (x <= 0.0) return 0.0;
      const double q = x / bin;
      const int k = q >= (double)kWBins ? kWBins : (int)q;
      const uint32_t a = pre(k), b = pre(k + 1);
      return (double)a + (q - (double)k) * (double)(b - a);
    };
    const uint32_t rank = (tot - 1u) >> 1;
    const int k = first_of(0, kWBins - 1, lane, [&](int b) { return pre(b + 1) > rank; });
    const uint32_t cnt = pre(k + 1) - pre(k);  // at least 1
    const double c = bin * ((double)k + ((double)(rank - pre(k)) + 0.5) / (double)cnt);
    const double half = 0.5 * (double)tot;
    double dl = 0.0, dh = bin * (double)kWBins;
    while (dh - dl > 0.25) {  // 64 distances at a time
      const double step = (dh - dl) * (1.0 / 64.0), d = dl + step * (double)(lane + 1);
      const uint64_t mk = ballot(F(c + d) - F(c - d) > half);
      if (!mk) break;
      dl += step * (double)ctz(mk);
      dh = dl + step;
    }
    // how far the estimates may be off: the interpolation and three deviations
    // of the sampled rank (fewer where neighbouring positions share samples)
    const double err = 0.25 * bin + (whole ? bin : bin * sqrt((double)tot) / (2.0 * (double)cnt) * spread);
    const int64_t em = (int64_t)err + 32, ed = (int64_t)(2.0 * err) + 32;
    const int64_t ck = (int64_t)sm.lo[j] + (int64_t)c;
    const bool dense = sh <= kDenseShift && cnt > tot / kDenseShare;
    if (lane == 0) set_windows(sm, j, ck - em, 2 * em, ck, (int64_t)dh - ed, 2 * ed, dense);
  }
  clear_bins(h, lane);
}

// After an exact pass, by one wave: c_w and MAD_w of width j (live 0),
// narrower windows (live 1), or a miss (live -1).
__device__ __forceinline__ void read_windows(WidthShared& sm, const int j, const int lane, const int n) {
  uint32_t* h = sm.hist[j];
  const uint32_t tot = prefix_bins(h, lane);
  const uint32_t rho = (uint32_t)(n - 1) >> 1;
  WidthWindows w = sm.win[j];  // the same in every lane: scalar branches and loops
  w.mlo = (uint32_t)readfirst((int)w.mlo);
  w.cen = (uint32_t)readfirst((int)w.cen);
  w.dlo = (uint32_t)readfirst((int)w.dlo);
  w.lim[0] = (uint32_t)readfirst((int)w.lim[0]);
  w.lim[1] = (uint32_t)readfirst((int)w.lim[1]);
  const int gm = readfirst(w.sh[0]), gs = readfirst(w.sh[1]);
  const uint32_t bm = (uint32_t)readfirst((int)sm.below[j][0]), bd = (uint32_t)readfirst((int)sm.below[j][1]);
  const uint32_t p0 = (uint32_t)readfirst((int)h[kWMid]), p1 = (uint32_t)readfirst((int)h[kWMid + kWSide]);
  const int nm = (int)(w.lim[0] >> gm), nd = (int)(w.lim[1] >> gs);  // bins in use
  auto FM = [&](int k) { return bm + h[k]; };  // #{key < mlo + (k << gm)}, k <= nm
  // keys below cen (L) and from it on (U) at distances dlo .. dlo + (k << gs) - 1, k <= nd
  auto CL = [&](int k) { return (int)(h[kWMid + k] - p0); };
  auto CU = [&](int k) { return (int)((k == kWSide ? tot : h[kWMid + kWSide + k]) - p1); };
  int live = -1;
  int64_t c0 = 0, d1 = 0, d2 = 0;
  const int64_t cw = (int64_t)1 << gm;
  if (FM(0) <= rho && FM(nm) > rho) {
    const int a = first_of(1, nm, lane, [&](int k) { return FM(k) > rho; }) - 1;
    c0 = (int64_t)w.mlo + ((int64_t)a << gm);  // c in [c0, c0 + cw)
    // #{|key - c| <= d} = bd + the keys from cen on up to c + d + those below
    // it down to c - d, less those on the far side of c that are further than
    // d from it (c +- d need not reach cen when d < |c - cen|): at most
    // upper, at least lower, for any such c, from the nearest bin edges. D = d -
    // dlo in [da, db] keeps both ends inside the window, and the keys nearer to
    // cen than it within d of c; with none of those (dlo = 0) any d may be
    // asked, and only then are there keys on the far side. (Windows are shorter
    // than 2^30, so all of this fits 32 bits.)
    const int g = 1 << gs;
    const bool far = w.dlo == 0u;
    const int u0 = (int)(c0 - (int64_t)w.cen), u1 = u0 + (int)cw - 1;  // c - cen in [u0, u1]
    const int umin = min(u0, -u1), umax = -umin;
    const int da = far ? 0 : -1 - umin, db = (nd << gs) - 1 - umax;
    // distances dlo .. dlo + x: x + 1 values
    auto up = [&](int x) { return x < 0 ? 0 : (x + g) >> gs; };
    auto down = [&](int x) { return x < 0 ? 0 : (x + 1) >> gs; };
    auto upper = [&](int D) {
      const int n = (int)bd + CU(up(u1 + D)) + CL(up(D - u0));
      return far ? n - CU(down(u0 - D - 1)) - CL(down(-u1 - D - 1)) : n;
    };
    auto lower = [&](int D) {
      const int n = (int)bd + CU(down(u0 + D)) + CL(down(D - u1));
      return far ? n - CU(up(u1 - D - 1)) - CL(up(-u0 - D - 1)) : n;
    };
    const bool first_d = (int64_t)w.dlo + da == 0;  // no smaller d to rule out
    if (da <= db && lower(db) > (int)rho && (first_d || upper(da) <= (int)rho)) {
      d1 = (int64_t)w.dlo + first_of(da, db, lane, [&](int D) { return upper(D) > (int)rho; });
      d2 = (int64_t)w.dlo + first_of(da, db, lane, [&](int D) { return lower(D) > (int)rho; });
      live = d1 == d2 && cw == 1 ? 0 : 1;
    }
  }
  if (lane == 0) {
    sm.live[j] = live;
    if (live == 0) {
      sm.cen[j] = (int)((uint32_t)c0 ^ 0x80000000u);
      sm.res[j] = (uint32_t)d1;
    } else if (live == 1) {
      // counts are exact at bin edges only, so the next windows count their own
      // keys below; margins so that the answer is not the first d tested
      set_windows(sm, j, c0, cw, c0 + cw / 2, d1 - cw - 2, d2 - d1 + 2 * cw + 6, w.dense);
      if (sm.win[j].sh[0] >= gm && sm.win[j].sh[1] >= gs) sm.live[j] = -1;  // no progress
    }
  }
  clear_bins(h, lane);
}

template <int NW>
__global__ __launch_bounds__(kWT) void k_width_stats(WidthStatsArgs A) {
  __shared__ WidthShared sm;
  constexpr int NWU = NW > 0 ? NW : kMaxWidths;  // widths unrolled in the streaming loop
  const int row = blockIdx.x;
  const int tid = threadIdx.x, lane = lane_id(), wave = readfirst(tid >> 6);
  const int nw = NW > 0 ? NW : A.nw;
  const int N = A.N;
  for (int i = tid; i < kMaxWidths * kWBins; i += kWT) (&sm.hist[0][0])[i] = 0u;
  if (tid < kMaxWidths) {
    sm.mn[tid] = INT_MAX;
    sm.mx[tid] = INT_MIN;
    sm.cen[tid] = 0;  // widths longer than the row: c_w = 0, MAD 0
    sm.res[tid] = 0u;
    sm.live[tid] = tid < nw && (1 << tid) <= N ? 1 : 0;
  }
  __syncthreads();
  auto widths_with = [&](int state) {
    uint32_t m = 0;
    for (int j = 0; j < nw; ++j) m |= sm.live[j] == state ? 1u << j : 0u;
    return (uint32_t)readfirst((int)m);
  };

  // Key range of the series, of all positions or of every 4th.
  auto range_pass = [&](uint32_t active, auto QN) {
    uint32_t mn[kMaxWidths], mx[kMaxWidths];
#pragma unroll
    for (int j = 0; j < kMaxWidths; ++j) {
      mn[j] = kNoKey;
      mx[j] = 0u;
    }
    stream_row<NWU, QN.value>(A, row, sm, nw, active,
                              [&](int j, const uint32_t (&key)[QN.value], bool clean, const bool (&v)[QN.value]) {
#pragma unroll
      for (int q = 0; q < QN.value; ++q) {
        mn[j] = min(mn[j], key[q]);
        if (clean) mx[j] = max(mx[j], key[q]);
        else mx[j] = v[q] ? max(mx[j], key[q]) : mx[j];
      }
    });
#pragma unroll
    for (int j = 0; j < kMaxWidths; ++j) {
      if (j >= nw || !((active >> j) & 1u)) continue;
      const int a = wave_min_u((int)(mn[j] ^ 0x80000000u)), b = wave_max_u((int)(mx[j] ^ 0x80000000u));
      if (lane == 0) {
        atomicMin(&sm.mn[j], a);
        atomicMax(&sm.mx[j], b);
      }
    }
    __syncthreads();
  };
  using One = std::integral_constant<int, 1>;
  using Four = std::integral_constant<int, 4>;

  // ---- sampled estimates and exact windows
  {
    const bool whole = N < 32768;
    if (whole) range_pass(widths_with(1), Four{});
    else range_pass(widths_with(1), One{});
    if (tid < nw && sm.live[tid] == 1) {
      const int j = tid;
      const uint32_t lo = (uint32_t)sm.mn[j] ^ 0x80000000u, hi = (uint32_t)sm.mx[j] ^ 0x80000000u;
      sm.lo[j] = lo;
      sm.sh[j] = max(0, bits_of(hi - lo) - kWBits);
      if (sm.mn[j] > sm.mx[j]) {
        sm.live[j] = -1;  // no sampled position
      } else if (lo == hi) {
        set_windows(sm, j, (int64_t)lo - 32, 64, lo, 0, 64, true);  // nothing to sort into bins
        if (sm.live[j] == 1) sm.live[j] = 2;
      }
    }
    __syncthreads();
    {
      uint32_t lo[kMaxWidths];
      int sh[kMaxWidths];
#pragma unroll
      for (int j = 0; j < kMaxWidths; ++j) {
        lo[j] = j < nw ? sm.lo[j] : 0u;
        sh[j] = j < nw ? sm.sh[j] : 0;
      }
      // wide boxcars change little over 16 positions: a quarter of the lanes, in a long row
      const bool sparse = N >= 131072 && (lane & 3) != 0;
      auto count = [&](int j, uint32_t key, uint32_t n) {
        const uint32_t b = (key - lo[j]) >> sh[j];
        if (key != kNoKey && b < (uint32_t)kWBins && !(sparse && j >= 6)) atomicAdd(&sm.hist[j][b], n);
      };
      const uint32_t active = widths_with(1);
      if (whole)
        stream_row<NWU, 4>(A, row, sm, nw, active, [&](int j, const uint32_t (&key)[4], bool, const bool (&)[4]) {
          if (all_equal(key)) {
            count(j, key[0], 4u);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) count(j, key[q], 1u);
          }
        });
      else
        stream_row<NWU, 1>(A, row, sm, nw, active,
                           [&](int j, const uint32_t (&key)[1], bool, const bool (&)[1]) { count(j, key[0], 1u); });
    }
    for (int j = wave; j < nw; j += kWaves)
      if (sm.live[j] == 1) aim_windows(sm, j, lane, whole, j < 6 ? 3.0 : 3.0 * fmax(sqrt(32.0 / (double)(1 << j)), 0.3));
    __syncthreads();
    if (tid < nw && sm.live[tid] == 2) sm.live[tid] = 1;
    __syncthreads();
    for (int pass = 0; pass < 4; ++pass) {
      const uint32_t active = widths_with(1);
      if (!active) break;
      uint32_t below[kMaxWidths][2];
#pragma unroll
      for (int j = 0; j < kMaxWidths; ++j) below[j][0] = below[j][1] = 0u;
      uint32_t dense = 0;
      for (int j = 0; j < nw; ++j) dense |= sm.win[j].dense ? 1u << j : 0u;
      dense = (uint32_t)readfirst((int)(dense & active));
      auto count = [&](int j, const uint32_t (&key)[4], auto DENSE) {
        const WidthWindows w = sm.win[j];
        const uint32_t ndlo = 0u - w.dlo;
        uint32_t* h = sm.hist[j];
        bool at_cen[4];
        if (DENSE) {
          // the keys that equal cen by ballots, one addition to each of their bins for the wave
          int n = 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            at_cen[q] = key[q] == w.cen;
            n += popc(ballot(at_cen[q]));
          }
          if (lane == 0 && n) {
            if (w.cen - w.mlo < w.lim[0]) atomicAdd(&h[(w.cen - w.mlo) >> w.sh[0]], (uint32_t)n);
            if (w.dlo == 0u) atomicAdd(&h[kWMid + kWSide], (uint32_t)n);
          }
        }
        // one branch for the four keys: most waves have none inside a wide boxcar's windows
        uint32_t t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          t[q] = key[q] - w.mlo;
          if (DENSE) t[q] = at_cen[q] ? kNoKey : t[q];
          below[j][0] += key[q] < w.mlo ? 1u : 0u;
        }
        if (min(min(t[0], t[1]), min(t[2], t[3])) < w.lim[0]) {
          if (DENSE && all_equal(key)) {
            atomicAdd(&h[t[0] >> w.sh[0]], 4u);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (t[q] < w.lim[0]) atomicAdd(&h[t[q] >> w.sh[0]], 1u);
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // |key - cen| - dlo, modulo 2^32: above ~dlo for the distances below dlo
          asm("v_sad_u32 %0, %1, %2, %3" : "=v"(t[q]) : "v"(key[q]), "v"(w.cen), "v"(ndlo));
          below[j][1] += t[q] > ~w.dlo ? 1u : 0u;
          if (DENSE) t[q] = at_cen[q] ? kNoKey : t[q];
        }
        if (min(min(t[0], t[1]), min(t[2], t[3])) < w.lim[1]) {
          if (DENSE && all_equal(key)) {
            atomicAdd(&h[(key[0] < w.cen ? kWMid : kWMid + kWSide) + (t[0] >> w.sh[1])], 4u);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (t[q] < w.lim[1])
                atomicAdd(&h[(key[q] < w.cen ? kWMid : kWMid + kWSide) + (t[q] >> w.sh[1])], 1u);
          }
        }
      };
      // (a loop of its own for rows with dense widths: their branch in every
      // row's loop cost 4 %)
      if (dense)
        stream_row<NWU, 4>(A, row, sm, nw, active, [&](int j, const uint32_t (&key)[4], bool, const bool (&)[4]) {
          if ((dense >> j) & 1u) count(j, key, std::true_type{});
          else count(j, key, std::false_type{});
        });
      else
        stream_row<NWU, 4>(A, row, sm, nw, active, [&](int j, const uint32_t (&key)[4], bool, const bool (&)[4]) {
          count(j, key, std::false_type{});
        });
#pragma unroll
      for (int j = 0; j < kMaxWidths; ++j) {
        if (j >= nw || !((active >> j) & 1u)) continue;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int b = wave_sum_u((int)below[j][k]);
          if (lane == 0 && b) atomicAdd(&sm.below[j][k], (uint32_t)b);
        }
      }
      __syncthreads();
      for (int j = wave; j < nw; j += kWaves)
        if (sm.live[j] == 1) read_windows(sm, j, lane, N - (1 << j) + 1);
      __syncthreads();
    }
  }

  // ---- general selection of the widths that are left
  if (tid < nw && sm.live[tid] == 1) sm.live[tid] = -1;
  __syncthreads();
  const uint32_t rest = widths_with(-1);
  if (rest) {
    if (tid < kMaxWidths) {
      sm.mn[tid] = INT_MAX;
      sm.mx[tid] = INT_MIN;
      sm.sh[tid] = -1;
    }
    __syncthreads();
    range_pass(rest, Four{});
    // median of each series: keys S ^ 0x80000000 in [key(min), key(max)]
    if (tid < nw && ((rest >> tid) & 1u)) {
      const int j = tid, n = N - (1 << j) + 1;
      const uint32_t lo = (uint32_t)sm.mn[j] ^ 0x80000000u, hi = (uint32_t)sm.mx[j] ^ 0x80000000u;
      sm.lo[j] = lo;
      sm.rank[j] = (uint32_t)((n - 1) >> 1);
      sm.sh[j] = max(0, bits_of(hi - lo) - kWBits);
    }
    __syncthreads();
    for (int mad = 0; mad < 2; ++mad) {
      int cj[kMaxWidths];
      if (mad) {
        // MAD of each series: keys |S - c| in [0, max(max - c, c - min)]
        if (tid < nw && ((rest >> tid) & 1u)) {
          const int j = tid, n = N - (1 << j) + 1;
          const int c = (int)(sm.res[j] ^ 0x80000000u);
          sm.cen[j] = c;
          sm.lo[j] = 0u;
          const uint32_t r = max(absdiff_u(sm.mx[j], c), absdiff_u(c, sm.mn[j]));
          sm.rank[j] = (uint32_t)((n - 1) >> 1);
          sm.sh[j] = max(0, bits_of(r) - kWBits);
        }
        __syncthreads();
      }
#pragma unroll
      for (int j = 0; j < kMaxWidths; ++j) cj[j] = j < nw ? sm.cen[j] : 0;
      for (int level = 0; level < 3; ++level) {
        uint32_t active = 0;
        for (int j = 0; j < nw; ++j) active |= sm.sh[j] >= 0 ? 1u << j : 0u;
        active = (uint32_t)readfirst((int)active);
        if (!active) break;
        uint32_t lo[kMaxWidths];
        int sh[kMaxWidths];
#pragma unroll
        for (int j = 0; j < kMaxWidths; ++j) {
          lo[j] = j < nw ? sm.lo[j] : 0u;
          sh[j] = j < nw ? sm.sh[j] : -1;
        }
        stream_row<NWU, 4>(A, row, sm, nw, active,
                           [&](int j, const uint32_t (&key)[4], bool, const bool (&v)[4]) {
          uint32_t k[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) k[q] = mad ? absdiff_u((int)(key[q] ^ 0x80000000u), cj[j]) : key[q];
          hist_keys(sm.hist[j], k, v, lo[j], sh[j]);
        });
        resolve_level(sm, nw);
        __syncthreads();
      }
    }
  }
  if (tid < nw) {
    const int64_t o = (int64_t)row * nw + tid;
    A.center[o] = sm.cen[tid];
    // a MAD beyond INT32_MAX (half the series more than 2^31 from its median)
    // is reported as INT32_MAX
    A.mad[o] = (int32_t)min(sm.res[tid], (uint32_t)INT_MAX);
  }
}

}  // namespace

hipError_t launch_width_stats(const WidthStatsArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  if (a.nw == kMaxWidths) hipLaunchKernelGGL((k_width_stats<kMaxWidths>), dim3(a.rows), dim3(kWT), 0, s, a);
  else hipLaunchKernelGGL((k_width_stats<0>), dim3(a.rows), dim3(kWT), 0, s, a);
  return hipGetLastError();
}

}  // namespace sps
