// sps_chain.h - the baseline and normalisation chain (Heimdall++, Section
// II-B): the device code behind k_block_stats, shared by the statistics
// kernels and the fused batch kernel. See sps_stats.hip for the design.
#pragma once

#include "sps_internal.h"
#include "sps_wave.h"

namespace sps {

namespace {

// Virtual row: samples t < Hx come from the stream history h, the rest from
// the input g (g[t - Hx]). VIRT = false: no history, t indexes g directly.
template <bool VIRT>
struct RowRef {
  gbl_f32* g;
  gbl_f32* h;
  int Hx;
  __device__ __forceinline__ float at(int t) const {
    if (VIRT) return *(t < Hx ? h + t : g + (t - Hx));  // one load from the selected address
    return g[t];
  }
  __device__ __forceinline__ int iat(int t) const { return (int)at(t); }
};

__device__ __forceinline__ uint32_t absdiff(int v, int m) {
  return v >= m ? (uint32_t)v - (uint32_t)m : (uint32_t)m - (uint32_t)v;
}

__device__ __forceinline__ void hist_add(uint32_t* H, uint32_t idx, uint32_t one) {
  // one = 1 (insert) or 0xFFFFFFFF (remove); the count lives in the idx&1 half
  atomicAdd(&H[idx >> 1], one << ((idx & 1u) << 4));
}

__device__ __forceinline__ int hist_get(const uint32_t* H, int idx) {
  return (int)((H[idx >> 1] >> ((idx & 1) << 4)) & 0xFFFFu);
}

template <int NB, bool VIRT>
struct Chain {
  uint32_t* H;        // this wave's NB/2 histogram words
  RowRef<VIRT> row;
  int L;
  int lane;
  int base;           // value of histogram bin 0
  int n;              // window size
  int m, cm;          // median, #{x < m}
  int d, cL, cU;      // MAD, #{x < m - d}, #{x < m + d + 1}
  bool raw;           // histogram not maintained (data too spread)
};

// f(x, ok) for samples lo + lane, lo + 64 + lane, ... of the window [lo, hi) (ok:
// inside it; else x is its last sample). Bound by load latency: the next eight
// wave loads are in flight while eight are used (one load at a time, a
// 4096-sample recount took 64 dependent round trips to L2).
template <bool VIRT, class F>
__device__ __forceinline__ void each_sample(const RowRef<VIRT>& row, int lo, int hi, int lane, F&& f) {
  constexpr int kU = 8;
  float nv[kU];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int q = 0; q < kU; ++q) nv[q] = row.at(min(t0 + 64 * q + lane, hi - 1));
  };
  fetch(lo);
  int t0 = lo;
  for (; t0 + 64 * kU <= hi; t0 += 64 * kU) {
    float v[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) v[q] = nv[q];
    fetch(t0 + 64 * kU);
#pragma unroll
    for (int q = 0; q < kU; ++q) f((int)v[q], true);
  }
#pragma unroll
  for (int q = 0; q < kU; ++q)
    if (t0 + 64 * q < hi) f((int)nv[q], t0 + 64 * q + lane < hi);
}

// Element of 0-based rank `rank` of the keys of samples [lo, hi):
// MODE 0 keys are x ^ 0x80000000 (order of int32 x), MODE 1 keys are |x - m|.
// Four passes over the window, 8 key bits each; H[0..255] serves as the
// digit histogram (callers recount or abandon the value histogram afterwards).
// The upper digits are one value for most samples, whose additions to one word
// would take their turns in LDS: the lanes that share the first lane's digit
// make one (256 x 131072, window 4096, noise of sigma 20000: 31.0 ms with one
// load and one addition at a time, 28.9 with eight loads in flight, now 12.9).
template <int MODE, bool VIRT>
__device__ __forceinline__ uint32_t radix_select(uint32_t* H, const RowRef<VIRT>& row, int lo, int hi, int rank, int m, int lane) {
  uint32_t prefix = 0, pmask = 0;
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int i = lane; i < 256; i += 64) H[i] = 0;
    wave_lds_fence();
    each_sample(row, lo, hi, lane, [&](int v, bool ok) {
      const uint32_t key = MODE == 0 ? ((uint32_t)v ^ 0x80000000u) : absdiff(v, m);
      const bool in = ok && (key & pmask) == prefix;
      const uint32_t digit = (key >> shift) & 255u;
      const uint64_t any = ballot(in);
      if (any) {
        const int first = ctz(any);
        const bool same = in && digit == (uint32_t)readlane((int)digit, first);
        const int n = popc(ballot(same));
        if (in && (!same || lane == first)) atomicAdd(&H[digit], same ? (uint32_t)n : 1u);
      }
    });
    wave_lds_fence();
    const int c0 = (int)H[4 * lane], c1 = (int)H[4 * lane + 1], c2 = (int)H[4 * lane + 2];
    const int c3 = (int)H[4 * lane + 3];
    const int s = c0 + c1 + c2 + c3;
    const int inc = wave_scan_incl(s);
    const int j = ctz(ballot(inc > rank));  // total count > rank, so some lane qualifies
    int r = rank - (readlane(inc, j) - readlane(s, j));
    const int d0 = readlane(c0, j), d1 = readlane(c1, j), d2 = readlane(c2, j);
    int dig = 4 * j;
    if (r >= d0) {
      r -= d0; ++dig;
      if (r >= d1) {
        r -= d1; ++dig;
        if (r >= d2) { r -= d2; ++dig; }
      }
    }
    rank = r;
    prefix |= (uint32_t)dig << shift;
    pmask |= 0xFFu << shift;
    wave_lds_fence();
  }
  return prefix;
}

// Recount the window [lo, hi) into a histogram centred on `centre`, and the
// pivots' counts for median m0 and MAD d0 (guesses or known values) from the
// samples themselves.
template <int NB, bool VIRT>
__device__ __forceinline__ void recount(Chain<NB, VIRT>& c, int lo, int hi, int centre, int m0, int d0) {
  c.base = centre - NB / 2;
  c.m = m0;
  c.d = d0;
  for (int i = 4 * c.lane; i < NB / 2; i += 256) *reinterpret_cast<uint4*>(&c.H[i]) = make_uint4(0u, 0u, 0u, 0u);
  wave_lds_fence();
  const int pL = m0 - d0, pU = m0 + d0 + 1;
  int cm = 0, cL = 0, cU = 0;
  each_sample(c.row, lo, hi, c.lane, [&](int x, bool ok) {
    const uint64_t okm = ballot(ok);
    const uint32_t idx = (uint32_t)x - (uint32_t)c.base;
    if (ok && idx < (uint32_t)NB) hist_add(c.H, idx, 1u);
    cm += popc(ballot(x < m0) & okm);
    cL += popc(ballot(x < pL) & okm);
    cU += popc(ballot(x < pU) & okm);
  });
  wave_lds_fence();
  c.cm = cm;
  c.cL = cL;
  c.cU = cU;
  c.raw = false;
}

template <int NB>
__device__ __forceinline__ int hist_or_0(const uint32_t* H, int i) {
  const int k = min(max(i, 0), NB - 1);
  const int h = hist_get(H, k);
  return i == k ? h : 0;
}

// General query: walks from the current pivots, 64 bins a step, to the new
// median and from there to the new MAD; any distance inside the histogram.
// The cost is a few steps per 64 values moved, so a baseline that moves by a
// large part of a sigma per block (a drift shorter than the window) stays
// within a small factor of the narrow query. Returns false, with the chain
// unchanged, when a pivot leaves the histogram. It starts inside only if all
// three pivots are: a new histogram is centred on other samples than the pivots
// come from, and with samples outside the input domain the differences wrap
// (each test below is of a value that cannot).
template <int NB, bool VIRT>
__device__ __forceinline__ bool walk_query(Chain<NB, VIRT>& c) {
  const int rho = (c.n - 1) >> 1, lane = c.lane;
  const int im = (int)((uint32_t)c.m - (uint32_t)c.base);
  if ((uint32_t)im >= (uint32_t)NB || (uint32_t)c.d > (uint32_t)min(im, NB - 1 - im)) return false;
  int iL = im - c.d, iU = im + c.d + 1;  // in [0, NB]
  // median: windows of 64 bins from p, cp = #{x < base + p}
  int p = im - 32;
  int h = hist_or_0<NB>(c.H, p + lane), inc = wave_scan_incl(h);
  int cp = c.cm - readlane(inc, 31);
  uint64_t mk;
  while (true) {
    if (cp > rho) {
      if (p <= 0) return false;
      p -= 64;
      h = hist_or_0<NB>(c.H, p + lane);
      inc = wave_scan_incl(h);
      cp -= readlane(inc, 63);
    } else {
      mk = ballot(cp + inc > rho);
      if (mk) break;
      if (p + 64 >= NB) return false;
      p += 64;
      cp += readlane(inc, 63);
      h = hist_or_0<NB>(c.H, p + lane);
      inc = wave_scan_incl(h);
    }
  }
  const int j = ctz(mk);
  const int im2 = p + j, cm2 = cp + readlane(inc, j) - readlane(h, j);
  // the outer pivots follow the median at the old MAD
  const int delta = im2 - im;
  int cL = c.cL, cU = c.cU;
  {
    const int len = delta < 0 ? -delta : delta;
    const int aL = delta < 0 ? iL + delta : iL, aU = delta < 0 ? iU + delta : iU;
    if (aL < 0 || iL + delta < 0 || iU + delta > NB) return false;
    int sL = 0, sU = 0;
    for (int i = lane; i < len; i += 64) {
      sL += hist_get(c.H, aL + i);
      sU += hist_get(c.H, aU + i);
    }
    sL = wave_sum_u(sL);
    sU = wave_sum_u(sU);
    cL += delta < 0 ? -sL : sL;
    cU += delta < 0 ? -sU : sU;
    iL += delta;
    iU += delta;
  }
  // MAD: #{|x - m| <= d} = cU - cL; one bin at each side per unit of d
  int d = c.d;
  if (cU - cL > rho) {  // at most d: lane l tests d - 1 - l
    while (true) {
      const bool ok = lane < d;
      const int hU = ok ? hist_get(c.H, iU - 1 - lane) : 0, hL = ok ? hist_get(c.H, iL + lane) : 0;
      const int incU = wave_scan_incl(hU), incL = wave_scan_incl(hL);
      const int k = popc(ballot(ok && cU - cL - incU - incL > rho));  // the first k lanes
      if (k == 0) break;
      cU -= readlane(incU, k - 1);
      cL += readlane(incL, k - 1);
      d -= k;
      iU -= k;
      iL += k;
      if (k < 64) break;
    }
  } else {  // more than d: lane l tests d + 1 + l
    while (true) {
      const bool ok = iU + lane < NB && iL - 1 - lane >= 0;
      const int hU = ok ? hist_get(c.H, iU + lane) : 0, hL = ok ? hist_get(c.H, iL - 1 - lane) : 0;
      const int incU = wave_scan_incl(hU), incL = wave_scan_incl(hL);
      const uint64_t mm = ballot(ok && cU - cL + incU + incL > rho);
      const int k = mm ? ctz(mm) : 63;
      if (!mm && ballot(!ok)) return false;
      cU += readlane(incU, k);
      cL -= readlane(incL, k);
      d += k + 1;
      iU += k + 1;
      iL -= k + 1;
      if (mm) break;
    }
  }
  c.m = c.base + im2;
  c.cm = cm2;
  c.d = d;
  c.cL = cL;
  c.cU = cU;
  return true;
}

// Narrow local query (the common case): 16 bins around each of the three
// pivots, one DPP row (16 lanes) per pivot, one row-local prefix sum for all
// three. Row 0 finds the new median within [m - 8, m + 7]; row 3 lanes test
// MAD candidates d + t around it from rows 1 (lower pivot) and 2 (upper
// pivot). Returns false when the answer may lie outside these windows.
template <int NB, bool VIRT>
__device__ __forceinline__ bool narrow_query(Chain<NB, VIRT>& c) {
  const int rho = (c.n - 1) >> 1;
  const int im = c.m - c.base, iL = c.m - c.d - c.base, iU = c.m + c.d + 1 - c.base;
  if (iL - 8 < 0 || iU + 8 > NB) return false;  // im lies between them
  const int lane = c.lane, r = lane >> 4, k = lane & 15;
  // per-row selects written as a chain of two-way selects (a nested
  // conditional on scalar operands compiles to branches)
  int ib = iU;
  ib = r == 1 ? iL : ib;
  ib = r == 0 ? im : ib;
  const int h = hist_get(c.H, ib - 8 + k);
  const int inc = row_scan_incl(h);
  const int i0 = readlane(inc, 7), i1 = readlane(inc, 23), i2 = readlane(inc, 39);
  int cb = c.cU - i2;
  cb = r == 1 ? c.cL - i1 : cb;
  cb = r == 0 ? c.cm - i0 : cb;
  const int lt = cb + inc - h;  // #{x < pivot - 8 + k} in rows 0..2
  const uint64_t mk = ballot(lt + h > rho) & 0xFFFFull;
  if (!mk) return false;       // median above the window
  const int j = ctz(mk);
  const int ltj = readlane(lt, j);
  if (ltj > rho) return false;  // median below the window
  const int delta = j - 8;
  // row 3: lane tests d' = d + t, t = k - 8, around m' = m + delta:
  // #{|x - m'| <= d'} = #{x < pU + delta + t} - #{x < pL + delta - t}
  const int t = k - 8;
  const int kl = 8 + delta - t, ku = 8 + delta + t;
  const bool ok = r == 3 && kl >= 0 && kl < 16 && ku >= 0 && ku < 16 && c.d + t >= 0;
  const int va = __shfl(lt, 16 + (kl & 15), 64), vb = __shfl(lt, 32 + (ku & 15), 64);
  const uint64_t okm = ballot(ok), fm = ballot(ok && vb - va > rho);
  if (!fm) return false;        // MAD above the tested range
  const int jj = ctz(fm);
  const int dp = c.d + readlane(t, jj);
  if (jj == ctz(okm) && dp > 0) return false;  // MAD may be smaller still
  c.m = c.m + delta;
  c.cm = ltj;
  c.d = dp;
  c.cL = readlane(va, jj);
  c.cU = readlane(vb, jj);
  return true;
}

// Lower median of the wave's 4 x 64 keys, the first ns of them in use (the
// others ~0): a bitwise binary search counted with ballots.
__device__ __forceinline__ uint32_t key_median(const uint32_t (&k)[4], int ns) {
  const int rank = (ns - 1) >> 1;
  uint32_t p = 0;  // largest key with #{k < p} <= rank
  for (int b = 31; b >= 0; --b) {
    const uint32_t cand = p | (1u << b);
    int cnt = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) cnt += popc(ballot(k[q] < cand));
    if (cnt <= rank) p = cand;
  }
  return p;
}

// Median and MAD of up to 256 samples spread evenly over [lo, hi) (four per lane).
template <bool VIRT>
__device__ __forceinline__ void sample_stats(const RowRef<VIRT>& row, int lo, int hi, int lane, int& m, int& d) {
  const int n = hi - lo;
  const int ns = n < 256 ? n : 256;
  int x[4];
  uint32_t k[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = min(lane + 64 * q, ns - 1);
    x[q] = row.iat(lo + (int)(((int64_t)i * n) / ns));
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) k[q] = lane + 64 * q < ns ? ((uint32_t)x[q] ^ 0x80000000u) : 0xFFFFFFFFu;
  m = (int)(key_median(k, ns) ^ 0x80000000u);
#pragma unroll
  for (int q = 0; q < 4; ++q) k[q] = lane + 64 * q < ns ? absdiff(x[q], m) : 0xFFFFFFFFu;
  d = (int)key_median(k, ns);
}

// The answer of window [lo, hi) where the narrow query did not give it. What
// is tried, in order (one site for each, so that the code stays small):
//   the walk, from a chain in use (kWalk);
//   a new histogram and new pivots (kFresh, also a chain's first block; when
//   the quantiles moved out of the histogram), then the walk. The histogram
//   is centred on the median of samples spread over [lo, span_hi): a
//   contiguous run of samples can sit far from the window's median when the
//   data drift, and for a window clipped at the row start (span_hi > hi) the
//   samples that the growing windows will take in count too, so that it need
//   not be recentred as they grow. The pivots start from the sample median
//   and MAD of the window itself;
//   the exact select (kExact, also every block while the data are too spread
//   for the histogram), then a histogram about its result where one fits.
// A walk that ends near the histogram's edge recentres it (kCentre), to keep
// the local queries' windows inside.
enum { kWalk = 0, kFresh = 1, kExact = 2, kCentre = 3 };

template <int NB, bool VIRT>
__device__ __forceinline__ void refresh_body(Chain<NB, VIRT>& c, int mode, int lo, int hi, int span_hi) {
  while (true) {
    if (mode != kWalk) {
      int centre = c.m, m0 = c.m, d0 = c.d;
      if (mode == kFresh) {
        sample_stats(c.row, lo, span_hi, c.lane, centre, d0);
        m0 = centre;
        if (span_hi != hi) sample_stats(c.row, lo, hi, c.lane, m0, d0);
      } else if (mode == kExact) {
        const int rho = (c.n - 1) >> 1;
        m0 = (int)(radix_select<0, VIRT>(c.H, c.row, lo, hi, rho, 0, c.lane) ^ 0x80000000u);
        d0 = (int)radix_select<1, VIRT>(c.H, c.row, lo, hi, rho, m0, c.lane);
        centre = m0;
        if ((uint32_t)d0 >= (uint32_t)(NB / 2 - 128)) {
          c.m = m0;
          c.d = d0;
          c.raw = true;
          return;
        }
      }
      recount(c, lo, hi, centre, m0, d0);
      if (mode != kFresh) return;
    }
    if (!walk_query(c)) {
      mode = mode == kWalk ? kFresh : kExact;
      continue;
    }
    if (mode == kFresh || c.d >= NB / 2 - 128 || (c.m - c.d - 96 >= c.base && c.m + c.d + 97 <= c.base + NB)) return;
    mode = kCentre;
  }
}

// refresh_body as one real call for all its sites, the chain's state passed
// and returned by value in registers: inlined at five sites it spilled the
// block loop's scalar registers, and by reference the state lives in memory.
// (Pointers go with their address space: through generic ones the call would
// use flat accesses.)
typedef __attribute__((address_space(3))) uint32_t lds_u32;

struct ChainState {
  int base, m, cm, d, cL, cU, raw;
};

template <int NB, bool VIRT>
__device__ __noinline__ ChainState refresh_call(lds_u32* H, gbl_f32* g, gbl_f32* h, int Hx, int n, int base,
                                                int m, int cm, int d, int cL, int cU, int mode, int lo, int hi,
                                                int span_hi) {
  Chain<NB, VIRT> c;
  c.H = (uint32_t*)H;
  c.row.g = uniform_ptr(g);
  c.row.h = VIRT ? uniform_ptr(h) : g;
  c.row.Hx = VIRT ? readfirst(Hx) : 0;
  c.lane = lane_id();
  c.n = readfirst(n);
  c.base = readfirst(base);
  c.m = readfirst(m);
  c.cm = readfirst(cm);
  c.d = readfirst(d);
  c.cL = readfirst(cL);
  c.cU = readfirst(cU);
  c.raw = false;
  refresh_body(c, readfirst(mode), readfirst(lo), readfirst(hi), readfirst(span_hi));
  return {c.base, c.m, c.cm, c.d, c.cL, c.cU, c.raw ? 1 : 0};
}

template <int NB, bool VIRT>
__device__ __forceinline__ void refresh(Chain<NB, VIRT>& c, int mode, int lo, int hi, int span_hi) {
  const ChainState s = refresh_call<NB, VIRT>((lds_u32*)c.H, c.row.g, c.row.h, c.row.Hx, c.n, c.base, c.m, c.cm, c.d, c.cL, c.cU,
                                              mode, lo, hi, span_hi);
  c.base = readfirst(s.base);
  c.m = readfirst(s.m);
  c.cm = readfirst(s.cm);
  c.d = readfirst(s.d);
  c.cL = readfirst(s.cL);
  c.cU = readfirst(s.cU);
  c.raw = readfirst(s.raw) != 0;
}

// Moves the window to the next block: av enters and bv leaves in the lanes of
// a_ok and b_ok (FULL: in every lane, the window's size unchanged).
template <bool FULL, int NB, bool VIRT>
__device__ __forceinline__ void chain_step(Chain<NB, VIRT>& c, int lo, int hi, bool a_ok, int av, bool b_ok, int bv) {
  // lane masks of the entering (a) and leaving (b) samples; the counts below
  // AND raw comparison ballots with them (a comparison's ballot is its own
  // lane mask, a combined condition would be materialised and compared again)
  const uint64_t aM = FULL ? ~0ull : ballot(a_ok), bM = FULL ? ~0ull : ballot(b_ok);
  if (!FULL) c.n += popc(aM) - popc(bM);
  int mode = kExact;
  if (!c.raw) {
    const uint32_t ua = (uint32_t)av - (uint32_t)c.base, ub = (uint32_t)bv - (uint32_t)c.base;
    if ((FULL || a_ok) && ua < (uint32_t)NB) hist_add(c.H, ua, 1u);
    if ((FULL || b_ok) && ub < (uint32_t)NB) hist_add(c.H, ub, 0xFFFFFFFFu);
    const int pL = c.m - c.d, pU = c.m + c.d + 1;
    c.cm += popc(ballot(av < c.m) & aM) - popc(ballot(bv < c.m) & bM);
    c.cL += popc(ballot(av < pL) & aM) - popc(ballot(bv < pL) & bM);
    c.cU += popc(ballot(av < pU) & aM) - popc(ballot(bv < pU) & bM);
    wave_lds_fence();
    if (narrow_query(c)) return;
    mode = kWalk;
  }
  refresh(c, mode, lo, hi, hi);
}

// WPG chains (waves) per workgroup; LDS = WPG * NB * 2 bytes. Blocks
// [kb_first, nblocks) of every row are computed; windows never reach below
// the device value *tmin (the first sample of a stream). LEAD: the window
// reaches a.lead samples past its block (false: trailing, offset compiled out).
template <int NB, bool VIRT, bool LEAD, class Args>
__device__ __forceinline__ void stats_chain(const Args& a, const int chain, uint32_t* H, const int lane) {
  const int row = chain / a.nseg;
  const int seg = chain - row * a.nseg;
  // segment 0 has head_blocks blocks, the others seg_blocks each
  const int kb0 = a.kb_first + (seg == 0 ? 0 : a.head_blocks + (seg - 1) * a.seg_blocks);
  const int kb1 = min(a.nblocks, seg == 0 ? a.kb_first + a.head_blocks : kb0 + a.seg_blocks);
  const int N = a.N, L = a.L, lead = LEAD ? a.lead : 0;
  const int t0 = a.tmin ? *a.tmin : 0;
  Chain<NB, VIRT> c;
  c.H = H;
  c.row.g = (gbl_f32*)a.x + (int64_t)row * a.ld;
  c.row.h = VIRT ? (gbl_f32*)a.hist + (int64_t)row * a.ldh : c.row.g;
  c.row.Hx = VIRT ? a.Hx : 0;
  c.L = L;
  c.lane = lane;
  gbl_i32* med = (gbl_i32*)a.med + (int64_t)row * a.nblocks;
  gbl_i32* mad = (gbl_i32*)a.mad + (int64_t)row * a.nblocks;

  // Block k's window is [max(t0, E_k - L), min(N, E_k)) with E_k = min(64k + 64, N) + lead:
  // from block k-1 to k the samples [min(N, E_{k-1}), min(N, E_k)) enter it and
  // [max(t0, E_{k-1} - L), max(t0, E_k - L)) leave it, at most 64 each.
  // Interior blocks [fi, fe), where exactly 64 enter and 64 leave
  // (64 kk + lead >= t0 + L and 64 kk + 64 + lead <= N), are walked four at a
  // time without clamps or lane masks; the others (a row's first windows, and
  // its last) one by one.
  const int fi = max(kb0 + 1, (t0 + L - lead + kStride - 1) / kStride);
  const int fe = min(kb1, (N - lead) / kStride);
  const int fend = fe - fi >= 4 ? fi + (fe - fi) / 4 * 4 : fi;
  int kk = kb0;
  while (true) {
    const int stop = fend > fi && kk < fend ? fi : kb1;
    // a lane's entering and leaving samples of block kk (a clamped in-row position where unused)
    float na, nb;
    auto fetch = [&](int k) {
      const int Ep = min(k * kStride, N) + lead;
      na = c.row.at(min(min(N, Ep) + lane, N - 1));
      nb = c.row.at(min(max(t0, Ep - L) + lane, N - 1));
    };
    fetch(kk);
    for (; kk < stop; ++kk) {
      const int Ep = min(kk * kStride, N) + lead, E = min(kk * kStride + kStride, N) + lead;
      const int ep = min(N, Ep), e = min(N, E), lp = max(t0, Ep - L), lo = max(t0, E - L);
      const float va = na, vb = nb;
      fetch(kk + 1);
      if (kk == kb0) {
        c.n = e - lo;
        c.raw = false;
        refresh(c, kFresh, lo, e, min(N, max(e, lo + L)));
      } else {
        chain_step<false>(c, lo, e, lane < e - ep, (int)va, lane < lo - lp, (int)vb);
      }
      // every lane stores the same (wave-uniform) values: no branch around the stores
      med[kk] = c.m;
      mad[kk] = c.d;
    }
    if (kk >= kb1) break;
    // Samples are prefetched four blocks ahead, by every lane: loads under a
    // branch would leave the compiler unsure how many are in flight, and it
    // would then wait for all of them, the prefetch included, before each block.
    float pa[4], pb[4];
    auto fetch_full = [&](int k, float& va, float& vb) {
      va = c.row.at(k * kStride + lead + lane);
      vb = c.row.at(k * kStride + lead - L + lane);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) fetch_full(kk + j, pa[j], pb[j]);
    for (; kk < fend; kk += 4) {
      const int kn = kk + 4 < fend ? kk + 4 : kk;  // the last group fetches itself again
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float va = pa[j], vb = pb[j];
        fetch_full(kn + j, pa[j], pb[j]);
        const int e = (kk + j) * kStride + kStride + lead;
        chain_step<true>(c, e - L, e, true, (int)va, true, (int)vb);
        med[kk + j] = c.m;
        mad[kk + j] = c.d;
      }
    }
    if (kk >= kb1) break;
  }
}

}  // namespace

}  // namespace sps
