// sps_dedisp.hip - incoherent dedispersion on the device (Heimdall++,
// Section II-B, "Incoherent Dedispersion"; the DM of Eq. 1): for every trial
// d, out[d][t] = sum over channels f of fil[f][t + delay[d][f]], from an 8-bit
// channel-major filterbank to the FP32 [ndm][nsamp_out] block the search
// consumes. Exact integer sums.
//
// Design (gfx950, wave64). One add per (trial, channel, sample) is far too
// much for the vector units, but most of these sums are shared: the delays of
// 1 to 4 neighbouring channels, relative to the first of them, take few
// distinct patterns over the 8, 16 or 32 trials of a workgroup (1.6 and 2.7 for
// pairs and threes over 16 trials, on 1024 channels and trials). So a workgroup first builds, for a
// subband of G channels, the 16-bit sums of each pattern once, in LDS, over
// the span that the pattern's trials need, and each trial then adds one
// 16-bit subband sample where it would have added G bytes. The host lays out
// the patterns per (trial group, subband) from the delay table, whatever it
// holds, and picks G by modelled cost.
//
//   build: a wave makes 252 subband samples at a time, four per lane: one
//     aligned 4-byte load per channel, joined with the next lane's to the
//     channel's alignment, two byte permutes that widen it to 16-bit pairs,
//     and adds. The next subband's loads are in flight while
//     this one is summed (two LDS buffers, one barrier per subband). Each
//     block is written twice, as pairs from even and from odd samples
//     (the last lane only lends its first sample to its neighbour's odd
//     pair), because an LDS read or a load that is not aligned to its own size takes
//     64 cycles here, against 2.4 for an aligned LDS word (measured);
//   sum: a wave owns TPW trials of the group and all of the tile's samples,
//     2 NP per lane: per trial one address add, NP words read from the copy
//     of the trial's parity and NP adds of 16-bit pairs, whose upper halves are
//     moved to a second pair every 256 channels.
//
// Bound by the latency of a subband (sums, builds and one barrier; about half
// of it is LDS reads at 2.35 cycles a word) at 16 to 20 waves per CU. 1024
// channels x 1024 trials x 2^18 samples: 17.4 ms with a byte pair added per
// trial, channel and four samples -> 7.8 ms (35 TOP/s of sample additions);
// 256 x 128 x 40001: 0.247 -> 0.133 ms. Tried on the way: 16-byte LDS reads at
// 2-byte offsets (20.5 ms, serialised), record reads by the scalar unit
// (14.4 ms), loads two subbands ahead (8.0 ms), 32-bit sums (8.1 ms).
//
// Workgroups are ordered XCD by XCD over time tiles, all trial groups of a
// time tile on one XCD, sharing its L2.
#include <hip/hip_runtime.h>

#include "sps_internal.h"
#include "sps_wave.h"

namespace sps {
namespace {

typedef __attribute__((address_space(1))) const uint32_t gbl_cu32;
typedef __attribute__((address_space(1))) const int32_t gbl_ci32;
typedef __attribute__((address_space(1))) const uint8_t gbl_u8;
typedef float f32x2 __attribute__((ext_vector_type(2)));

// G channels per subband, W waves, TPW trials per wave, NP words (sample
// pairs) per lane and trial. EDGE: the tile's loads in the last rows may reach
// past the filterbank's end.
template <int G, int W, int TPW, int NP, bool EDGE>
__device__ __forceinline__ void dedisp_tile(const DedispArgs& a, char* lds, const int dg, const int t0) {
  constexpr int kTile = NP / 2 * kDedispBlock;
  // blocks per wave whose words are loaded a subband ahead (the rest follow the sums)
  constexpr int kPF = W == 8 ? 3 : 4;
  static_assert(kPF * W <= kDedispAhead, "records hold the blocks loaded ahead");
  static_assert(TPW % 2 == 0 && kPF * G + TPW / 2 < 64, "the wave's part of a record fits its lanes");
  const int lane = lane_id(), wave = readfirst(threadIdx.x >> 6);
  const int nsub = a.nsub;
  const int copy = dedisp_copy_bytes(a.lds_blocks);
  gbl_u8* const fil = (gbl_u8*)a.fil + t0;
  const int lane4 = 4 * lane;

  // The wave's part of a record, one word per lane: its first kPF blocks'
  // channels, the block count, its trials' offsets. Read a subband before its
  // loads are issued, so that neither its latency nor the scalar unit's waits
  // (which the LDS reads share) stand between the subbands.
  constexpr int kN = kPF * G, kBase = kN + 1;
  const int word = lane < kN    ? kDedispHead + G * (wave + W * (lane / G)) + lane % G
                   : lane == kN ? 0
                                : 1 + wave * (TPW / 2) + min(lane - kBase, TPW / 2 - 1);
  gbl_ci32* rec = (gbl_ci32*)a.rec + (int64_t)dg * nsub * a.rec_words;  // of the next record() call
  int rec_left = nsub;
  auto record = [&]() {
    const int v = rec[word];
    if (--rec_left > 0) rec += a.rec_words;
    return v;
  };

  // Aligned words of a block's channel: `e` is its record entry, `row` the
  // channel's first byte; joined with the next lane's (wave_shl:1) by align().
  const int64_t nfull = (a.total_bytes - t0) >> 2;  // whole words from `fil` on (t0 is a multiple of 4)
  uint32_t tail = 0;                                // the partial word after them
  if (EDGE)
    for (int64_t i = 4 * nfull; i < a.total_bytes - t0; ++i) tail |= (uint32_t)fil[i] << (8 * (int)(i & 3));
  const int64_t reach = (int64_t)t0 + a.max_delay + kTile + 2 * kDedispBlock;  // of any block into its row
  auto at_end = [&](int s) { return EDGE && (int64_t)(min(G * s + G, a.nchan) - 1) * a.ld + reach > a.total_bytes; };
  auto load = [&](int64_t row, int e, bool end) -> uint32_t {
    const int64_t base = row & ~(int64_t)3;
    if (!end) return *(gbl_cu32*)(fil + base + (uint32_t)((e << 2) + lane4));
    // words past the last one are never summed into an output
    const int64_t w = (base >> 2) + (uint32_t)(e & 0x3FFFFFFF) + lane;
    uint32_t v = tail;
    if (w < nfull) v = *(gbl_cu32*)(fil + 4 * w);
    return v;
  };
  auto align = [&](uint32_t w, int e) {
    return __builtin_amdgcn_alignbyte((uint32_t)dpp<0x130>(0, (int)w), w, (uint32_t)e >> 30);
  };
  // block k of subband samples from its channels' words, into both copies;
  // of the subband's channels the first `have` exist
  auto build = [&](const uint32_t (&v)[G], const int (&e)[G], int have, int k, char* at) {
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const uint32_t x = align(v[i], e[i]);
      const uint32_t l = __builtin_amdgcn_perm(0u, x, i == 0 || i < have ? 0x0c010c00u : 0x0c0c0c0cu);
      const uint32_t h = __builtin_amdgcn_perm(0u, x, i == 0 || i < have ? 0x0c030c02u : 0x0c0c0c0cu);
      lo = i == 0 ? l : lo + l;
      hi = i == 0 ? h : hi + h;
    }
    // samples 4l+1 .. 4l+4: the last comes from the next lane (wave_shl:1)
    const uint32_t next = (uint32_t)dpp<0x130>(0, (int)lo);
    const uint32_t olo = __builtin_amdgcn_alignbit(hi, lo, 16), ohi = __builtin_amdgcn_alignbit(next, hi, 16);
    char* const p = at + k * (2 * kDedispBlock) + 2 * lane4;
    if (lane < 63) {
      *reinterpret_cast<uint2*>(p) = make_uint2(lo, hi);
      *reinterpret_cast<uint2*>(p + copy) = make_uint2(olo, ohi);
    }
  };

  int64_t rows = 0;  // first byte of the row of the next subband to load
  // rows past the last channel read the subband's first, which build() drops
  auto fetch = [&](int s, int rv, uint32_t (&pv)[kPF][G], int (&pe)[kPF][G]) {
    const int have = a.nchan - G * s;
    auto all = [&](bool end) {
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const int64_t row = rows + (i == 0 || i < have ? i * a.ld : 0);
#pragma unroll
        for (int p = 0; p < kPF; ++p) {
          pe[p][i] = readlane(rv, G * p + i);
          pv[p][i] = load(row, pe[p][i], end);
        }
      }
    };
    if (at_end(s)) all(true);
    else all(false);
    rows += G * a.ld;
  };
  auto store = [&](int s, int rv, const uint32_t (&pv)[kPF][G], const int (&pe)[kPF][G], char* at) {
    const int n = readlane(rv, kN), have = a.nchan - G * s;
#pragma unroll
    for (int p = 0; p < kPF; ++p)
      if (wave + p * W < n) build(pv[p], pe[p], have, wave + p * W, at);
    if (n > kPF * W) {
      gbl_ci32* r = (gbl_ci32*)a.rec + ((int64_t)dg * nsub + s) * a.rec_words + kDedispHead;
      for (int k = wave + kPF * W; k < n; k += W) {
        uint32_t v[G];
        int e[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
          e[i] = readfirst(r[G * k + i]);
          v[i] = load((G * s + (i == 0 || i < have ? i : 0)) * a.ld, e[i], at_end(s));
        }
        build(v, e, have, k, at);
      }
    }
  };

  // 16-bit pair sums, and pairs of the multiples of 256 moved out of them
  // (at most 65536 channels x 255 / 256 < 2^16): half the registers of 32-bit sums
  uint32_t pk[TPW][NP];
  uint32_t hi[TPW][NP];
#pragma unroll
  for (int j = 0; j < TPW; ++j)
#pragma unroll
    for (int q = 0; q < NP; ++q) pk[j][q] = hi[j][q] = 0u;
  constexpr int kFlush = 256 / G;  // 255 left + 256 channels x 255 < 2^16
  int left = kFlush;
  int rv[3];  // records of subbands s, s + 1, s + 2
#pragma unroll
  for (int k = 0; k < 3; ++k) rv[k] = record();
  uint32_t pv[kPF][G];
  int pe[kPF][G];
  fetch(0, rv[0], pv, pe);
  store(0, rv[0], pv, pe, lds);
  if (nsub > 1) fetch(1, rv[1], pv, pe);
  __syncthreads();
  auto step = [&](int s, uint32_t (&pv)[kPF][G], int (&pe)[kPF][G]) {
    const char* cur = lds + (s & 1) * (2 * copy) + lane4;
    const bool more = s + 1 < nsub;
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
      const int w = readlane(rv[0], kBase + j / 2);
      const int base = j & 1 ? (int)((uint32_t)w >> 16) : w & 0xFFFF;
      const uint32_t* src = reinterpret_cast<const uint32_t*>(cur + base);
#pragma unroll
      for (int q = 0; q < NP; ++q) pk[j][q] += src[64 * q];
    }
    if (--left == 0) {
      left = kFlush;
#pragma unroll
      for (int j = 0; j < TPW; ++j)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          hi[j][q] += (pk[j][q] >> 8) & 0x00FF00FFu;
          pk[j][q] &= 0x00FF00FFu;
        }
    }
    if (more) store(s + 1, rv[1], pv, pe, lds + ((s + 1) & 1) * (2 * copy));
    rv[0] = rv[1];
    rv[1] = rv[2];
    if (s + 2 < nsub) fetch(s + 2, rv[1], pv, pe);
    rv[2] = record();
    __syncthreads();
  };
  for (int s = 0; s < nsub; ++s) step(s, pv, pe);
#pragma unroll
  for (int j = 0; j < TPW; ++j) {
    const int d = dg * (W * TPW) + wave * TPW + j;
    if (d >= a.ndm) break;
    float* o = a.out + (int64_t)d * a.nsamp_out;
    const int end = min(t0 + kTile, a.nsamp_out);
    const bool pairs = (reinterpret_cast<uintptr_t>(o) & 7u) == 0;  // t is even
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int t = t0 + 128 * q + 2 * lane;
      const float x = (float)((pk[j][q] & 0xFFFFu) + ((hi[j][q] & 0xFFFFu) << 8));
      const float y = (float)((pk[j][q] >> 16) + ((hi[j][q] >> 16) << 8));
      if (pairs && t + 1 < end) {
        *reinterpret_cast<f32x2*>(o + t) = f32x2{x, y};
      } else {
        if (t < end) o[t] = x;
        if (t + 1 < end) o[t + 1] = y;
      }
    }
  }
}

template <int G, int W, int TPW, int NP>
__global__ __launch_bounds__(64 * W, 4) void k_dedisp(DedispArgs a) {
  extern __shared__ __align__(16) char lds[];
  constexpr int kTile = NP / 2 * kDedispBlock;
  const int b = blockIdx.x;
  const int tile = (b & 7) * a.per_xcd + (b >> 3);
  if (tile >= a.ntiles) return;  // whole workgroup leaves; no barrier passed yet
  const int dg = tile % a.ngroups, t0 = tile / a.ngroups * kTile;
  // a block's words end at most this far into its row, its last channel's row being the last
  const int64_t reach = (int64_t)(a.nchan - 1) * a.ld + t0 + a.max_delay + kTile + 2 * kDedispBlock;
  if (reach > a.total_bytes) dedisp_tile<G, W, TPW, NP, true>(a, lds, dg, t0);
  else dedisp_tile<G, W, TPW, NP, false>(a, lds, dg, t0);
}

template <int W, int TPW, int NP>
hipError_t launch(const DedispArgs& a, hipStream_t s) {
  const dim3 g(8 * a.per_xcd), b(64 * W);
  const size_t lds = 4 * (size_t)dedisp_copy_bytes(a.lds_blocks);  // at most 64 KB
  switch (a.gch) {
    case 1: hipLaunchKernelGGL((k_dedisp<1, W, TPW, NP>), g, b, lds, s, a); break;
    case 2: hipLaunchKernelGGL((k_dedisp<2, W, TPW, NP>), g, b, lds, s, a); break;
    case 3: hipLaunchKernelGGL((k_dedisp<3, W, TPW, NP>), g, b, lds, s, a); break;
    case 4: hipLaunchKernelGGL((k_dedisp<4, W, TPW, NP>), g, b, lds, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dedisp(const DedispArgs& a, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  if (a.tile == 4 * kDedispBlock && a.trials == 32) return launch<8, 4, 8>(a, s);
  if (a.tile == 4 * kDedispBlock && a.trials == 16) return launch<4, 4, 8>(a, s);
  if (a.tile == 2 * kDedispBlock && a.trials == 16) return launch<4, 4, 4>(a, s);
  if (a.tile == 2 * kDedispBlock && a.trials == 8) return launch<4, 2, 4>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace sps
