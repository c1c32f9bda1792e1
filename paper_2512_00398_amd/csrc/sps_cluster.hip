// sps_cluster.hip - candidate merging and clustering (Heimdall++, Section
// II-B "Candidate Merging and Clustering", Section III's analysis of that
// stage and the last step of Algorithm 1).
//
// Candidates a and b are linked when their samples differ by at most
// time_tol, their DM indices by at most dm_tol and their log2 widths by at
// most width_tol; clusters are the connected components of the links, each
// reported by its member of largest S/N (equal S/N: smallest dm, width,
// sample) with its member count and extents.
//
// The paper's point about this stage is that all-pairs comparison is
// quadratic and scattered. Here the candidates are first bucketed by (time,
// DM) cell with a counting sort (cells at least time_tol + 1 samples and
// dm_tol + 1 trials wide, so linked candidates are in the same or adjacent
// cells) and gathered into bucket order; each candidate is then compared only
// with the candidates of its own cell and of the four neighbouring cells that
// follow it, read contiguously. Components are found by union-find on the
// bucketed positions (a root is always the smallest position of its tree;
// hooking a root under a smaller one is a compare-and-swap).
//
// Bound by the dependent loads of the union-find, so almost all of it runs in
// LDS: a workgroup takes 1024 consecutive positions (some time rows of
// cells), links the pairs among them, and sums up each local component
// (members, extents, best member). Only the pairs that cross a tile's end,
// from its last time rows, are then linked in global memory, and only the
// local components, not the candidates, are merged into their final roots.
// 2.1 M candidates of a flooded 256 x 2^20 search: 0.125 ms for the tiles,
// 0.043 across them and 0.023 for the merge; 1.27 ms of linking and 0.20 of
// collecting when all of it was done in global memory.
#include <algorithm>
#include <climits>

#include "sps_cluster_cells.h"
#include "sps_internal.h"
#include "sps_wave.h"

namespace sps {

namespace {

__device__ __forceinline__ int ld_relaxed(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int lds_ld(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Union-find over an array that all threads of SCOPE (the chip, or a workgroup
// with the array in LDS) work on at once, with parent[v] <= v always.
//
// Root of x's tree by path splitting (Tarjan and van Leeuwen, "Worst-case analysis
// of set union algorithms", 1984; on GPUs also known as intermediate pointer
// jumping): every node on the way is put under its grandparent. A store that
// races with another leaves one of the node's ancestors either way. (Path
// halving, which goes on from the grandparent, took 7 % longer on dense sets.)
template <int SCOPE>
__device__ __forceinline__ int root_of(int* parent, int x) {
  int up = __hip_atomic_load(&parent[x], __ATOMIC_RELAXED, SCOPE);
  while (up != x) {
    const int top = __hip_atomic_load(&parent[up], __ATOMIC_RELAXED, SCOPE);
    if (top != up) __hip_atomic_store(&parent[x], top, __ATOMIC_RELAXED, SCOPE);
    x = up;
    up = top;
  }
  return x;
}

// Joins the trees of a and b: the later root goes under the earlier one, by a
// compare-and-swap that fails if it is no root any more.
template <int SCOPE>
__device__ __forceinline__ void join(int* parent, int a, int b) {
  a = root_of<SCOPE>(parent, a);
  b = root_of<SCOPE>(parent, b);
  while (a != b) {
    const int later = max(a, b);
    const int earlier = min(a, b);
    int seen = later;
    if (__hip_atomic_compare_exchange_strong(&parent[later], &seen, earlier, __ATOMIC_RELAXED, __ATOMIC_RELAXED, SCOPE))
      return;
    a = root_of<SCOPE>(parent, seen);  // where it was put meanwhile
    b = root_of<SCOPE>(parent, earlier);
  }
}

constexpr int kChip = __HIP_MEMORY_SCOPE_AGENT, kGroup = __HIP_MEMORY_SCOPE_WORKGROUP;

__device__ __forceinline__ int log2w(uint32_t w) { return 31 - __clz((int)w); }

// Number of lanes below this one in mask m.
__device__ __forceinline__ int lanes_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__global__ __launch_bounds__(256) void k_cluster_range(const sps_cand* c, uint32_t n, ClusterScratch s) {
  __shared__ int red[4][4];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  int smin = INT_MAX, smax = INT_MIN, dmin = INT_MAX, dmax = INT_MIN;
  for (uint64_t i0 = blockIdx.x * 1024ull; i0 < n; i0 += gridDim.x * 1024ull) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t i = i0 + k * 256 + threadIdx.x;
      const sps_cand a = c[i < n ? i : n - 1];  // (the last record again, past the end)
      smin = min(smin, a.sample);
      smax = max(smax, a.sample);
      dmin = min(dmin, (int)a.dm_idx);
      dmax = max(dmax, (int)a.dm_idx);
    }
  }
  // sample and DM ranges: one atomic per workgroup and value
  smin = wave_min_u(smin);
  smax = wave_max_u(smax);
  dmin = wave_min_u(dmin);
  dmax = wave_max_u(dmax);
  if (lane == 0) {
    red[0][wave] = smin;
    red[1][wave] = smax;
    red[2][wave] = dmin;
    red[3][wave] = dmax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    atomicMin(&s.geo[0], min(min(red[0][0], red[0][1]), min(red[0][2], red[0][3])));
    atomicMax(&s.geo[1], max(max(red[1][0], red[1][1]), max(red[1][2], red[1][3])));
    atomicMin(&s.geo[4], min(min(red[2][0], red[2][1]), min(red[2][2], red[2][3])));
    atomicMax(&s.geo[5], max(max(red[3][0], red[3][1]), max(red[3][2], red[3][3])));
  }
}

__global__ void k_cluster_begin(ClusterScratch s, uint32_t* nout) {
  if (threadIdx.x != 0) return;
  s.geo[0] = INT_MAX;
  s.geo[1] = INT_MIN;
  s.geo[4] = INT_MAX;
  s.geo[5] = INT_MIN;
  *nout = 0u;
}

// Entries of `count` in use: the cells and two more (a cell's range ends at
// the next one's start). A short or narrow set has few, which the host does not
// know, so the kernels over them stride over those in use with a grid that the
// chip holds at once (100 candidates in all: 74 us with a workgroup for every 256
// or 1024 possible entries, 67 with this and no launches across a single tile).
constexpr int kCellGrid = 1024;
__device__ __forceinline__ int used_cells(const ClusterScratch& s) { return s.geo[3] * s.geo[7] + 2; }

__global__ __launch_bounds__(256) void k_cluster_clear(ClusterScratch s) {
  const int used = used_cells(s);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < used; i += kCellGrid * 256) s.count[i] = 0u;
}

__global__ void k_cluster_geometry(int time_tol, int dm_tol, ClusterScratch s) {
  if (blockIdx.x == 0 && threadIdx.x == 0) cluster_cells(time_tol, dm_tol, s.geo);
}

__device__ __forceinline__ uint32_t cell_of(const ClusterScratch& s, int sample, uint32_t dm, int& ct, int& cd) {
  return cluster_cell(s.geo, sample, dm, ct, cd);
}

__device__ __forceinline__ uint32_t cell_of(const ClusterScratch& s, const sps_cand& a) {
  int ct, cd;
  return cell_of(s, a.sample, a.dm_idx, ct, cd);
}

// Cell sizes, and each candidate's rank in its cell (in the order of the
// atomics; kept in `parent` until the positions are known). Bound by the rate
// of atomics on global memory (about 20 G/s): candidates that were written
// together share cells, so a workgroup counts its 2048 in an LDS hash table
// first and adds each cell's number once (2.1 M candidates 120 -> 78 us; 4096
// in a table of 64 KB the same).
constexpr int kCountThreads = 512;
constexpr int kCountEach = 4;          // candidates per thread
constexpr int kCountShift = 20;
constexpr int kCountSlots = 1 << (32 - kCountShift);
static_assert(kCountSlots >= 2 * kCountThreads * kCountEach, "an insertion always finds a free slot");

__global__ __launch_bounds__(kCountThreads) void k_cluster_count(const sps_cand* c, uint32_t n, ClusterScratch s) {
  __shared__ int key[kCountSlots];
  __shared__ uint32_t cnt[kCountSlots];
  for (int i = threadIdx.x; i < kCountSlots; i += kCountThreads) {
    key[i] = -1;
    cnt[i] = 0u;
  }
  __syncthreads();
  const uint32_t base = blockIdx.x * (kCountThreads * kCountEach) + threadIdx.x;
  int slot[kCountEach];
  uint32_t rank[kCountEach];
#pragma unroll
  for (int k = 0; k < kCountEach; ++k) {
    const uint32_t i = base + k * kCountThreads;
    slot[k] = -1;
    if (i < n) {
      const int cell = (int)cell_of(s, c[i]);
      int h = (int)(((uint32_t)cell * 2654435761u) >> kCountShift);
      while (true) {  // at most half of the slots are ever taken
        const int was = atomicCAS(&key[h], -1, cell);
        if (was == -1 || was == cell) break;
        h = (h + 1) & (kCountSlots - 1);
      }
      slot[k] = h;
      rank[k] = atomicAdd(&cnt[h], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kCountSlots; i += kCountThreads)
    if (key[i] != -1) cnt[i] = atomicAdd(&s.count[key[i]], cnt[i]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kCountEach; ++k)
    if (slot[k] >= 0) s.parent[base + k * kCountThreads] = (int)(cnt[slot[k]] + rank[k]);
}

// Exclusive prefix sums of the used part of count[0 .. kClusterCells + 2), in place, in three
// passes: 1024 entries per workgroup, then the workgroup totals, then the
// offsets added back.
constexpr int kScanTile = 1024;

__global__ __launch_bounds__(256) void k_scan_tiles(ClusterScratch s) {
  __shared__ uint32_t wsum[4];
  const int t = threadIdx.x, lane = lane_id(), wave = t >> 6;
  const int used = used_cells(s);
  for (int tile = blockIdx.x; tile * kScanTile < used; tile += kCellGrid) {  // the same for the whole workgroup
    const int base = tile * kScanTile + 4 * t;
    uint32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = base + q < used ? s.count[base + q] : 0u;
    const uint32_t own = v[0] + v[1] + v[2] + v[3];
    const uint32_t incl = (uint32_t)wave_scan_incl((int)own);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t off = 0;
    for (int w = 0; w < wave; ++w) off += wsum[w];
    uint32_t run = off + incl - own;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (base + q < used) s.count[base + q] = run;
      run += v[q];
    }
    if (t == 255) s.bsum[tile] = off + incl;
    __syncthreads();  // wsum is free again
  }
}

__global__ __launch_bounds__(1024) void k_scan_totals(ClusterScratch s) {
  __shared__ uint32_t wsum[16];
  __shared__ uint32_t carry;
  const int t = threadIdx.x, lane = lane_id(), wave = t >> 6;
  const int tiles = (used_cells(s) + kScanTile - 1) / kScanTile;
  if (t == 0) carry = 0u;
  __syncthreads();
  for (int b0 = 0; b0 < tiles; b0 += 1024) {
    const uint32_t own = b0 + t < tiles ? s.bsum[b0 + t] : 0u;
    const uint32_t incl = (uint32_t)wave_scan_incl((int)own);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t off = carry;
    for (int w = 0; w < wave; ++w) off += wsum[w];
    if (b0 + t < tiles) s.bsum[b0 + t] = off + incl - own;
    __syncthreads();
    if (t == 1023) carry = off + incl;
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_scan_add(ClusterScratch s) {
  const int used = used_cells(s);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < used; i += kCellGrid * 256) s.count[i] += s.bsum[i / kScanTile];
}

// Records in bucket order.
__global__ void k_cluster_scatter(const sps_cand* c, uint32_t n, ClusterScratch s) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const sps_cand a = c[i];
    s.sorted[s.count[cell_of(s, a)] + (uint32_t)s.parent[i]] = a;
  }
}

__device__ __forceinline__ bool linked(const sps_cand& a, int la, const sps_cand& b, int tt, int dt, int wt) {
  const int64_t ds = (int64_t)b.sample - a.sample;
  const int64_t dd = (int64_t)b.dm_idx - a.dm_idx;
  const int dw = log2w(b.width) - la;
  return (ds <= tt && ds >= -tt) && (dd <= dt && dd >= -dt) && (dw <= wt && dw >= -wt);
}

// The later positions that position p is compared with: the rest of its own
// cell and the cell (t, d+1), which follows it, in [p + 1, e0), and the cells
// (t+1, d-1 .. d+1) in [b1, e1). Each pair of neighbouring cells is visited
// from one side only. (Cells are numbered row by row (time), DM cells within
// a row: a run of neighbouring DM cells is one contiguous range of positions.)
__device__ __forceinline__ void link_ranges(const ClusterScratch& s, const sps_cand& a, uint32_t& e0, uint32_t& b1,
                                            uint32_t& e1) {
  int ct, cd;
  const uint32_t cell = cell_of(s, a.sample, a.dm_idx, ct, cd);
  const int nd = s.geo[3], nt = s.geo[7];
  e0 = s.count[cell + (cd + 1 < nd ? 2 : 1)];
  b1 = e1 = 0;
  if (ct + 1 < nt) {
    const uint32_t r = (uint32_t)(ct + 1) * (uint32_t)nd;
    b1 = s.count[r + (uint32_t)(cd > 0 ? cd - 1 : 0)];
    e1 = s.count[r + (uint32_t)(cd + 1 < nd ? cd + 1 : nd - 1) + 1];
  }
}

// (dm, log2 width, sample) in one key that orders as the tie-break does.
__device__ __forceinline__ unsigned long long tie_key(const sps_cand& a) {
  return ((unsigned long long)a.dm_idx << 37) | ((unsigned long long)log2w(a.width) << 32) |
         (unsigned long long)((uint32_t)a.sample ^ 0x80000000u);
}

// S/N as an unsigned number (S/N > 0: its bits order as the values).
__device__ __forceinline__ uint32_t snr_bits(const sps_cand& a) { return __float_as_uint(a.snr); }

constexpr int kTilePos = 1024;     // positions per workgroup
constexpr int kTileThreads = 512;
// positions past a tile's end held in LDS: as many as leave three workgroups
// per CU (51 KB each). Pairs further on are linked in global memory, which
// dense time rows do much of (8.49 M candidates of 1024 trials, whole
// clustering: 1024 held 3.45 ms, 2048 2.57; 2.1 M of 256 trials 0.55 for both;
// 3072 at one workgroup per CU 2.80 and 0.60).
constexpr int kCrossPos = 2048;
// lanes that share one position's comparisons (the longest of a wave's loops is shorter)
constexpr int kTileLanes = 4;

// Links the pairs among the tile's positions and sums up its components: for
// each local root, members, extents and the best member (its S/N bits and
// position, in `tie`); members is 0 for the other positions.
__global__ __launch_bounds__(kTileThreads) void k_cluster_tile(uint32_t n, int tt, int dt, int wt, ClusterScratch s) {
  __shared__ __align__(16) sps_cand rec[kTilePos];
  __shared__ unsigned long long key[kTilePos];
  __shared__ int parent[kTilePos];
  __shared__ uint32_t members[kTilePos], snr[kTilePos], dlo[kTilePos], dhi[kTilePos];
  __shared__ int slo[kTilePos], shi[kTilePos];
  const uint32_t base = blockIdx.x * kTilePos;
  const int len = (int)min((uint32_t)kTilePos, n - base);
  const int tid = threadIdx.x, lane = lane_id();
  for (int i = tid; i < len; i += kTileThreads) {
    rec[i] = s.sorted[base + i];
    parent[i] = i;
    key[i] = ~0ull;
    members[i] = snr[i] = dhi[i] = 0u;
    dlo[i] = UINT_MAX;
    slo[i] = INT_MAX;
    shi[i] = INT_MIN;
  }
  __syncthreads();
  for (int i = tid / kTileLanes; i < len; i += kTileThreads / kTileLanes) {
    const sps_cand a = rec[i];
    const int la = log2w(a.width);
    uint32_t e0, b1, e1;
    link_ranges(s, a, e0, b1, e1);
    const uint32_t end = base + (uint32_t)len;
    auto link = [&](int b, int e) {
      for (int q = b + tid % kTileLanes; q < e; q += kTileLanes)
        if (linked(a, la, rec[q], tt, dt, wt) && lds_ld(&parent[i]) != lds_ld(&parent[q])) join<kGroup>(parent, i, q);
    };
    link(i + 1, (int)(min(e0, end) - base));
    if (b1 < end) link((int)(max(b1, base) - base), (int)(max(min(e1, end), base) - base));
  }
  __syncthreads();
  // A component's members are mostly neighbours, so lanes that share the root
  // of the first pending lane are combined in the wave first (at most two
  // such groups of four or more lanes); the other lanes add their own values.
  int root[kTilePos / kTileThreads];
#pragma unroll
  for (int k = 0; k < kTilePos / kTileThreads; ++k) {
    const int i = tid + k * kTileThreads;
    const bool valid = i < len;
    const int r = valid ? root_of<kGroup>(parent, i) : -1;
    root[k] = r;
    sps_cand a;
    a.sample = 0;
    a.dm_idx = 0u;
    a.width = 1u;
    a.snr = 0.f;
    if (valid) a = rec[i];
    const uint32_t q = snr_bits(a);
    bool done = !valid;
    for (int it = 0; it < 2; ++it) {
      const uint64_t pend = ballot(!done);
      if (!pend) break;
      const int leader = ctz(pend);
      const int rl = readlane(r, leader);
      const bool mine = !done && r == rl;
      const uint64_t grp = ballot(mine);
      if (popc(grp) < 4) break;
      const uint32_t gq = (uint32_t)wave_max_u(mine ? (int)(q ^ 0x80000000u) : INT_MIN) ^ 0x80000000u;
      const int gslo = wave_min_u(mine ? a.sample : INT_MAX), gshi = wave_max_u(mine ? a.sample : INT_MIN);
      const int gdlo = wave_min_u(mine ? (int)a.dm_idx : INT_MAX), gdhi = wave_max_u(mine ? (int)a.dm_idx : -1);
      if (lane == leader) {
        atomicAdd(&members[rl], (uint32_t)popc(grp));
        atomicMax(&snr[rl], gq);
        atomicMin(&slo[rl], gslo);
        atomicMax(&shi[rl], gshi);
        atomicMin(&dlo[rl], (uint32_t)gdlo);
        atomicMax(&dhi[rl], (uint32_t)gdhi);
      }
      done = done || mine;
    }
    if (!done) {
      atomicAdd(&members[r], 1u);
      atomicMax(&snr[r], q);
      atomicMin(&slo[r], a.sample);
      atomicMax(&shi[r], a.sample);
      atomicMin(&dlo[r], a.dm_idx);
      atomicMax(&dhi[r], a.dm_idx);
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kTilePos / kTileThreads; ++k) {
    const int i = tid + k * kTileThreads;
    if (i < len && snr_bits(rec[i]) == snr[root[k]]) atomicMin(&key[root[k]], tie_key(rec[i]));
  }
  __syncthreads();
  // the position of the best member: any of those that hold the key (equal records)
#pragma unroll
  for (int k = 0; k < kTilePos / kTileThreads; ++k) {
    const int i = tid + k * kTileThreads;
    if (i < len && snr_bits(rec[i]) == snr[root[k]] && tie_key(rec[i]) == key[root[k]])
      s.tie[base + root[k]] = ((unsigned long long)snr[root[k]] << 32) | (base + (uint32_t)i);
    if (i < len) {
      s.parent[base + i] = (int)base + root[k];
      s.members[base + i] = members[i];  // 0 unless a root
      if (root[k] != i) {
        s.slo[base + i] = (int)base + root[k];  // (its own extent is the root's business)
      } else {
        s.slo[base + i] = slo[i];
        s.shi[base + i] = shi[i];
        s.dlo[base + i] = dlo[i];
        s.dhi[base + i] = dhi[i];
      }
    }
  }
}

// The pairs across the end of a tile: from its positions in the last time
// rows that reach the next tile's first row. Most of them join the same few
// local components, so the components of the two tiles (by their roots'
// positions) are joined in LDS first and each join is then made once in
// global memory; pairs that reach past the positions held go there directly,
// each position comparing roots only where it meets a component for the first
// time in a row. gridDim.y workgroups share a tile's positions where there are
// few tiles (large tolerances put a small set into a few cells, all of whose
// pairs are compared): 20000 candidates in one cell, all linked, 12.6 -> 1.8 ms
// (6.0 when one thread per position linked them all in global memory).
__global__ __launch_bounds__(kTileThreads) void k_cluster_cross(uint32_t n, int tt, int dt, int wt, ClusterScratch s) {
  constexpr int kHeld = kTilePos + kCrossPos;
  static_assert(kHeld <= 65536, "positions from the tile's base fit 16 bits");
  __shared__ __align__(16) sps_cand rec[kCrossPos];  // from the tile's end
  __shared__ uint16_t root[kHeld];                   // position's local root, from the tile's base
  __shared__ int parent[kHeld];                      // joined roots
  const uint32_t base = blockIdx.x * kTilePos, end = base + kTilePos;
  if (end >= n) return;
  const int tid = threadIdx.x;
  const int nd = s.geo[3], nt = s.geo[7];
  int ct, cd, cl;
  const sps_cand f = s.sorted[end], g = s.sorted[end - 1];
  cell_of(s, f.sample, f.dm_idx, ct, cd);
  cell_of(s, g.sample, g.dm_idx, cl, cd);
  const uint32_t row = ct > 0 ? s.count[(uint32_t)(ct - 1) * (uint32_t)nd] : 0u;
  const uint32_t first = max(row, base);  // positions before it reach no further than `end`
  if (first >= end) return;               // whole workgroup; no barrier passed yet
  // the last position that any of them is compared with is in row cl + 1
  const uint32_t reach = cl + 2 <= nt ? s.count[(uint32_t)(cl + 2) * (uint32_t)nd] : n;
  const uint32_t held = min(min(reach, n), end + kCrossPos);
  for (uint32_t p = first + tid; p < held; p += kTileThreads) {
    const int i = (int)(p - base);
    if (p >= end) rec[p - end] = s.sorted[p];
    root[i] = (uint16_t)(s.members[p] ? i : s.slo[p] - (int)base);
  }
  const int len = (int)(held - base);
  for (int i = tid; i < len; i += kTileThreads) parent[i] = i;
  __syncthreads();
  const uint32_t each = kTileThreads / kTileLanes;
  for (uint32_t p = first + blockIdx.y * each + tid / kTileLanes; p < end; p += gridDim.y * each) {
    const sps_cand a = s.sorted[p];
    const int la = log2w(a.width), ra = root[p - base];
    uint32_t e0, b1, e1;
    link_ranges(s, a, e0, b1, e1);
    int joined = -1;  // a node of the tree that p is in since the last join
    auto link = [&](uint32_t b, uint32_t e) {
      for (uint32_t q = b + tid % kTileLanes; q < e; q += kTileLanes) {
        if (q < held) {
          if (linked(a, la, rec[q - end], tt, dt, wt)) {
            const int rq = root[q - base];
            if (lds_ld(&parent[ra]) != lds_ld(&parent[rq])) join<kGroup>(parent, ra, rq);
          }
        } else if (linked(a, la, s.sorted[q], tt, dt, wt)) {
          // q's parent, perhaps an older one: still a node of q's tree
          const int up = __hip_atomic_load(&s.parent[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (up != joined) {
            join<kChip>(s.parent, (int)p, (int)q);
            joined = up;
          }
        }
      }
    };
    link(end, e0);
    link(max(b1, end), e1);
  }
  __syncthreads();
  for (int i = tid; i < len; i += kTileThreads) {
    const int r = lds_ld(&parent[i]);
    if (r != i) join<kChip>(s.parent, (int)base + r, (int)base + i);
  }
}

// Local components into their final roots.
__global__ void k_cluster_merge(uint32_t n, ClusterScratch s) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const uint32_t m = s.members[p];
  if (m == 0u) return;
  const int r = root_of<kChip>(s.parent, (int)p);  // trees no longer change; roots stay roots
  if (r == (int)p) return;
  // p is no root, so nothing is added to its own values
  atomicAdd(&s.members[r], m);
  atomicMin(&s.slo[r], s.slo[p]);
  atomicMax(&s.shi[r], s.shi[p]);
  atomicMin(&s.dlo[r], s.dlo[p]);
  atomicMax(&s.dhi[r], s.dhi[p]);
  const unsigned long long v = s.tie[p];
  const unsigned long long kv = tie_key(s.sorted[(uint32_t)v]);
  unsigned long long old = __hip_atomic_load(&s.tie[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  while ((v >> 32) > (old >> 32) || ((v >> 32) == (old >> 32) && kv < tie_key(s.sorted[(uint32_t)old]))) {
    const unsigned long long seen = atomicCAS(&s.tie[r], old, v);
    if (seen == old) break;
    old = seen;
  }
}

// One record per root; the workgroup claims its output slots for `chunks` x
// 256 positions with one atomic (same-address atomics serialise; 1 to 16
// chunks, for about 512 workgroups).
__global__ __launch_bounds__(256) void k_cluster_emit(uint32_t n, int chunks, ClusterScratch s, sps_cluster_rec* out,
                                                      uint32_t* nout) {
  __shared__ uint32_t wcount[4];
  __shared__ uint32_t base;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  uint32_t mine = 0u;
  for (int k = 0; k < chunks; ++k) {
    const uint32_t p = (blockIdx.x * chunks + k) * 256 + threadIdx.x;
    mine += (uint32_t)popc(ballot(p < n && ld_relaxed(&s.parent[p]) == (int)p));
  }
  if (lane == 0) wcount[wave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) base = atomicAdd(nout, wcount[0] + wcount[1] + wcount[2] + wcount[3]);
  __syncthreads();
  uint32_t at = base;
  for (int v = 0; v < wave; ++v) at += wcount[v];
  for (int k = 0; k < chunks; ++k) {
    const uint32_t p = (blockIdx.x * chunks + k) * 256 + threadIdx.x;
    const bool root = p < n && ld_relaxed(&s.parent[p]) == (int)p;
    const uint64_t m = ballot(root);
    if (root) {
      const sps_cand best = s.sorted[(uint32_t)s.tie[p]];
      sps_cluster_rec r;
      r.dm_idx = best.dm_idx;
      r.width = 1u << (log2w(best.width) & 31);
      r.sample = best.sample;
      r.snr = best.snr;
      r.members = s.members[p];
      r.sample_lo = s.slo[p];
      r.sample_hi = s.shi[p];
      r.dm_lo = s.dlo[p];
      r.dm_hi = s.dhi[p];
      r.reserved = 0u;
      out[at + (uint32_t)lanes_below(m)] = r;
    }
    at += (uint32_t)popc(m);
  }
}

}  // namespace

hipError_t launch_cluster(const sps_cand* c, uint32_t n, int tt, int dt, int wt, const ClusterScratch& s,
                          sps_cluster_rec* out, uint32_t* nout, hipStream_t st) {
  const dim3 b(256);
  const dim3 gc(kCellGrid);
  hipLaunchKernelGGL(k_cluster_begin, dim3(1), dim3(64), 0, st, s, nout);
  if (n > 0) {
    const dim3 gn((n + 255) / 256);
    hipLaunchKernelGGL(k_cluster_range, dim3(std::min(256u, (n + 1023) / 1024)), b, 0, st, c, n, s);
    hipLaunchKernelGGL(k_cluster_geometry, dim3(1), dim3(64), 0, st, tt, dt, s);
    hipLaunchKernelGGL(k_cluster_clear, gc, b, 0, st, s);
    hipLaunchKernelGGL(k_cluster_count, dim3((n + kCountThreads * kCountEach - 1) / (kCountThreads * kCountEach)),
                       dim3(kCountThreads), 0, st, c, n, s);
    hipLaunchKernelGGL(k_scan_tiles, gc, b, 0, st, s);
    hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(1024), 0, st, s);
    hipLaunchKernelGGL(k_scan_add, gc, b, 0, st, s);
    hipLaunchKernelGGL(k_cluster_scatter, gn, b, 0, st, c, n, s);
    const dim3 gt((n + kTilePos - 1) / kTilePos);
    hipLaunchKernelGGL(k_cluster_tile, gt, dim3(kTileThreads), 0, st, n, tt, dt, wt, s);
    if (gt.x > 1) {  // a single tile's components are final
      const dim3 gx(gt.x, std::min(8u, std::max(1u, 512 / gt.x)));
      hipLaunchKernelGGL(k_cluster_cross, gx, dim3(kTileThreads), 0, st, n, tt, dt, wt, s);
      hipLaunchKernelGGL(k_cluster_merge, gn, b, 0, st, n, s);
    }
    const int chunks = (int)std::min(16u, std::max(1u, gn.x / 512));
    hipLaunchKernelGGL(k_cluster_emit, dim3((gn.x + chunks - 1) / chunks), b, 0, st, n, chunks, s, out, nout);
  }
  return hipGetLastError();
}

}  // namespace sps
