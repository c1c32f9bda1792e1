// sps_cluster_cells.h - the (time, DM) cells that candidates are bucketed by
// (see sps_cluster.hip), for the device and, without HIP, for the host.
#pragma once

#include <climits>
#include <cstdint>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define SPS_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SPS_HOST_DEVICE inline
#endif

namespace sps {

constexpr int kClusterCells = 1 << 22;  // most cells

// geo: [0, 1] sample range, [2] time cell width, [3] DM cells per time row,
// [4, 5] DM range, [6] DM cell width, [7] time rows. Fills [2, 3, 6, 7] from
// the ranges, so that linked candidates (samples at most time_tol and trials
// at most dm_tol apart) are in the same or neighbouring cells, every candidate
// is in a cell below rows x DM cells, and there are at most kClusterCells of
// them. Linked samples may be a whole cell width apart (they are then exactly
// one row apart), so the width that int32 can hold serves time_tol = INT_MAX
// too; the rows are counted with that width.
SPS_HOST_DEVICE void cluster_cells(int32_t time_tol, int32_t dm_tol, int32_t* geo) {
  const int64_t tlo = geo[0], thi = geo[1], dlo = geo[4], dhi = geo[5];
  const int64_t trange = thi >= tlo ? thi - tlo + 1 : 1, drange = dhi >= dlo ? dhi - dlo + 1 : 1;
  // at most a quarter of the cells across DM, so that at least four time rows
  // fit (four rows of any width that is needed cover the int32 range)
  int64_t cd = (int64_t)dm_tol + 1;
  const int64_t dneed = (drange + kClusterCells / 4 - 1) / (kClusterCells / 4);
  if (cd < dneed) cd = dneed;
  const int64_t nd = (drange + cd - 1) / cd;
  const int64_t nt_max = kClusterCells / nd;
  int64_t cw = (int64_t)time_tol + 1;
  const int64_t tneed = (trange + nt_max - 1) / nt_max;
  if (cw < tneed) cw = tneed;
  if (cw > INT_MAX) cw = INT_MAX;
  geo[2] = (int32_t)cw;
  geo[3] = (int32_t)nd;
  geo[6] = (int32_t)(uint32_t)cd;  // (2^31 for dm_tol = INT_MAX: read as unsigned)
  geo[7] = (int32_t)((trange + cw - 1) / cw);
}

// Cell of a candidate and its (time, DM) cell coordinates. The differences
// from the range's start fit 32 unsigned bits.
SPS_HOST_DEVICE uint32_t cluster_cell(const int32_t* geo, int32_t sample, uint32_t dm, int& ct, int& cd) {
  ct = (int)(((uint32_t)sample - (uint32_t)geo[0]) / (uint32_t)geo[2]);
  cd = (int)((dm - (uint32_t)geo[4]) / (uint32_t)geo[6]);
  return (uint32_t)ct * (uint32_t)geo[3] + (uint32_t)cd;
}

}  // namespace sps
