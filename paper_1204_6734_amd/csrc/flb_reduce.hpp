// flb_reduce.hpp — reductions of the per-tile correlator partials
// ([ntiles][NSTAT] FP64 sums, one row per tile) into a time-block record or
// the open sums, shared by the D2Q9 (54 statistics) and D3Q19 (209) paths.
// The order of every addition depends only on the tile count, so a lattice
// gives the same sums whatever else runs and however it was launched.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "flb_kernels.hpp"

namespace flb {

// Thread layout (v, j): v = statistic (padded to VP), j = one of J lanes
// over the tiles.
template <int NSTAT>
struct SumShape {
  static constexpr int VP = NSTAT <= 64 ? 64 : 256;
  static constexpr int J = 1024 / VP;
};

// Stage one of closing a block: workgroup b sums tiles [b c, min((b+1) c, n))
// (lane j takes every J-th tile, then the J lane sums are added in order),
// writes the sum into the range's first row and clears the others.
template <int NSTAT>
__device__ __forceinline__ void fold_tiles(double* partials, int ntiles, int chunk) {
  constexpr int VP = SumShape<NSTAT>::VP, J = SumShape<NSTAT>::J;
  __shared__ double red[J][VP];
  const int v = threadIdx.x % VP, j = threadIdx.x / VP;
  const int t0 = blockIdx.x * chunk, t1 = min(t0 + chunk, ntiles);
  double s = 0.0;
  if (v < NSTAT) {
    for (int t = t0 + j; t < t1; t += J) {
      double* q = partials + (size_t)t * NSTAT + v;
      s += *q;
      if (t != t0) *q = 0.0;
    }
  }
  red[j][v] = s;
  __syncthreads();
  if (j == 0 && v < NSTAT) {
    double tot = red[0][v];
#pragma unroll
    for (int k = 1; k < J; ++k) tot += red[k][v];
    partials[(size_t)t0 * NSTAT + v] = tot;
  }
}

// Ranges of stage one: at most kFoldRows workgroups of at least one tile.
// Ranges of one tile each (up to kFoldRows tiles) are their own sums: stage
// two reads the partials themselves and stage one, which would write each sum
// over itself, is not launched.
__host__ __device__ inline void fold_ranges(int ntiles, int* chunk, int* nranges) {
  const int c = ntiles > kFoldRows ? (ntiles + kFoldRows - 1) / kFoldRows : 1;
  *chunk = c;
  *nranges = (ntiles + c - 1) / c;
}

// Stage two: the folded rows (row b at folds + b stride) summed in range
// order, thread v its statistic.  The chain of additions is short (256 FP64
// additions, ~1 us); what bounds it is the latency of the loads, so they are
// issued kGatherBatch at a time before the additions that use them.  One
// load per addition took 41 us for 256 ranges of 54 statistics and 66 us for
// 209 (MI355X, kernel trace); batched, the same additions in the same order
// take 10 and 20 us (64 loads at a time spilled registers: 13 and 68 us).
constexpr int kGatherBatch = 32;
template <int NSTAT>
__device__ __forceinline__ double sum_folds(const double* folds, int nranges, size_t stride) {
  const int v = threadIdx.x;
  double s = 0.0;
  for (int b0 = 0; b0 < nranges; b0 += kGatherBatch) {
    double x[kGatherBatch];
    // past the end the last row is read again and not added
#pragma unroll
    for (int k = 0; k < kGatherBatch; ++k)
      x[k] = folds[(size_t)min(b0 + k, nranges - 1) * stride + v];
#pragma unroll
    for (int k = 0; k < kGatherBatch; ++k)
      if (b0 + k < nranges) s += x[k];
  }
  return s;
}

// Stage two of closing a block: record = the folded rows' sum, by the first
// threads of one workgroup; then all its threads clear the rows (one
// wavefront clearing 256 rows held the kernel at 14 us).
template <int NSTAT>
__device__ __forceinline__ void gather_folds(double* partials, int nranges, int chunk,
                                             double* record) {
  constexpr int VP = SumShape<NSTAT>::VP, J = SumShape<NSTAT>::J;
  const int v = threadIdx.x % VP, j = threadIdx.x / VP;
  const size_t stride = (size_t)chunk * NSTAT;
  if (j == 0 && v < NSTAT) record[v] = sum_folds<NSTAT>(partials, nranges, stride);
  __syncthreads();
  if (v < NSTAT)
    for (int b = j; b < nranges; b += J) partials[b * stride + v] = 0.0;
}

template <int NSTAT>
__global__ __launch_bounds__(1024) void fold_tiles_kernel(double* partials, int ntiles,
                                                          int chunk) {
  fold_tiles<NSTAT>(partials, ntiles, chunk);
}

template <int NSTAT>
__global__ __launch_bounds__(1024) void gather_folds_kernel(double* partials, int nranges, int chunk, double* record) {
  gather_folds<NSTAT>(partials, nranges, chunk, record);
}

// The same two stages for several lattices of one tile count at once, the
// lattice in blockIdx.y: each one's sums are added in the order above.
template <int NSTAT>
__global__ __launch_bounds__(1024) void fold_tiles_many_kernel(double* const* partials, int ntiles,
                                                               int chunk) {
  fold_tiles<NSTAT>(partials[blockIdx.y], ntiles, chunk);
}

template <int NSTAT>
__global__ __launch_bounds__(1024) void gather_folds_many_kernel(double* const* partials, int nranges, int chunk,
                                         double* const* records, size_t record_offset) {
  gather_folds<NSTAT>(partials[blockIdx.y], nranges, chunk, records[blockIdx.y] + record_offset);
}

// And for lattices of any tile counts, listed in the kernel's arguments (a
// server's requests that close at the same step).
constexpr int kCloseList = 32;
struct CloseList {
  double* partials[kCloseList];
  double* record[kCloseList];
  int ntiles[kCloseList];
};

template <int NSTAT>
__global__ __launch_bounds__(1024) void fold_tiles_list_kernel(const CloseList L) {
  const int ntiles = L.ntiles[blockIdx.y];
  int chunk = 1, nranges = 1;
  fold_ranges(ntiles, &chunk, &nranges);
  if (chunk == 1 || (int)blockIdx.x >= nranges) return;
  fold_tiles<NSTAT>(L.partials[blockIdx.y], ntiles, chunk);
}

template <int NSTAT>
__global__ __launch_bounds__(1024) void gather_folds_list_kernel(const CloseList L) {
  int chunk = 1, nranges = 1;
  fold_ranges(L.ntiles[blockIdx.y], &chunk, &nranges);
  gather_folds<NSTAT>(L.partials[blockIdx.y], nranges, chunk, L.record[blockIdx.y]);
}

// Open sums (partials left as they are): workgroup b sums tiles
// [b chunk, min((b+1) chunk, n)) into row b of out, lanes as above.
template <int NSTAT>
__global__ __launch_bounds__(1024) void open_folds_kernel(const double* partials, int ntiles,
                                                          int chunk, double* out) {
  constexpr int VP = SumShape<NSTAT>::VP, J = SumShape<NSTAT>::J;
  __shared__ double red[J][VP];
  const int v = threadIdx.x % VP, j = threadIdx.x / VP;
  const int t0 = blockIdx.x * chunk, t1 = min(t0 + chunk, ntiles);
  double s = 0.0;
  if (v < NSTAT)
    for (int t = t0 + j; t < t1; t += J) s += partials[(size_t)t * NSTAT + v];
  red[j][v] = s;
  __syncthreads();
  if (j == 0 && v < NSTAT) {
    double tot = red[0][v];
#pragma unroll
    for (int k = 1; k < J; ++k) tot += red[k][v];
    out[(size_t)blockIdx.x * NSTAT + v] = tot;
  }
}

template <int NSTAT>
__global__ void open_gather_kernel(const double* folds, int nranges, double* out) {
  if (threadIdx.x < NSTAT) out[threadIdx.x] = sum_folds<NSTAT>(folds, nranges, NSTAT);
}

// record[NSTAT] = sum of the partials over all tiles; partials cleared.
template <int NSTAT>
hipError_t close_block_sums(double* partials, int ntiles, double* record, hipStream_t st) {
  if (ntiles <= 0) return hipErrorInvalidValue;
  int chunk = 1, nranges = 1;
  fold_ranges(ntiles, &chunk, &nranges);
  if (chunk > 1) {
    hipLaunchKernelGGL(fold_tiles_kernel<NSTAT>, dim3(nranges), dim3(1024), 0, st, partials,
                       ntiles, chunk);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(gather_folds_kernel<NSTAT>, dim3(1), dim3(1024), 0, st,
                     partials, nranges, chunk, record);
  return hipGetLastError();
}

// For n lattices of ntiles tiles each (device arrays of their partials and
// record bases): records[k] + record_offset = lattice k's sums; its
// partials cleared.  The same sums as close_block_sums for each.
template <int NSTAT>
hipError_t close_block_sums_many(double* const* partials, double* const* records,
                                 size_t record_offset, int n, int ntiles, hipStream_t st) {
  if (ntiles <= 0 || n <= 0) return hipErrorInvalidValue;
  int chunk = 1, nranges = 1;
  fold_ranges(ntiles, &chunk, &nranges);
  if (chunk > 1) {
    hipLaunchKernelGGL(fold_tiles_many_kernel<NSTAT>, dim3(nranges, n), dim3(1024), 0, st,
                       partials, ntiles, chunk);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(gather_folds_many_kernel<NSTAT>, dim3(1, n), dim3(1024), 0,
                     st, partials, nranges, chunk, records, record_offset);
  return hipGetLastError();
}

// For the first n <= kCloseList lattices of a list.
template <int NSTAT>
hipError_t close_block_sums_list(const CloseList& L, int n, hipStream_t st) {
  if (n <= 0 || n > kCloseList) return hipErrorInvalidValue;
  int most = 0;
  for (int i = 0; i < n; ++i) {
    if (L.ntiles[i] <= 0) return hipErrorInvalidValue;
    int chunk = 1, nranges = 1;
    fold_ranges(L.ntiles[i], &chunk, &nranges);
    if (chunk > 1) most = std::max(most, nranges);
  }
  if (most) {
    hipLaunchKernelGGL(fold_tiles_list_kernel<NSTAT>, dim3(most, n), dim3(1024), 0, st, L);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(gather_folds_list_kernel<NSTAT>, dim3(1, n), dim3(1024), 0, st, L);
  return hipGetLastError();
}

// out[NSTAT] = sum of the partials over all tiles (partials unchanged);
// folds: kFoldRows rows of scratch.  Few tiles are summed by one workgroup in
// one launch; above kOpenOneBlock tiles a single workgroup's walk over the
// partials is far below the memory's rate (65536 tiles of 209 statistics,
// 110 MB: 7.2 ms, 15 GB/s), so ranges of tiles go to up to 256 workgroups and
// a second launch adds the ranges in order (0.05 ms).
constexpr int kOpenOneBlock = 64;
template <int NSTAT>
hipError_t open_sums(const double* partials, int ntiles, double* out, double* folds,
                     hipStream_t st) {
  if (ntiles <= 0) return hipErrorInvalidValue;
  if (ntiles <= kOpenOneBlock) {
    hipLaunchKernelGGL(open_folds_kernel<NSTAT>, dim3(1), dim3(1024), 0, st, partials, ntiles,
                       ntiles, out);
    return hipGetLastError();
  }
  const int chunk = std::max(16, (ntiles + kFoldRows - 1) / kFoldRows);
  const int nranges = (ntiles + chunk - 1) / chunk;
  hipLaunchKernelGGL(open_folds_kernel<NSTAT>, dim3(nranges), dim3(1024), 0, st, partials, ntiles,
                     chunk, folds);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(open_gather_kernel<NSTAT>, dim3(1), dim3(SumShape<NSTAT>::VP), 0, st, folds,
                     nranges, out);
  return hipGetLastError();
}

}  // namespace flb
