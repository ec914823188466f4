// SDDMM, row-strip family, dot products of fewer than four columns (wider ones: the strips of
// sddmm_group.hpp).  One wave owns strips of 64 consecutive nonzeros of one sparse row, a nonzero to a lane
// (paper Sec. "Sampled Dense--Dense Matrix Multiplication", 1-D tiling over nonzero strips): with one to
// three columns there is nothing to share out among lanes, and no lane multiplies what is not its
// own (0 * Inf).  `split` waves share a row, taking strips round-robin, so the grid is m*split waves.
// Bound by the gathers of R, 64 cache lines per load.  (64 lanes to a strip's dot products, as this kernel did at any
// width: 61 or more of them idle; 8192 x 10240 at 10 %, n = 3: 1680 us against 53; 1024 x 1024, n = 2: 73 against 2.6.)
#pragma once
#include "common.hpp"
#include "sddmm_group.hpp"

namespace spdl {

template <typename T>
__global__ __launch_bounds__(256) void sddmm_rowstrip_kernel(
    int m, int n, int split, const int* __restrict__ row_offsets,
    const int* __restrict__ column_indices, const T* __restrict__ L, const T* __restrict__ R,
    T* __restrict__ out, const T* __restrict__ scale) {
  const int lane = threadIdx.x % kWave;
  const int wave = uniform(blockIdx.x * 4 + threadIdx.x / kWave);
  const int row = wave / split;
  const int part = wave - row * split;
  if (row >= m) return;
  const int end = row_offsets[row + 1];
  for (int p = row_offsets[row] + part * kWave + lane; p < end; p += split * kWave)
    sddmm_store<T>(out, scale, p, sddmm_plain_dot<T>(n, L + (size_t)row * n, R + (size_t)column_indices[p] * n));
}

}  // namespace spdl
