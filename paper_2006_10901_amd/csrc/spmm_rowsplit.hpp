// SpMM, row-splitting family: a group of G lanes owns one sparse row and a 1-D tile of
// G*VEC output columns (paper Sec. "Hierarchical 1-Dimensional Tiling" and "Subwarp Tiling").
// Dense rows of B are gathered straight from global memory, one vector load per lane per
// nonzero.  This is the general kernel: any n, any alignment, any column order inside a row.
#pragma once
#include "common.hpp"

namespace spdl {

// I is the type of the column indices (int32, or int16 in the mixed-precision form of paper Sec.
// "Mixed Precision", which halves the index traffic).
// SEG lane groups of one wave share a row: group s takes the batches s, s+SEG, ... of the row's
// nonzeros and the partial sums are added across the groups at the end.  Used when there are too
// few rows to fill the machine with one group per row (each lane then walks a shorter list).
// WAVES = 4: all four waves of a workgroup share a row, the waves' sums are added through LDS.  (What bounds the smallest problems is the
// chain of latencies: offsets, indices, a batch of rows of B after the other.)
// TEAM (a wave per row): a row of more than team_above entries is walked by the workgroup's four waves, each a quarter of its batches, and
// added up through LDS by the wave whose row it is.  What bounds rows of unequal length is the chain of the longest one, which the row order
// starts first but cannot shorten: 1172 x 731, log-normal rows of 84, n = 392 in half precision: 32.4 us -> 10.7.  Whether a row is shared
// depends on its own length alone, so that the order of the rows does not change the bits.
template <typename T, int VEC, int G, typename I = int, int SEG = 1, int WAVES = 1, bool TEAM = false>
__global__ __launch_bounds__(256) void spmm_rowsplit_kernel(
    int m, int n, const int* __restrict__ row_offsets,
    const I* __restrict__ column_indices, const T* __restrict__ values, const int* __restrict__ row_order,
    const T* __restrict__ B, T* __restrict__ C, const T* __restrict__ bias, int relu, int team_above) {
  static_assert(G * SEG <= kWave && (WAVES == 1 || (WAVES == 4 && G * SEG == kWave)), "groups of one wave, or of all four");
  static_assert(!TEAM || (G == kWave && WAVES == 1), "a wave per row");
  constexpr int ALL = SEG * WAVES;
  constexpr int U = (G == kWave && VEC * sizeof(T) <= 16) ? 16 : 8;   // nonzeros in flight per lane
  const int sub = threadIdx.x / G;
  const int lane = threadIdx.x % G;
  // Row binning and bundling (paper Sec. "Row Swizzle Load Balancing"): the rows of one wave
  // are adjacent in the row order (a bundle of similar lengths, so the lanes of a wave finish
  // together), while the four waves of a block take bundles a quarter of the order apart, so
  // every block, and with it every CU, gets the same mix of long and short rows.
  constexpr int RPW = kWave / (G * SEG);               // rows per wave
  const int wave_in_block = TEAM ? uniform(threadIdx.x / kWave) : (int)threadIdx.x / kWave;
  const int seg = WAVES == 1 ? sub % SEG : sub;
  const int slot = TEAM ? wave_in_block * (int)gridDim.x + (int)blockIdx.x
                   : WAVES == 1 ? (wave_in_block * (int)gridDim.x + (int)blockIdx.x) * RPW + (sub / SEG) % RPW : (int)blockIdx.x;
  if (!TEAM && slot >= m) return;
  int row = -1, start = 0, end = 0;                      // (no row: the wave is there to help)
  int from[4], to[4], team = 0;                          // the workgroup's rows, those that are shared
  if constexpr (TEAM) {
    int r[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) r[w] = min(w * (int)gridDim.x + (int)blockIdx.x, m - 1);
    if (row_order) {                                       // (all four loads at once)
#pragma unroll
      for (int w = 0; w < 4; ++w) r[w] = row_order[r[w]];
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      from[w] = row_offsets[r[w]];
      to[w] = row_offsets[r[w] + 1];
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const bool there = w * (int)gridDim.x + (int)blockIdx.x < m;
      if (there && to[w] - from[w] > team_above) team |= 1 << w;
      if (w == wave_in_block && there) {
        row = r[w];
        start = from[w];
        end = to[w];
      }
    }
  } else {
    row = row_order ? row_order[slot] : slot;              // row swizzle: one extra load
    if (G * SEG == kWave) row = uniform(row);              // whole wave on one row: scalar loads
    start = row_offsets[row];
    end = row_offsets[row + 1];
  }
  const int col = piece_start((blockIdx.y * G + lane) * VEC, n, VEC);
  const bool active = col < n;
  const T* Bcol = B + (active ? col : 0);

  float acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.f;

  // Adds every step-th batch of U nonzeros of [from, to), from the first-th on.
  auto walk = [&](int from, int to, int first, int step) __attribute__((always_inline)) {
    int p = from + first * U;
    // Full batches of U nonzeros.  The values and column indices of the next batch are requested
    // before the gathers of the current one are waited for, so a batch costs one memory latency
    // (the rows of B), not two in a row (indices, then rows).  The indices go first: the gathers' addresses
    // wait for them alone.  (The values first, with lane groups of 8 and 16 and narrow pieces: 8000 rows of 300, n = 5: 30.7 us
    // against 23.0; 1420 rows of 184, n = 11: 13.5 against 10.8; elsewhere level.  Not where a wave has one row: scalar loads.)
    auto fetch = [&](int q, float& value, int& column) __attribute__((always_inline)) {
      if (G == kWave) value = (float)values[q];
      column = (int)column_indices[q];
      if (G < kWave) value = (float)values[q];
    };
    float a[U];
    int c[U];
    if (p + U <= to) {
#pragma unroll
      for (int u = 0; u < U; ++u) fetch(p + u, a[u], c[u]);
    }
    for (; p + U <= to; p += step * U) {
      float b[U][VEC];
#pragma unroll
      for (int u = 0; u < U; ++u) Pack<T, VEC>::load(Bcol + (size_t)c[u] * n, b[u]);
      float an[U];
      int cn[U];
      const int pn = p + step * U;
      if (pn + U <= to) {
#pragma unroll
        for (int u = 0; u < U; ++u) fetch(pn + u, an[u], cn[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = __builtin_fmaf(a[u], b[u][v], acc[v]);
#pragma unroll
      for (int u = 0; u < U; ++u) { a[u] = an[u]; c[u] = cn[u]; }
    }
    // after the full batches, p is the start of this group's next batch: past the row end for every
    // group but the one that owns the short last batch
    // What is left of the row, fewer than U nonzeros: R at once as well (one after the other each costs two
    // memory latencies, index and row of B: 512 x 512 at 10 %, n = 128: 5.5 us against 5.05; 8192 x 8192 with
    // rows of 8, n = 128: 8.5 against 6.8).  Four where a wave works on one row; one where half-precision rows
    // are loaded in narrow pieces, which takes so many waves that the instructions count, not the latency.
    constexpr int R = sizeof(T) == 2 && VEC < 8 ? 1 : G == kWave ? 4 : U;
    typedef T raw __attribute__((ext_vector_type(VEC)));
    typedef raw raw_any __attribute__((aligned(sizeof(T))));
    for (; p < to; p += R) {
      // (as stored: a conversion beside a load that not all lanes make would wait for it)
      T ra[R];
      raw rb[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        ra[u] = (T)0.f;
        c[u] = 0;
        if (p + u < to) { ra[u] = values[p + u]; c[u] = (int)column_indices[p + u]; }
      }
      // (the first value is needed last, and the compiler would load it after the rows of B, a latency later)
      if constexpr (G == kWave && sizeof(T) == 4 && SEG * WAVES == 1) asm volatile("" : "+s"(ra[0]));
#pragma unroll
      for (int u = 0; u < R; ++u) {
        rb[u] = (raw)(T)0.f;
        if (p + u < to) rb[u] = *reinterpret_cast<const raw_any*>(Bcol + (size_t)c[u] * n);
      }
#pragma unroll
      for (int u = 0; u < R; ++u)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = __builtin_fmaf((float)ra[u], (float)rb[u][v], acc[v]);
      if (R == U) break;                                   // (SEG groups: only one of them owns a short batch)
    }
  };
  auto finish = [&]() __attribute__((always_inline)) {
    spmm_epilogue<T, VEC>(acc, bias, row, relu);
    if (active) Pack<T, VEC>::store(C + (size_t)row * n + col, acc);
  };
  constexpr int kHelpers = WAVES > 1 || TEAM ? 3 : 1;
  __shared__ float sums[kHelpers][VEC][G];
  if constexpr (TEAM) {
    if (row >= 0 && !(team >> wave_in_block & 1)) {
      walk(start, end, 0, 1);
      finish();
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    }
    for (; team != 0; team &= team - 1) {
      const int w = __builtin_ctz(team);
      const int f = w == 0 ? from[0] : w == 1 ? from[1] : w == 2 ? from[2] : from[3];
      const int t = w == 0 ? to[0] : w == 1 ? to[1] : w == 2 ? to[2] : to[3];
      const int part = (wave_in_block - w) & 3;
      walk(f, t, part, 4);
      if (part > 0) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          sums[part - 1][v][lane] = acc[v];
          acc[v] = 0.f;
        }
      }
      __syncthreads();
      if (part == 0) {                                     // (its own row)
#pragma unroll
        for (int h = 0; h < 3; ++h)
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[v] += sums[h][v][lane];
        finish();
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
      }
      if ((team & (team - 1)) != 0) __syncthreads();
    }
    return;
  }
  walk(start, end, seg, ALL);
  if (SEG > 1) {
#pragma unroll
    for (int d = G; d < G * SEG; d *= 2)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] += __shfl_xor(acc[v], d, kWave);
  }
  if constexpr (WAVES > 1) {
    if (wave_in_block > 0 && threadIdx.x % kWave < G) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) sums[wave_in_block - 1][v][lane] = acc[v];
    }
    __syncthreads();
    if (wave_in_block > 0) return;
#pragma unroll
    for (int w = 0; w < WAVES - 1; ++w)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] += sums[w][v][lane];
  }
  if (seg != 0) return;
  finish();
}

}  // namespace spdl
