// SDDMM, group family: a 16-lane group owns 16 consecutive nonzeros of one sparse row (a
// strip, paper Sec. "Sampled Dense--Dense Matrix Multiplication": 1-D tiling over strips of
// consecutive nonzeros).  The lanes split the dot-product dimension four columns at a time,
// so rows of L and R are read contiguously; every lane keeps one partial sum per nonzero of
// the strip, and a transposing reduction over the 16 lanes leaves nonzero t's dot product in
// lane t, which stores it (same section: partial results for all outputs of the tile, then a
// reduction with shuffles).  Column indices are loaded once per strip, pre-scaled to row
// offsets of R, and handed out by DPP row broadcasts.
// Any n from 4 on, any element alignment; k*n < 2^31.
//
// Few entries: strips of four, a wave to a workgroup.  A wave with sixteen rows of R for each of its four groups takes 2 us for
// its 32 KB (64 bytes a clock, and the latency before), on a fraction of the compute units; a quarter of that per wave on all of
// them: 512 x 512 at 10 %, n = 128, 5.48 us -> 3.98 in a graph of launches, of which an empty one takes 1.93.
#pragma once
#include "common.hpp"

namespace spdl {

// x[t] holds this lane's partial sum for nonzero t (16 lanes, 16 nonzeros).  Returns the
// complete sum of nonzero (lane & 15).  row_ror:n hands lane l the value of lane l-n (mod 16).
// Row rotations with bank masks do the first
// two halvings in two instructions per surviving value; the last two use quad permutes.
__device__ __forceinline__ float reduce16x16(float (&x)[16], int l16) {
#define SPDL_ROR(DST, SRC, ROT, BANKS)                                                         \
  asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_ror:" #ROT " row_mask:0xf bank_mask:" #BANKS \
               : "+v"(DST) : "v"(SRC));
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    SPDL_ROR(x[t], x[t], 8, 0x3)          // lanes 0-7:  x[t]   += x[t]   from lane+8
    SPDL_ROR(x[t], x[t + 8], 8, 0xc)      // lanes 8-15: x[t+8] += x[t+8] from lane-8, kept in x[t]
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    SPDL_ROR(x[t], x[t], 12, 0x5)         // lanes with bit 2 clear: += lane+4 (rotate right by 12)
    SPDL_ROR(x[t], x[t + 4], 4, 0xa)      // lanes with bit 2 set:   x[t+4] += lane-4, kept in x[t]
  }
#undef SPDL_ROR
  const bool b1 = (l16 & 2) != 0;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const float keep = b1 ? x[t + 2] : x[t];
    const float send = b1 ? x[t] : x[t + 2];
    x[t] = keep + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                      0, __builtin_bit_cast(int, send), 0x4e /* quad_perm [2,3,0,1] */, 0xf, 0xf, false));
  }
  const bool b0 = (l16 & 1) != 0;
  const float keep = b0 ? x[1] : x[0];
  const float send = b0 ? x[0] : x[1];
  return keep + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                    0, __builtin_bit_cast(int, send), 0xb1 /* quad_perm [1,0,3,2] */, 0xf, 0xf, false));
}

// The same for four nonzeros, whose sums are added up in the same order: that of nonzero t ends in lanes 4 t .. 4 t + 3.
__device__ __forceinline__ float reduce4x16(float (&x)[4]) {
#define SPDL_ROR(DST, SRC, ROT, BANKS)                                                         \
  asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_ror:" #ROT " row_mask:0xf bank_mask:" #BANKS \
               : "+v"(DST) : "v"(SRC));
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    SPDL_ROR(x[t], x[t], 8, 0x3)
    SPDL_ROR(x[t], x[t + 2], 8, 0xc)
  }
  SPDL_ROR(x[0], x[0], 12, 0x5)
  SPDL_ROR(x[0], x[1], 4, 0xa)
#undef SPDL_ROR
  x[0] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x[0]), 0x4e, 0xf, 0xf, false));
  return x[0] + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x[0]), 0xb1, 0xf, 0xf, false));
}

// Dot products of one strip of up to 16 consecutive nonzeros [q, q+16) ∩ [q, end) of `row`,
// rows of L and R gathered straight from global memory.  Called by all 16 lanes of a group.
// The element offset in R of the row that lane l16 of a group gathers for the strip [q, q+16) of a
// sparse row ending at `end`: its own nonzero's column, past the end the last entry's again.
__device__ __forceinline__ int sddmm_strip_offset(int n, int q, int end, int l16,
                                                  const int* __restrict__ column_indices) {
  return column_indices[min(q + l16, end - 1)] * n;
}

// One dot product by one lane, for the rare paths.
template <typename T>
__device__ __forceinline__ float sddmm_plain_dot(int n, const T* l, const T* r) {
  float s = 0.f;
  for (int j = 0; j < n; ++j) s = __builtin_fmaf((float)l[j], (float)r[j], s);
  return s;
}

// n >= 4.  With n % 4 != 0 the lane at the row's end takes the row's last four columns (piece_start)
// and leaves out of its sum, with zeros for L, those that the lane before it has; an Inf there would
// still make the result NaN, so a NaN is looked at again.
// P: pieces of 64 columns whose gathers are all in flight at once.  Two, with strips of four, cost 16 registers more and take
// a memory latency off every strip of more than 64 columns.
// STRIP: nonzeros of a strip, 16 or 4 (lane l16 then has the offset of nonzero l16 / 4).
template <typename T, int P = 1, int STRIP = 16>
__device__ __forceinline__ void sddmm_strip_direct_at(int n, int q, int end, int l16, int roff,
                                                      const T* __restrict__ Lrow, const T* __restrict__ R,
                                                      T* __restrict__ out, const T* __restrict__ scale = nullptr) {
  static_assert(STRIP == 16 || STRIP == 4, "");
  const int cidx = q + l16 * STRIP / 16;
  float partial[STRIP];
#pragma unroll
  for (int t = 0; t < STRIP; ++t) partial[t] = 0.f;
  for (int col0 = 0; col0 < n; col0 += 64 * P) {
    // All gathers are issued before the first multiply-add (the scheduling barrier keeps
    // the compiler from interleaving them with the arithmetic, which it otherwise does whenever
    // the surrounding control flow changes, leaving two loads in flight instead of sixteen).
    float r[P][STRIP][4];
    float l[P][4];
#pragma unroll
    for (int h = 0; h < P; ++h) {
      const int col = col0 + 64 * h + 4 * l16;
      const int lane_off = col < n ? piece_start(col, n, 4) : 0;
#define SPDL_R1(T0, LANE) \
    Pack<T, 4>::load(R + (__builtin_amdgcn_update_dpp(0, roff, 0x150 + (LANE), 0xf, 0xf, false) + lane_off), r[h][T0]);
      if constexpr (STRIP == 16) {
        SPDL_R1(0, 0) SPDL_R1(1, 1) SPDL_R1(2, 2) SPDL_R1(3, 3) SPDL_R1(4, 4) SPDL_R1(5, 5) SPDL_R1(6, 6) SPDL_R1(7, 7)
        SPDL_R1(8, 8) SPDL_R1(9, 9) SPDL_R1(10, 10) SPDL_R1(11, 11) SPDL_R1(12, 12) SPDL_R1(13, 13) SPDL_R1(14, 14) SPDL_R1(15, 15)
      } else {
        SPDL_R1(0, 0) SPDL_R1(1, 4) SPDL_R1(2, 8) SPDL_R1(3, 12)
      }
#undef SPDL_R1
      Pack<T, 4>::load(Lrow + lane_off, l[h]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < P; ++h) {
      const int col = col0 + 64 * h + 4 * l16;
      const int colc = col < n ? piece_start(col, n, 4) : 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) l[h][v] = col < n && colc + v >= col ? l[h][v] : 0.f;
#pragma unroll
      for (int t = 0; t < STRIP; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) partial[t] = __builtin_fmaf(l[h][v], r[h][t][v], partial[t]);
    }
  }
  float total;
  if constexpr (STRIP == 16) total = reduce16x16(partial, l16);
  else total = reduce4x16(partial);
  const bool mine = cidx < end && (STRIP == 16 || (l16 & 3) == 0);
  if ((n & 3) != 0 && mine && total != total) total = sddmm_plain_dot<T>(n, Lrow, R + roff);
  if (mine) sddmm_store<T>(out, scale, cidx, total);
}

template <typename T>
__device__ __forceinline__ void sddmm_strip_direct(int n, int q, int end, int l16, const T* __restrict__ Lrow,
                                                   const int* __restrict__ column_indices,
                                                   const T* __restrict__ R, T* __restrict__ out,
                                                   const T* __restrict__ scale = nullptr) {
  sddmm_strip_direct_at<T>(n, q, end, l16, sddmm_strip_offset(n, q, end, l16, column_indices), Lrow, R, out, scale);
}

// Work is split by nonzeros, not by rows: every wave owns `per_wave` consecutive entries of
// the CSR arrays (a multiple of 64), finds the row of its first entry with a binary search in
// the row offsets, and walks on from there.  The walk is wave-uniform (scalar loads and
// arithmetic): it cuts the range into strips of up to 16 entries that end at row ends and
// deals them to the four 16-lane groups, four at a time, so consecutive strips of one row
// share its L row in cache and short rows still keep all four groups busy.  Outputs are
// independent, so rows shared by several waves need no reduction, and the load per wave is
// the same whatever the row lengths are (the balance the paper gets for SpMM from the row
// swizzle, Sec. "Row Swizzle Load Balancing", without needing a row order in the interface).
template <typename T, int P = 1, int STRIP = 16>
__global__ __launch_bounds__(STRIP == 16 ? 256 : 64) void sddmm_group_kernel(
    int m, int n, int nnz, int per_wave, const int* __restrict__ row_offsets,
    const int* __restrict__ column_indices, const T* __restrict__ L, const T* __restrict__ R,
    T* __restrict__ out, const T* __restrict__ scale) {
  const int l16 = threadIdx.x & 15;
  const int sub = (threadIdx.x & 63) >> 4;
  const int wave = STRIP == 16 ? uniform(blockIdx.x * 4 + (threadIdx.x >> 6)) : (int)blockIdx.x;
  const long long first = (long long)wave * per_wave;
  if (first >= nnz) return;
  int p = (int)first;
  const int range_end = (int)min((long long)nnz, first + per_wave);
  // Last row whose offset is <= p: the row of entry p (rows in between are empty).  A 64-way
  // search, one probe per lane: three rounds of dependent loads for up to 2^18 rows.
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = m;                          // invariant: row_offsets[lo] <= p < row_offsets[hi]
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6;
    const int probe = lo + (lane + 1) * step;
    const bool le = probe < hi && row_offsets[min(probe, hi)] <= p;     // true for a prefix of the lanes
    const int cnt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(le));
    lo += cnt * step;
    hi = min(hi, lo + step);
  }
  int row = lo;
  int row_end = row_offsets[row + 1];
  // The walk runs one round ahead of the arithmetic: the column indices of the next round's strips
  // are requested before the current round's gathers are waited for, so a round costs one memory
  // latency (the rows of R), not two in a row (indices, then rows).
  int cur_row = 0, cur_q = 0, cur_end = 0, cur_off = 0;
  bool have = false;
  while (true) {
    int my_row = 0, my_q = 0, my_end = 0;
    const bool next = p < range_end;
    if (next) {
      while (row_end <= p) {                     // p reached the end of this row: next non-empty row
        ++row;
        row_end = row_offsets[row + 1];
      }
      const int seg_end = min(row_end, range_end);
      if (p + 4 * STRIP <= seg_end) {            // four full strips of the same row
        my_row = row;
        my_q = p + STRIP * sub;
        my_end = seg_end;
        p += 4 * STRIP;
      } else {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if (p < range_end) {
            while (row_end <= p) {
              ++row;
              row_end = row_offsets[row + 1];
            }
            const int e = min(row_end, range_end);
            if (sub == g) { my_row = row; my_q = p; my_end = e; }
            p = min(p + STRIP, e);
          }
        }
      }
    }
    int my_off = 0;
    if (my_q < my_end) my_off = sddmm_strip_offset(n, my_q, my_end, l16 * STRIP / 16, column_indices);
    if (have && cur_q < cur_end)
      sddmm_strip_direct_at<T, P, STRIP>(n, cur_q, cur_end, l16, cur_off, L + (size_t)cur_row * n, R, out, scale);
    if (!next) break;
    cur_row = my_row; cur_q = my_q; cur_end = my_end; cur_off = my_off;
    have = true;
  }
}

}  // namespace spdl
