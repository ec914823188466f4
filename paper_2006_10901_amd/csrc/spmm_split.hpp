// SpMM of dense sparse matrices on the matrix cores, fp32: whole blocks of A, zeros included, times B, from products of two
// fp16 terms per number.
//
// A number taken times a power of two is high + low / 2048, both fp16: low is the rounded rest, which has at most one bit more than fp16
// holds, so what is left out is no more than 2^-23 of the number.  All four products of terms are taken: high high in one
// accumulator, the three small ones in another, so that these are not rounded to the large sum's last place one by one.  The power of two
// is chosen for each row of A and for each column of B (and quarter of A's columns), from the first numbers that are not zero, whose
// largest comes to 2^12 .. 2^13; a number beyond 2^15 makes it smaller, and the sums so far with it.  Numbers far below the row's or
// column's largest lose bits of `low` to fp16's smallest exponent, so that a sum may be wrong that is small beside what these two could give:
// such sums are gathered (scaled_floor, by the powers of two that the row and the quarters of the column have in the end, the smallest ones), unless
// there are several and a count shows that too few numbers have lost any (kDsCount).
//
// A workgroup owns 64 sparse rows and 64 columns of C and walks A's columns in stages of 128.  Eight waves scatter: sixteen lanes to
// a row, they find the row's entries of the stage by a cursor, take each apart into its terms and write these into a block of
// zeros in LDS, in the order in which the lanes read them as MFMA operands.  Eight waves multiply: each has 32 of the 64 columns and a
// quarter of the stage's columns of A, copies its rows of B into a ring of its own in LDS (16 bytes per lane: loaded into registers, a lane's operand
// takes an instruction for each of its numbers, 18 clocks of the compute unit's address path apiece), splits
// them in registers, one step of sixteen ahead, and multiplies them with both 32-row tiles of the block; the quarters are
// added at the end.  Three blocks: one is multiplied, the next one written, the one before cleared, a barrier per stage, which
// a multiplying wave reaches with what it still needs of the block in registers, so that half a step of products lies behind it.
//
// Against 64 bits, normally distributed values, 2-norm of the error over that of the result: rows of 30 % of 10240 columns 3.2e-7, where six
// products of three bf16 terms in one accumulator have 7.0e-7 and the slab kernel 9.9e-7.  With few entries the roundings of a sum that are no
// entry's count: such rows are gathered (kDsEntries).
//
// What bounds it: the power limit (1.5 .. 1.7 GHz) and the issue of vector instructions beside the MFMA.  A stage is 64 MFMA of 32 clocks on two of a
// SIMD's waves, 170 vector instructions of these and 130 (10 %) to 260 (30 %) of the scattering waves, 4 clocks each or 5 where a wave is
// alone; it takes 2700 to 3100 clocks.  8192 x 10240 at 10 / 30 %, n = 128, launches back to back, 136 / 161 us: without MFMA 101 / 123, without storing what is
// scattered 123 / 141, without copies of B 116 / 147, without the three small products' smallest 125 / 152.  (A launch among others finds the chip
// cooler: 113 / 133.)  A step's operands all read a step ahead, one accumulator and registers for
// two blocks instead: 7 % slower.  8192 x 10240, n = 128, three bf16 terms and six products -> here, inputs in turn: 20 % 136.8 us -> 126.5, 30 %
// 149.8 -> 132.9; 5923 x 6704 at 20 % 77.6 -> 69.6; 4368 x 5000 at 20 % 56.4 -> 53.6 (slab kernel at these: 143, 200, 86.6, 65.1).
//
// Rows that are not ascending, or hold a column twice, are noticed (an entry that does not come right after a smaller column of the
// same stage; a cursor short of the row's end) and gathered at the end (split_gather), as is what is not finite: a zero of the
// block times an infinity of B must not reach the result.  (Sums from some 2^98 of B's numbers' on come out as infinities too, and are gathered.)
#pragma once
#include "f16_split.hpp"

namespace spdl {

constexpr int kDsRows = 64;                              // sparse rows per workgroup
constexpr int kDsCols = 64;                              // columns of C per workgroup
constexpr int kDsS = 128;                                // columns of A per stage
constexpr int kDsGroup = kDsRows * 16 + 16;              // bytes of eight columns, one term: the next eight lie four banks on
constexpr int kDsPlane = kDsS / 8 * kDsGroup;            // one term of a stage's block of A
constexpr int kDsBuf = 2 * kDsPlane;
constexpr int kDsMulWaves = 8, kDsScatterWaves = 8;
constexpr int kDsThreads = 64 * (kDsMulWaves + kDsScatterWaves);
constexpr int kDsRing = 3, kDsChunk = 16 * 32 * 4;       // a multiplying wave's sixteen rows of 32 columns of B, as they come
constexpr int kDsRingOff = 3 * kDsBuf;
constexpr int kDsRedoOff = kDsRingOff + kDsMulWaves * kDsRing * kDsChunk;
constexpr int kDsScaleOff = kDsRedoOff + kDsRows * 4;
constexpr int kDsShiftOff = kDsScaleOff + kDsRows * 4;
constexpr int kDsLdsBytes = kDsShiftOff + 3 * kDsRows * 8 + 16;
// In the shifts' place, in the end: by the quarter and the column of B what a scaled one is, 0 if all are zeros; the rows' scaled_floor, likewise.
constexpr int kDsUnitOff = kDsShiftOff, kDsFloorOff = kDsUnitOff + 4 * kDsCols * 4;
static_assert(kDsFloorOff + kDsRows * 4 <= kDsShiftOff + 3 * kDsRows * 8, "LDS");

// Results that the matrix cores cannot give, from the rows of B themselves: of row i of the workgroup the fours of columns that lane i's `mask`
// names.  The threads of the workgroup share out the list of all such fours and parts of each one's entries, sixteen of
// them in flight for each thread: a single four waits for a few gathers, not for as many as its row has sixteens, fours here and there take as many
// threads as they are, and where whole rows are needed sixteen lanes read 256 bytes of B in a row.  A part whose sums are
// all NaN already is done.  (8192 x 10240 at 30 %, n = 128, inputs from a fresh generator, 149 us with nothing
// to gather: one infinity in B 281, a row of them 671; sums below scaled_floor: a row of B 2^10 times the others 128, 2^20 times 307; A and B
// log-normal, sigma 1 / 3, 165 / 262.  With whole rows shared out, not fours, and nothing counted (kDsCount): 2^20 634, log-normal 165 / 462; sums that
// are small and right, A and B all +-1, where one in 140 is zero, 476, of -1, 0 and 1 688, B with one number in a thousand that is not zero 681:
// now 158, 161, 166.  What is gathered is read from the L2s entry by entry, all of it at their rate.)
__device__ __forceinline__ void split_gather(unsigned mask, int i0, int j0, int m, int n,
                                             const int* __restrict__ row_offsets, const int* __restrict__ column_indices,
                                             const float* __restrict__ values, const float* __restrict__ B, float* __restrict__ C,
                                             const float* __restrict__ bias, int relu, char* lds) {
  const int tid = threadIdx.x, lane = tid & 63;
  f32x4* const sums = reinterpret_cast<f32x4*>(lds);                   // (the products' sums before have been read)
  unsigned short* const list = reinterpret_cast<unsigned short*>(lds + 16 * kDsThreads);
  int through = __builtin_popcount(mask);                              // fours of the rows up to the lane's
#pragma unroll
  for (int d = 1; d < kWave; d *= 2) {
    const int before = __shfl_up(through, d, kWave);
    through += lane >= d ? before : 0;
  }
  const int fours = __builtin_amdgcn_readlane(through, 63);
  if (tid < kWave) {
    int at = through - __builtin_popcount(mask);
    for (unsigned left = mask; left != 0; left &= left - 1) list[at++] = (unsigned short)(lane * 16 + __builtin_ctz(left));
  }
  __syncthreads();
  const int parts = min(kDsThreads / fours, 64), part = tid / fours;
  const bool on = part < parts;
  const int which = list[on ? tid - part * fours : 0];
  const int row = i0 + which / 16, first = j0 + 4 * (which & 15), col = min(first, n - 4);  // (the last four columns of B's row at its end)
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  if (on) {
    constexpr int U = 16;
    const int begin = row_offsets[row], end = row_offsets[row + 1];
    const int share = end - begin > 2 * U ? parts : 1;                 // (an entry by itself would be rounded once more)
    const float* const Bcol = B + col;
    for (int p = part < share ? begin + U * part : end; p < end; p += U * share) {
      int c[U];
      float a[U], b[U][4];
      if (p + U <= end) {
        typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int u = 0; u < U; u += 4) {
          const i32x4_any x = *reinterpret_cast<const i32x4_any*>(column_indices + p + u);
          const f32x4_any y = *reinterpret_cast<const f32x4_any*>(values + p + u);
#pragma unroll
          for (int t = 0; t < 4; ++t) { c[u + t] = x[t]; a[u + t] = y[t]; }
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = column_indices[min(p + u, end - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = values[min(p + u, end - 1)];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) Pack<float, 4>::load(Bcol + (size_t)c[u] * n, b[u]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (p + u < end) {
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = __builtin_fmaf(a[u], b[u][t], v[t]);
        }
      if (v[0] != v[0] && v[1] != v[1] && v[2] != v[2] && v[3] != v[3]) break;
    }
  }
  sums[tid] = f32x4{v[0], v[1], v[2], v[3]};
  __syncthreads();
  if (!on || part > 0) return;
#pragma unroll 4
  for (int i = 1; i < parts; ++i) {
    const f32x4 x = sums[tid + i * fours];
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] += x[t];
  }
  spmm_epilogue<float, 4>(v, bias, row, relu);
  float* const c = C + (size_t)row * n + col;
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (col + t >= first) c[t] = v[t];
}

// Entries from which on a row's sum on the matrix cores is no less exact than a chain of multiply-adds: 2-norm of the error over the chain's, rows
// of 20 / 30 / 40 / 100 / 500 entries 1.05 / 0.92 / 0.81 .. 0.86 / 0.60 / 0.31 .. 0.48, at 833 .. 10240 columns alike (of 2: 2.2).
constexpr int kDsEntries = 32;

// Fours of columns with a sum below the floor of its entries from which on the numbers that lose bits (scaled_loses) are counted, in the tile of B and in
// these rows of A, before what is still below the floor of as many products is gathered.  (Numbers rounded to whole ones, from more
// to fewer sums of zero, us, counted / not: 8192 x 10240 at 30 %, 2 / 7 / 12 / 27 fours of a workgroup 137 / 141 / 141 / 142 and 133 / 164 / 189 / 245; 8192 x 3000 at
// 20 %, 4 / 16 / 28 / 61 fours 50 / 50 / 50 / 51 and 45 / 51 / 55 / 71; 4096 x 1024 at 30 %, n = 1024, 2 / 6 / 23 fours 89 / 89 / 90 and 84 / 91 / 109.  Of normally
// distributed numbers one workgroup in ten has one.)
constexpr int kDsCount = 8;

// NC sixteens of a row's entries fetched a stage ahead.  (k >= 16, n >= 4, 0 < nnz < 2^28.)
template <int NC>
__global__ __launch_bounds__(kDsThreads) void spmm_split_kernel(
    int m, int k, int n, int nnz, int tiles_n, int panels, const int* __restrict__ row_offsets,
    const int* __restrict__ column_indices, const float* __restrict__ values, const float* __restrict__ B,
    float* __restrict__ C, const float* __restrict__ bias, int relu, int tiles_first) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  int panel, tile;
  if (tiles_first ? !slab_wg_map(blockIdx.x, tiles_n, panels, tile, panel)
                  : !slab_wg_map(blockIdx.x, panels, tiles_n, panel, tile)) return;
  const int i0 = panel * kDsRows;
  const int nst = (k + kDsS - 1) / kDsS;
  PhaseClocks clocks;
  clocks.start();
  int* const redo = reinterpret_cast<int*>(lds_raw + kDsRedoOff);       // rows to be gathered
  int* const row_scale = reinterpret_cast<int*>(lds_raw + kDsScaleOff);
  // {stage + 1, by how many powers of two the row's sums go down before it}, and the stage + 1 of which a row has such
  i32x2* const row_shift = reinterpret_cast<i32x2*>(lds_raw + kDsShiftOff);
  int* const shifted = reinterpret_cast<int*>(lds_raw + kDsShiftOff + 3 * kDsRows * 8);
  auto barrier = [&]() __attribute__((always_inline)) {                // (no wait for memory)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < (3 * kDsBuf + 16 * kDsThreads - 1) / (16 * kDsThreads); ++i)
      if ((i * kDsThreads + tid) * 16 < 3 * kDsBuf) *reinterpret_cast<f32x4*>(lds_raw + (i * kDsThreads + tid) * 16) = zero;
    if (tid < 3 * kDsRows) row_shift[tid] = i32x2{0, 0};
    if (tid < 3) shifted[tid] = 0;
  }
  barrier();

  if (wave < kDsMulWaves) {
    const int r = lane & 31, h = lane >> 5, quarter = wave & 3, half = wave >> 2;
    const int col0 = tile * kDsCols + half * 32;
    // B's rows come by way of LDS, sixteen of them in a kilobyte pair of this wave's own, three steps ahead: row 8 h + e, column
    // r of them is at 256 e + 128 h + 4 r, so that the lanes read 256 bytes in a row.  A lane brings four columns of a row;
    // the four that would reach past the row's end start at n - 4.  (Columns past n: those of the last four.)
    char* const ring = lds_raw + kDsRingOff + wave * (kDsRing * kDsChunk);
    const unsigned ring_m0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)ring;
    const unsigned row_bytes = (unsigned)n * 4u;
    const unsigned lane_off = (unsigned)(8 * ((lane >> 3) & 1) + (lane >> 4)) * row_bytes + (unsigned)min(col0 + 4 * (lane & 7), n - 4) * 4u;
    const int piece = min(col0 + (r & ~3), n - 4);
    const char* const ring_lane = ring + h * 128 + (r & ~3) * 4 + min(col0 + r - piece, 3) * 4;
    // Rows of the wave's columns: step 2 q + s is columns 128 q + 32 quarter + 16 s .. of A.  The sixteen that k ends in, and steps
    // past it, take A's last sixteen: an entry of theirs is scattered to where its row of B then comes.
    auto bring = [&](int q, int s, unsigned slot) __attribute__((always_inline)) {
      const int k0 = uniform(min(q * kDsS + quarter * 32 + s * 16, k - 16));
      const float* const base = B + (size_t)k0 * (unsigned)n;
      const unsigned to = ring_m0 + slot * kDsChunk;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %4"
                   :: "s"(to), "s"(to + kDsChunk / 2), "v"(lane_off), "s"(base), "s"(base + (size_t)4 * (unsigned)n) : "memory", "m0");
    };
    float raw[8];
    auto read_b = [&](unsigned slot) __attribute__((always_inline)) {  // (all but the last two chunks that were asked for are there)
      asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      const char* const p = ring_lane + slot * kDsChunk;
#pragma unroll
      for (int e = 0; e < 8; ++e) raw[e] = *reinterpret_cast<const float*>(p + e * 256);
    };
    int scale = kNoScale, shift = 0;                                 // of the lane's column: the exponent of the power of two it is taken times
    float limit = 0.f;
    unsigned long long raised = 0;
    struct Terms { f16x8 high, low; };
    auto split = [&]() __attribute__((always_inline)) -> Terms {
      float largest = __builtin_fabsf(raw[0]);
#pragma unroll
      for (int e = 1; e < 8; ++e) largest = fmaxf(largest, __builtin_fabsf(raw[e]));
      raised = __builtin_amdgcn_ballot_w64(largest > limit);
      if (__builtin_expect(raised != 0, 0)) {
        largest = max_of_halves(largest);                              // (the column's other half)
        const int to = largest > limit ? scale_for(largest) : scale;
        shift = to - scale;
        scale = to;
        limit = largest > limit ? scale_limit(to) : limit;
      }
      const float times = __builtin_bit_cast(float, scale << 23);
      Terms t;
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        f16x2 x, y;
        split_f16(raw[e], raw[e + 1], times, x, y);
        t.high[e] = x[0]; t.high[e + 1] = x[1];
        t.low[e] = y[0]; t.low[e + 1] = y[1];
      }
      return t;
    };
    // A lane's operand of a term, eight columns of row 32 i + r: 16 bytes at group * kDsGroup + 512 i + 16 r.
    const unsigned a_off = (unsigned)((4 * quarter + h) * kDsGroup + (r << 4));
    f16x8 high[2], low[2];
    auto load_a = [&](f16x8 (&x)[2], const char* p) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = *reinterpret_cast<const f16x8*>(p + i * 512);
    };
    acc32x32 sum[2], rest[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int x = 0; x < 16; ++x) sum[i][x] = rest[i][x] = 0.f;
    auto two = [&](acc32x32 (&to)[2], const f16x8 (&x)[2], const f16x8& y) __attribute__((always_inline)) {
      to[0] = mfma_f16(x[0], y, to[0]);
      to[1] = mfma_f16(x[1], y, to[1]);
    };
    // (chunk t is in slot t % kDsRing)
    unsigned slot = 0;
    auto next_slot = [](unsigned x) { return x == kDsRing - 1 ? 0u : x + 1u; };
    int bring_q = 0, bring_s = 0;
    auto bring_next = [&](unsigned to) __attribute__((always_inline)) {
      bring(bring_q, bring_s, to);
      bring_s ^= 1;
      if (bring_s == 0) ++bring_q;
    };
    for (unsigned i = 0; i < kDsRing; ++i) bring_next(i);
    read_b(0);
    Terms b = split();
    asm volatile("" :: "v"(b.high), "v"(b.low));                       // (the chunk has been read)
    bring_next(0);
    read_b(1);
    slot = 1;                                                          // of the chunk in `raw`
    barrier();                                                         // the first stage's block is there
    load_a(high, lds_raw + a_off);
    load_a(low, lds_raw + a_off + kDsPlane);
    clocks.lap(kPhaseSetup);
    char* const clear = lds_raw + wave * (kDsBuf / kDsMulWaves) + lane * 16;
    static_assert(kDsBuf / kDsGroup % kDsMulWaves == 0, "whole groups for a wave");
    // One step of sixteen columns; `next` is where the next one's operands are, each read as soon as its registers are done
    // with.  `last` of a stage: half of the products need nothing of the stage's block that is not in registers.
    auto step = [&](const char* next, bool last, int before, int q, int x) __attribute__((always_inline)) {
      const Terms c = split();
      two(rest, low, b.low * (_Float16)(1.f / kLowScale));
      two(rest, low, b.high);
      asm volatile("" :: "v"(c.high), "v"(c.low));
      bring_next(slot);
      slot = next_slot(slot);
      if (last) {
        clocks.lap(kPhaseSteps);
        __builtin_amdgcn_sched_barrier(0);
        barrier();                                                     // this block may be cleared; the next one is there
        clocks.lap(kPhaseBarrier);
      }
      const int other_scales = last ? shifted[x] : 0;
      load_a(low, next + kDsPlane);
      read_b(slot);
      if (!last) {
        const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < kDsBuf / kDsGroup / kDsMulWaves; ++i) *reinterpret_cast<u32x4*>(clear + before * kDsBuf + i * kDsGroup) = zero;
      }
      two(rest, high, b.low);
      two(sum, high, b.high);
      load_a(high, next);
      if (__builtin_expect(raised != 0, 0)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int t = 0; t < 16; ++t) {
            sum[i][t] = __builtin_ldexpf(sum[i][t], shift);
            rest[i][t] = __builtin_ldexpf(rest[i][t], shift);
          }
        shift = 0;
      }
      if (last && __builtin_expect(uniform(other_scales) == q + 2, 0)) {   // rows of the next stage go by another power of two
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int t = 0; t < 16; ++t) {
            const i32x2 down = row_shift[x * kDsRows + 32 * i + 8 * (t / 4) + 4 * h + t % 4];
            const int by = down.x == q + 2 ? down.y : 0;
            sum[i][t] = __builtin_ldexpf(sum[i][t], by);
            rest[i][t] = __builtin_ldexpf(rest[i][t], by);
          }
      }
      b = c;
      __builtin_amdgcn_sched_barrier(0);
    };
    int x = 0, before = 2;
    for (int q = 0; q < nst; ++q) {
      const int next = x == 2 ? 0 : x + 1;
      step(lds_raw + x * kDsBuf + 2 * kDsGroup + a_off, false, before, q, next);
      step(lds_raw + next * kDsBuf + a_off, true, before, q, next);
      before = x;
      x = next;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // (what was asked for past the end)
    barrier();
    // This wave's sums.  Register t of lane (r, h) is row 8 (t / 4) + 4 h + t % 4 of the tile, column r.
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int row = 32 * i + 8 * (t / 4) + 4 * h + t % 4;
        *reinterpret_cast<float*>(lds_raw + quarter * (kDsRows * kDsCols * 4) + row * (kDsCols * 4) + (half * 32 + r) * 4) =
            __builtin_ldexpf(__builtin_fmaf(rest[i][t], 1.f / kLowScale, sum[i][t]), 127 - scale);
      }
    if (h == 0) reinterpret_cast<float*>(lds_raw + kDsUnitOff)[quarter * kDsCols + half * 32 + r] = limit > 0.f ? __builtin_ldexpf(1.f, 127 - scale) : 0.f;
  } else {
    const int tail = k & ~15, tail_shift = tail == k ? 0 : 16 - (k & 15);
    const int sub = lane >> 4, l16 = lane & 15;
    constexpr int NR = kDsRows / (4 * kDsScatterWaves);                // rows of a lane group
    constexpr unsigned long long kFirst = 0x0001000100010001ull;       // the first lane of each group
    // (loads past the last entry give 0.  The range check is on the lane's offset, so all of it is there.)
    const auto column_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(column_indices), 0, nnz * 4, 0x00020000);
    const auto value_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(values), 0, nnz * 4, 0x00020000);
    const int first_row = (wave - kDsMulWaves) * (4 * NR);
    // In bytes: this lane's first entry from the cursor on; the row's end, less 64 for each further sixteen.
    int at[NR], row_end[NR][NC];
    unsigned row_base[NR];
    unsigned long long strays[NR];
    int cc[NR][NC];
    float aa[NR][NC];
    int scale[NR];
    float limit[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int local = first_row + 4 * j + sub, row = min(i0 + local, m);
      at[j] = (row_offsets[row] + l16) * 4;
#pragma unroll
      for (int e = 0; e < NC; ++e) row_end[j][e] = row_offsets[min(row + 1, m)] * 4 - 64 * e;
      row_base[j] = (unsigned)((local >> 5) * 512 + ((local & 31) << 4));
      strays[j] = 0;
      scale[j] = kNoScale;
      limit[j] = 0.f;
    }
    auto fetch = [&](int j) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < NC; ++e) cc[j][e] = (int)__builtin_amdgcn_raw_buffer_load_b32(column_rsrc, at[j] + 64 * e, 0, 0);
#pragma unroll
      for (int e = 0; e < NC; ++e)
        aa[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(value_rsrc, at[j] + 64 * e, 0, 0));
    };
    const int shift16 = 16 * (sub & 1);
    const bool upper = sub >= 2;
    unsigned last = 0;                                                 // the last column of the round before, in a group's first lane
    // The fetched entries of row j in the stage's columns; whether there may be more of them.  What is fetched is used up
    // before the next fetch, which then has the same registers: the compiler copies nothing, and so waits for nothing, before the next stage.
    auto round = [&](int j, char* block, int q, int x, bool again) __attribute__((always_inline)) -> bool {
      const int start = q * kDsS;
      unsigned long long mk[NC], over = 0;
      unsigned rel[NC];
      float v[NC];
      unsigned count = 0;
#pragma unroll
      for (int e = 0; e < NC; ++e) {
        rel[e] = (unsigned)(cc[j][e] - start);
        v[e] = aa[j][e];
        mk[e] = __builtin_amdgcn_ballot_w64(at[j] < row_end[j][e]) & __builtin_amdgcn_ballot_w64(rel[e] < (unsigned)kDsS);
        over |= mk[e] & __builtin_amdgcn_ballot_w64(__builtin_fabsf(v[e]) > limit[j]);
        unsigned mine = upper ? (unsigned)(mk[e] >> 32) : (unsigned)mk[e];
        mine = (mine >> shift16) & 0xffffu;
        asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(count) : "v"(mine), "v"(count));
        asm volatile("" : "+v"(rel[e]), "+v"(v[e]));
      }
      if (start + kDsS > tail) {
#pragma unroll
        for (int e = 0; e < NC; ++e) rel[e] += (int)rel[e] >= tail - start ? (unsigned)tail_shift : 0u;
      }
      at[j] += 4 * count;
      __builtin_amdgcn_sched_barrier(0);
      fetch(j);
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_expect(over != 0, 0)) {
        // A row's scale comes from the largest entry of the stage that first has one, and falls where a later one is above its
        // limit: the sums go down with it (row_shift).  Not in a further round of a stage, whose entries are in the block already: the
        // row is gathered then (unless all before were zeros).
        float largest = 0.f;
#pragma unroll
        for (int e = 0; e < NC; ++e)
          if (__builtin_amdgcn_inverse_ballot_w64(mk[e])) largest = fmaxf(largest, __builtin_fabsf(v[e]));
#pragma unroll
        for (int d = 1; d < 16; d *= 2) largest = fmaxf(largest, __shfl_xor(largest, d, kWave));
        const bool raise = largest > limit[j], fresh = limit[j] == 0.f;
        const int to = raise ? scale_for(largest) : scale[j];
        strays[j] |= __builtin_amdgcn_ballot_w64(raise && again && !fresh);
        if (raise && !again && l16 == 0) {
          row_shift[x * kDsRows + first_row + 4 * j + sub] = i32x2{q + 1, to - scale[j]};
          shifted[x] = q + 1;
        }
        scale[j] = to;
        if (raise) limit[j] = scale_limit(to);
      }
      const float times = __builtin_bit_cast(float, scale[j] << 23);
      // An ascending row's entry comes right after a smaller column of the same stage or is its first one.  (Rows with one that
      // does not: what was counted says nothing, they are gathered.)  Every entry of the stage is looked at, also behind a sixteen that has
      // none in any of the four rows: what is counted is written or gives its row away.  So `last` needs no look at where the row
      // ends: a row that is not given away has an entry of the stage in the next round's first place only if all of this round's are the stage's.
      const unsigned base = row_base[j] + (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)block;
#pragma unroll
      for (int e = 0; e < NC; ++e) {
        if (e > 0 && mk[e] == 0) continue;
        unsigned before;
        if (e == 0 && !again) {
          before = (unsigned)__builtin_amdgcn_mov_dpp((int)rel[e], 0x111, 0xf, 0xf, true);                                  // row_shr:1
        } else {
          const unsigned old = e == 0 ? last : (unsigned)__builtin_amdgcn_mov_dpp((int)rel[e - 1], 0x121, 0xf, 0xf, true);  // row_ror:1
          before = (unsigned)__builtin_amdgcn_update_dpp((int)old, (int)rel[e], 0x111, 0xf, 0xf, false);
        }
        unsigned long long wrong = __builtin_amdgcn_ballot_w64(before >= rel[e]);
        if (e == 0 && !again) wrong &= ~kFirst;
        strays[j] |= wrong & mk[e];
        if (__builtin_amdgcn_inverse_ballot_w64(mk[e])) {
          unsigned d;                                                  // the next column: two bytes on, eight columns: a group
          asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(d) : "v"(rel[e]), "s"(kDsGroup / 8), "v"(base));
          asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(rel[e] & 7u), "s"(2 - kDsGroup / 8), "v"(d));
          typedef __attribute__((address_space(3))) _Float16 LdsHalf;
          LdsHalf* const to = (LdsHalf*)(uintptr_t)d;
          const _Float16 y = (_Float16)(v[e] * times);
          to[0] = y;
          to[kDsPlane / 2] = (_Float16)(__builtin_fmaf(v[e], times, -(float)y) * kLowScale);
        }
      }
      const bool more = (mk[NC - 1] & (kFirst << 15)) != 0;
      if (more) last = (unsigned)__builtin_amdgcn_mov_dpp((int)rel[NC - 1], 0x121, 0xf, 0xf, true);
      return more;
    };
    // (ahead of the multiplying waves, which have the MFMA to wait for)
    __builtin_amdgcn_s_setprio(1);
    auto fill = [&](int q, int x) __attribute__((always_inline)) {
      char* block = lds_raw + x * kDsBuf;
#pragma unroll
      for (int j = 0; j < NR; ++j)
        if (round(j, block, q, x, false))
          while (round(j, block, q, x, true)) {}
    };
#pragma unroll
    for (int j = 0; j < NR; ++j) fetch(j);
    fill(0, 0);
    barrier();
    int x = 1;
    clocks.lap(kPhaseSetup);
    for (int q = 1; q < nst; ++q) {
      fill(q, x);
      x = x == 2 ? 0 : x + 1;
      clocks.lap(kPhaseScan);
      barrier();
      clocks.lap(kPhaseBarrier);
    }
    barrier();                                                         // the last stage's
    barrier();
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const unsigned long long mine = 0xffffull << (16 * sub);
      const int local = first_row + 4 * j + sub, row = min(i0 + local, m);
      const int entries = row_offsets[min(row + 1, m)] - row_offsets[row];
      if (l16 == 0) {
        redo[local] = at[j] != row_end[j][0] || (strays[j] & mine) != 0 || (entries > 0 && entries < kDsEntries);
        row_scale[local] = 127 - scale[j];
        reinterpret_cast<float*>(lds_raw + kDsFloorOff)[local] = limit[j] > 0.f ? scaled_floor(entries) : 0.f;
      }
    }
  }
  clocks.lap(kPhaseRest);
  clocks.store(blockIdx.x * (kDsMulWaves + kDsScatterWaves) + wave);
  barrier();
  // The four sums of each result; four columns to a thread.
  static_assert(kDsThreads * 4 == kDsRows * kDsCols, "a thread for every four results");
  const int local = tid >> 4, c4 = (tid & 15) * 4, row = i0 + local, col = tile * kDsCols + c4;
  float v[4] = {0.f, 0.f, 0.f, 0.f}, floor[4] = {0.f, 0.f, 0.f, 0.f}, scaled[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(lds_raw + w * (kDsRows * kDsCols * 4) + local * (kDsCols * 4) + c4 * 4);
    const f32x4 unit = *reinterpret_cast<const f32x4*>(lds_raw + kDsUnitOff + (w * kDsCols + c4) * 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v[t] += x[t];
      floor[t] = fmaxf(floor[t], unit[t]);
    }
  }
  const float row_floor = reinterpret_cast<const float*>(lds_raw + kDsFloorOff)[local];
  const int cols = min(4, n - col), count = row < m ? cols : 0;
  bool failed = redo[local] != 0, small = false;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    scaled[t] = v[t];
    small |= __builtin_fabsf(v[t]) < floor[t] * row_floor;
    v[t] = __builtin_ldexpf(v[t], row_scale[local]);
    failed |= split_failed(v[t]);
  }
  failed &= count > 0;
  small &= count > 0 && !failed;
  auto store = [&]() __attribute__((always_inline)) {
    if (count > 0) spmm_epilogue<float, 4>(v, bias, row, relu);
    float* c = C + (size_t)row * n + col;
    if (count >= 4) {
      Pack<float, 4>::store(c, v);
    } else {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t < count) c[t] = v[t];
    }
  };
  // The row's fours of columns to be gathered, those that are only small beside the floor sixteen bits up.
  auto note = [&]() __attribute__((always_inline)) {
    const unsigned long long fails = __builtin_amdgcn_ballot_w64(failed), smalls = __builtin_amdgcn_ballot_w64(small);
    if ((tid & 15) == 0) redo[local] = (int)((unsigned)(fails >> (lane & 48)) & 0xffffu | (unsigned)(smalls >> (lane & 48)) << 16);
  };
  note();
  if (!failed && !small) store();
  barrier();
  unsigned mask = (unsigned)redo[lane];
  if (__builtin_amdgcn_ballot_w64(mask != 0) == 0) return;
  int smalls = __builtin_popcount(mask >> 16);
#pragma unroll
  for (int d = 1; d < kWave; d *= 2) smalls += __shfl_xor(smalls, d, kWave);
  if (smalls >= kDsCount) {
    int* const lost = reinterpret_cast<int*>(lds_raw);                 // of the tile's columns.  (The products' sums have been read.)
    if (tid < kDsCols) lost[tid] = 0;
    barrier();
    int mine[4] = {0, 0, 0, 0};
    if (cols >= 4) {
#pragma unroll 16
      for (int p = local; p < k; p += kDsRows) {
        float b[4];
        Pack<float, 4>::load(B + (size_t)p * n + col, b);
#pragma unroll
        for (int t = 0; t < 4; ++t) mine[t] += scaled_loses(b[t], floor[t]);
      }
    } else {
      for (int p = local; p < k; p += kDsRows)
#pragma unroll
        for (int t = 0; t < 3; ++t)
          if (t < cols) mine[t] += scaled_loses(B[(size_t)p * n + col + t], floor[t]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      mine[t] += __shfl_xor(mine[t], 16, kWave);
      mine[t] += __shfl_xor(mine[t], 32, kWave);
      if (lane < 16 && mine[t] != 0) atomicAdd(&lost[c4 + t], mine[t]);
    }
    int of_row = 0;
    if (((unsigned)redo[local] >> 16) != 0) {
      const float unit = __builtin_ldexpf(1.f, row_scale[local]);
      const int end = row_offsets[row + 1];
#pragma unroll 8
      for (int p = row_offsets[row] + (tid & 15); p < end; p += 16) of_row += scaled_loses(values[p], unit);
    }
#pragma unroll
    for (int d = 1; d < 16; d *= 2) of_row += __shfl_xor(of_row, d, kWave);
    barrier();
    const bool was = small;
    small = false;
#pragma unroll
    for (int t = 0; t < 4; ++t)
      small |= __builtin_fabsf(scaled[t]) <                            // (a column of tiny numbers: a part of the sum may have been a denormal one)
               floor[t] * (floor[t] < 0x1p-76f ? row_floor : fminf(row_floor, scaled_floor(of_row + lost[c4 + t])));
    small &= was;
    note();
    if (was && !small) store();
    barrier();
    mask = (unsigned)redo[lane];
  }
  mask = (mask | mask >> 16) & 0xffffu;
  if (__builtin_amdgcn_ballot_w64(mask != 0) == 0) return;
  split_gather(mask, i0, tile * kDsCols, m, n, row_offsets, column_indices, values, B, C, bias, relu, lds_raw);
}

}  // namespace spdl
