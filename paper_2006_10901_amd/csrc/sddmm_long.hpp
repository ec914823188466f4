// SDDMM of dense sparse matrices on the matrix cores, fp32, long dot products: whole 64 x 256 blocks of L R^T from
// products of two fp16 terms per number (f16_split.hpp), of which the entries that A stores are kept.
//
// A workgroup owns 64 sparse rows and 256 columns of A and walks the dot product in chunks of 128.  Four waves split L: the chunk's 64
// rows come 16 bytes per lane, half a wave to a row, two chunks ahead, and their terms go to LDS in the order in which the lanes read
// them as MFMA operands, each row times a power of two that falls when a larger number comes.  Eight waves multiply: each brings in its
// own 32 rows of R (direct-to-LDS copies of 32 columns at a time, swizzled so that neither the copies nor the reads meet in a bank,
// asked for up to three pieces ahead), splits them in registers, one step of sixteen ahead, each row times a power of two of its own, and
// multiplies two 32 x 32 tiles; high high in one accumulator, high low and low high in another.  (Low low is below 2^-22 of the product.)
// A sum that is small beside what the largest numbers of its two rows could give may have lost what it consists of to the common powers of two
// (scaled_floor): as any result that is not finite it is computed again from L and R by the wave that stores it, unless there are many and
// a count shows that too few numbers have lost any (kLgCount).
// At a chunk's end what the two hold is added to the sums: the matrix cores cut sums off where they add, which a chain of the whole dot
// product would feel.  (2-norm of the error in 1e-8, n = 700 / 4096: normal numbers 12.1 / 15.3, slab kernel 13.2 / 29.3; both operands cut at zero, so that
// all products have one sign, 5.1 / 9.0, slab kernel 3.9 / 5.2.  Added every 64 columns 11.7 / 17.7 and 5.4 / 12.5, 4 % slower; every 256 13.4 / 15.2 and 6.1 /
// 6.9; every 512 15.7 / 17.5 and 9.4 / 6.5.)  The waves meet once a chunk, when its terms of L have been read and the next one's are there.  In the
// end the sums go to LDS, and all waves pick the stored entries of their rows.
//
// What bounds it: a SIMD has 12 MFMA of 32 clocks and 140 vector instructions for a step of sixteen columns, which take about
// their sum, 820 clocks at 1.6 GHz (the clock of a machine at its power limit): 4096 x 1024, n = 4096: 129 us whatever the density, without
// the splitting of R 24 us less, without its copies 15 less, without that of L 3 less.  64 x 256 because a tile more per wave (128 rows)
// has no registers left: 12 waves have 168 each.  Waves that wait for counts in LDS in place of meeting, chunks of 64 and operands asked for
// half a step earlier: 135 us.  The slab kernel: 1024 x 4096, n = 4096, at 10 % 136 us, here 130; 4096 x 1024, n = 2048,
// at 20 % 157 us, here 69.
#pragma once
#include "f16_split.hpp"

namespace spdl {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kLgRows = 64, kLgCols = 256;               // sparse rows and columns of A per workgroup
constexpr int kLgChunk = 128;                            // columns of the dot product per chunk
constexpr int kLgWaves = 8, kLgSplitWaves = 4;
constexpr int kLgThreads = 64 * (kLgWaves + kLgSplitWaves);
constexpr int kLgHalf = 512 + 16;                        // bytes of eight columns, one term, 32 rows: the next eight columns lie four banks on,
constexpr int kLgTile = 2 * kLgHalf;
constexpr int kLgStep = 4 * kLgTile + 160;               // ... the next sixteen eight: the 32 lanes that store a row's terms meet in no bank
constexpr int kLgBuf = kLgChunk / 16 * kLgStep;          // L high, L low, 64 rows
constexpr int kLgPiece = 32 * 32 * 4;                    // a wave's rows of R, 32 columns; two in its ring
constexpr int kLgRingOff = 2 * kLgBuf;
constexpr int kLgShiftOff = kLgRingOff + kLgWaves * 2 * kLgPiece;   // by how much the powers of two of the rows of L rise in a chunk (three chunks'),
constexpr int kLgRaisedOff = kLgShiftOff + 3 * kLgRows * 4;                // ... and whether they do, by the wave that splits them;
constexpr int kLgScaleOff = kLgRaisedOff + 3 * kLgSplitWaves * 4;          // RowScale of the rows of L
constexpr int kLgBoundOff = kLgScaleOff + kLgRows * 8;                     // the sparse rows' first and last entry in the block
constexpr int kLgLdsBytes = kLgBoundOff + 2 * kLgRows * 4;
constexpr int kLgStride = (kLgCols + 8) * 4;             // bytes from row to row of the results: four rows on, the other 32 banks
static_assert(kLgStep % 256 == 32 && kLgHalf % 256 == 16, "see above");
// Where the terms and the rings were, in the end: the scaled sums, RowScale of the rows of R, and how many of a wave's sums are small.
constexpr int kLgColOff = kLgRows * kLgStride, kLgSmallOff = kLgColOff + kLgCols * 8;
static_assert(kLgSmallOff + kLgWaves * 4 <= kLgShiftOff, "LDS");
// Stored sums that are small beside the floor of n products, by their share of the block's, from which on the numbers that lose bits (scaled_loses) are
// counted in the block's rows before what is still small beside the floor of as many products is computed again: as many rows are
// read as for this many sums.  (4096 x 1024 at 10 %, n = 4096, few numbers that are not zero, 110 us, 206 / 299 / 434 stored sums of a block zero:
// counted 260, not 328 / 400 / 511; at 20 %, n = 2048, 60 us, 589 / 1064: 150, 276 / 422.)
constexpr int kLgCount = 160;

// The exponent of what a scaled one of a row of L or R is, and in how many of its numbers bits may have been lost to the common power of two: all
// n until they are counted; -infinity where all are zeros, whose sums are right whatever the other row holds.
struct RowScale { int unit; float lost; };

// (n > 32, k >= 32, 0 < nnz < 2^29, n < 2^21.)
__global__ __launch_bounds__(kLgThreads) void sddmm_long_kernel(
    int m, int k, int n, int nnz, int panels, int parts, int share_r, const int* __restrict__ row_offsets, const int* __restrict__ column_indices,
    const float* __restrict__ L, const float* __restrict__ R, float* __restrict__ out, const float* __restrict__ scale) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  int panel, part;
  if (!(share_r ? slab_wg_map(blockIdx.x, parts, panels, part, panel) : slab_wg_map(blockIdx.x, panels, parts, panel, part)))
    return;                                                            // whole workgroup, before any barrier
  const int i0 = panel * kLgRows, c0 = part * kLgCols;
  const int chunks = (n + kLgChunk - 1) / kLgChunk;
  PhaseClocks clocks;
  clocks.start();
  int* const row_shift = reinterpret_cast<int*>(lds_raw + kLgShiftOff);
  int* const row_raised = reinterpret_cast<int*>(lds_raw + kLgRaisedOff);
  RowScale* const of_row = reinterpret_cast<RowScale*>(lds_raw + kLgScaleOff);
  RowScale* const of_col = reinterpret_cast<RowScale*>(lds_raw + kLgColOff);
  int* const small_sums = reinterpret_cast<int*>(lds_raw + kLgSmallOff);
  int* const bounds = reinterpret_cast<int*>(lds_raw + kLgBoundOff);
  auto barrier = [&]() __attribute__((always_inline)) {                // (no wait for memory)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  auto window_of = [&](int begin, int end, int key) __attribute__((always_inline)) {
    const int guess = begin + (int)((float)(end - begin) * ((float)key / (float)k)) - kWave / 2;
    return max(begin, min(guess, end - kWave));
  };

  if (wave < kLgWaves) {
    const int r = lane & 31, h = lane >> 5;
    // Copy i of a piece (32 columns) fills slots 64 i .. of one half of the wave's ring: slot 8 row + (four of columns xor (row / 2) % 8).
    char* const ring = lds_raw + kLgRingOff + wave * (2 * kLgPiece);
    const unsigned ring_m0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)ring;
    const int row0 = min(c0 + 32 * wave, k - 32);                      // (past k: the last ones again)
    const float* const rows = R + (size_t)row0 * n;
    const int pieces = chunks * (kLgChunk / 32);
    unsigned row_off[2];                                               // (of copies 0 and 2, 1 and 3: rows 8 apart, the columns exchanged)
    const int four = 4 * ((lane & 7) ^ ((lane >> 4) & 3));
#pragma unroll
    for (int i = 0; i < 2; ++i) row_off[i] = (unsigned)(8 * i + (lane >> 3)) * (unsigned)n * 4u + 4u * (four ^ (16 * i));
    auto copy = [](unsigned to, unsigned off, const float* from) __attribute__((always_inline)) {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(to), "v"(off), "s"(from) : "memory", "m0");
    };
    auto bring = [&](int piece) __attribute__((always_inline)) {
      const unsigned to = ring_m0 + (unsigned)((piece & 1) * kLgPiece);
      if (32 * piece + 32 <= n) {
#pragma unroll
        for (int i = 0; i < 4; ++i) copy(to + i * 1024, row_off[i & 1], rows + 32 * piece + (size_t)(i >> 1) * 16 * n);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int mine = four ^ (16 * (i & 1));
          int col = min(piece, pieces - 1) * 32 + mine;                // (past the end: the last one again, not used)
          col = col < n ? piece_start(col, n, 4) : 0;                  // (columns past the dot product: L has zeros there)
          copy(to + i * 1024, row_off[i & 1] + 4u * (unsigned)(col - mine), rows + (size_t)(i >> 1) * 16 * n);
        }
      }
    };
    bring(0);
    bring(1);
    // The block's entries of this wave's eight sparse rows: the first ones with column c0 or more, and c0 + 256 (some fixed place in rows
    // that are not ascending).  64 neighbouring entries around the place that evenly spread columns would give, all
    // bounds at a time; if a bound is not among them, by halves.  Lane l < 8 looks after the start of row l, lane 8 + l after its end.
    {
      constexpr int NR = kLgRows / kLgWaves;
      const int row = i0 + NR * wave + (lane & (NR - 1));
      const int row_begin = row_offsets[min(row, m)], row_end = row_offsets[min(row + 1, m)];
      const bool is_end = (lane & NR) != 0;
      const int key = c0 + (is_end ? kLgCols : 0), window = window_of(row_begin, row_end, key);
      int probe[2 * NR], below = 0;
#pragma unroll
      for (int i = 0; i < 2 * NR; ++i)
        probe[i] = column_indices[max(0, min(__builtin_amdgcn_readlane(window, i) + lane, nnz - 1))];
#pragma unroll
      for (int i = 0; i < 2 * NR; ++i) {
        const unsigned long long less = __builtin_amdgcn_ballot_w64(lane < __builtin_amdgcn_readlane(row_end - window, i) &&
                                                                    probe[i] < c0 + (i >= NR ? kLgCols : 0));
        below = lane == i ? (less == ~0ull ? 64 : __builtin_ctzll(~less)) : below;
      }
      int lo = window + below, hi = lo;
      if (below == 0 && window > row_begin) lo = row_begin;
      if (below == 64) hi = row_end;
      if (lane >= 2 * NR) hi = lo;
      while (__builtin_amdgcn_ballot_w64(lo < hi) != 0) {
        if (lo < hi) {
          const int mid = (int)(((unsigned)lo + (unsigned)hi) >> 1);
          if (column_indices[mid] < key) lo = mid + 1; else hi = mid;
        }
      }
      if (part == 0 && !is_end) lo = row_begin;
      if (part == parts - 1 && is_end) lo = row_end;
      if (lane < 2 * NR) bounds[2 * (NR * wave + (lane & (NR - 1))) + (is_end ? 1 : 0)] = lo;
    }
    // A lane's operand of step j, term t, tile i, eight columns of row 32 i + r.
    const char* const left = lds_raw + h * kLgHalf + r * 16;
    f16x8 high[2], low[2];
    auto load_left = [&](f16x8 (&x)[2], int at) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = *reinterpret_cast<const f16x8*>(left + at + i * kLgTile);
    };
    float raw[2][8];
    auto fetch = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(ring + slot * kLgPiece + (8 * r + ((4 * j + 2 * h + half) ^ ((r >> 1) & 7))) * 16);
#pragma unroll
          for (int t = 0; t < 4; ++t) raw[j][4 * half + t] = x[t];
        }
    };
    // The largest number that the power of two in use of the lane's row of R is for, and by how much that has just risen.  (All zeros so far: 0, and
    // what these are taken times does not matter.)
    float limit = 0.f;
    int shift = 0;
    unsigned long long raised = 0;
    struct Terms { f16x8 high, low; };
    auto split = [&](const float (&v)[8]) __attribute__((always_inline)) -> Terms {
      float largest, other, both;
      asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(largest) : "v"(v[0]), "v"(v[1]), "v"(v[2]));
      asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(other) : "v"(v[3]), "v"(v[4]), "v"(v[5]));
      asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(both) : "v"(largest), "v"(v[6]), "v"(v[7]));
      asm("v_max_f32 %0, %1, %2" : "=v"(largest) : "v"(both), "v"(other));
      raised = __builtin_amdgcn_ballot_w64(largest > limit);
      if (__builtin_expect(raised != 0, 0)) {
        largest = max_of_halves(largest);                              // (the row's other eight columns)
        const float to = largest > limit ? scale_limit(scale_for(largest)) : limit;
        shift = (int)(__builtin_bit_cast(unsigned, limit) - __builtin_bit_cast(unsigned, to)) >> 23;
        limit = to;
      }
      const float times = __builtin_bit_cast(float, (269u << 23) - __builtin_bit_cast(unsigned, limit));
      Terms t;
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        f16x2 x, y;
        split_f16(v[e], v[e + 1], times, x, y);
        t.high[e] = x[0]; t.high[e + 1] = x[1];
        t.low[e] = y[0]; t.low[e + 1] = y[1];
      }
      return t;
    };
    acc32x32 total[2], sum[2], rest[2];
    acc32x32 zero;
#pragma unroll
    for (int t = 0; t < 16; ++t) zero[t] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) total[i] = sum[i] = rest[i] = zero;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    fetch(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bring(2);
    Terms b = split(raw[0]);
    clocks.lap(kPhaseSetup);
    barrier();                                                         // the first chunk's terms of L are there
    clocks.lap(kPhaseBarrier);
    load_left(low, 2 * kLgTile);
    load_left(high, 0);
    for (int q = 0; q < chunks; ++q) {
      const int buf = (q & 1) * kLgBuf, table = q % 3;
#pragma unroll
      for (int j = 0; j < kLgChunk / 16; ++j) {
        const bool first_step = j == 0, last_step = j == kLgChunk / 16 - 1, next_piece = (j & 1) != 0;
        const int next = last_step ? kLgBuf - buf : buf + (j + 1) * kLgStep;
        const int piece = q * (kLgChunk / 32) + (j >> 1);
        i32x4 rose;
        if (next_piece) {
          asm volatile("s_waitcnt vmcnt(4)" ::: "memory");             // (the piece after the next one may still be on its way)
          fetch((piece + 1) & 1);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) rest[i] = mfma_f16(low[i], b.high, first_step ? zero : rest[i]);
        __builtin_amdgcn_sched_barrier(0);
        if (last_step) {
          clocks.lap(kPhaseSteps);
          barrier();                                                   // this chunk's terms may be written over; the next one's are there
          clocks.lap(kPhaseBarrier);
        }
        load_left(low, next + 2 * kLgTile);                            // (past the last chunk: read, not used)
        if (j == 0) rose = *reinterpret_cast<const i32x4*>(row_raised + 4 * table);
        __builtin_amdgcn_sched_barrier(0);
        if (next_piece) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // (the piece has been read)
          bring(piece + 3);
        }
        __builtin_amdgcn_sched_barrier(0);
        const Terms c = split(raw[next_piece ? 0 : 1]);
#pragma unroll
        for (int i = 0; i < 2; ++i) rest[i] = mfma_f16(high[i], b.low, rest[i]);
#pragma unroll
        for (int i = 0; i < 2; ++i) sum[i] = mfma_f16(high[i], b.high, first_step ? zero : sum[i]);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_left(high, next);
        if (j == 0 && __builtin_expect((uniform(rose[0]) | uniform(rose[1]) | uniform(rose[2]) | uniform(rose[3])) != 0, 0)) {
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 16; ++t)                               // (register t of lane (r, h) is row 8 (t / 4) + 4 h + t % 4 of a tile, column r)
              if (rose[2 * i + t / 8] != 0) total[i][t] = __builtin_ldexpf(total[i][t], row_shift[table * kLgRows + 32 * i + 8 * (t / 4) + 4 * h + t % 4]);
        }
        if (last_step) {
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 16; ++t) total[i][t] += __builtin_fmaf(rest[i][t], 1.f / kLowScale, sum[i][t]);
        }
        if (__builtin_expect(raised != 0, 0)) {
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 16; ++t) {
              total[i][t] = __builtin_ldexpf(total[i][t], shift);
              sum[i][t] = __builtin_ldexpf(sum[i][t], shift);
              rest[i][t] = __builtin_ldexpf(rest[i][t], shift);
            }
        }
        b = c;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    clocks.lap(kPhaseSteps);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // (what was asked for past the end)
    barrier();                                                         // nobody reads terms or rings any more
    const int column = row0 - c0 + r;
    const RowScale mine = {(int)(__builtin_bit_cast(unsigned, limit) >> 23) - 142, limit > 0.f ? (float)n : -__builtin_inff()};
    const float floor = limit > 0.f ? scaled_floor(n) : 0.f;
    unsigned long long small = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < 16; ++t) small |= __builtin_amdgcn_ballot_w64(__builtin_fabsf(total[i][t]) < floor);
    int smalls = 0;
    if (small != 0) {                                                  // (rows of zeros need no look)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 16; ++t)
          smalls += __builtin_popcountll(__builtin_amdgcn_ballot_w64(__builtin_fabsf(total[i][t]) < floor && of_row[32 * i + 8 * (t / 4) + 4 * h + t % 4].lost > 0.f));
    }
    if (lane == 0) small_sums[wave] = smalls;
    if (column >= 0) {
      if (h == 0) of_col[column] = mine;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 16; ++t)
          *reinterpret_cast<float*>(lds_raw + (32 * i + 8 * (t / 4) + 4 * h + t % 4) * kLgStride + column * 4) = total[i][t];
    }
  } else {
    constexpr int NI = kLgRows / kLgSplitWaves / 2;                    // pairs of rows
    const int first = (kLgRows / kLgSplitWaves) * (wave - kLgWaves), half = lane >> 5, l32 = lane & 31;
    const int rows_here = min(kLgRows, m - i0);                        // (rows past the end come as zeros)
    const auto source = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(L + (size_t)i0 * n), 0, rows_here * n * 4, 0x00020000);
    const int off = (first + half) * n * 4 + 16 * l32, two_rows = 8 * n;
    f32x4 raw[2][NI];
    // Pieces that reach past the dot product start at n - 4; columns that are the lane before's, or nobody's, are zeros.
    auto fetch = [&](f32x4 (&to)[NI], int q) __attribute__((always_inline)) {
      int at = off + q * (kLgChunk * 4);
      if ((q + 1) * kLgChunk > n) {
        const int col = q * kLgChunk + 4 * l32;
        at += 4 * ((col < n ? piece_start(col, n, 4) : 0) - col);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
        to[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(source, at + i * two_rows, 0, 0));
    };
    // (columns 4 l32 ..: step l32 / 4, eight (l32 / 2) % 2 of it)
    char* const block = lds_raw + (l32 >> 2) * kLgStep + (first >> 5) * kLgTile + ((l32 >> 1) & 1) * kLgHalf + ((first & 31) + half) * 16 + (l32 & 1) * 8;
    int power[NI];                                                     // the exponents of the powers of two that rows are taken times,
    float limit[NI];                                                   // ... up to which numbers
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      power[i] = kNoScale;
      limit[i] = 0.f;
    }
    auto convert = [&](f32x4 (&x)[NI], int q) __attribute__((always_inline)) {
      if ((q + 1) * kLgChunk > n) {
        const int col = q * kLgChunk + 4 * l32, from = col < n ? piece_start(col, n, 4) : 0;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int t = 0; t < 4; ++t) x[i][t] = col < n && from + t >= col ? x[i][t] : 0.f;
      }
      float largest[NI];
      unsigned long long above = 0;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        largest[i] = fmaxf(fmaxf(__builtin_fabsf(x[i][0]), __builtin_fabsf(x[i][1])), fmaxf(__builtin_fabsf(x[i][2]), __builtin_fabsf(x[i][3])));
        above |= __builtin_amdgcn_ballot_w64(largest[i] > limit[i]);
      }
      if (__builtin_expect(above != 0, 0)) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float most = largest[i];
#pragma unroll
          for (int d = 1; d < 32; d *= 2) most = fmaxf(most, __shfl_xor(most, d, kWave));
          const int to = most > limit[i] ? scale_for(most) : power[i];
          if (l32 == 0) row_shift[q % 3 * kLgRows + first + 2 * i + half] = to - power[i];
          limit[i] = most > limit[i] ? scale_limit(to) : limit[i];
          power[i] = to;
        }
      }
      if (lane == 0) row_raised[q % 3 * kLgSplitWaves + wave - kLgWaves] = above != 0;
      char* const to = block + (q & 1) * kLgBuf;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const float times = __builtin_bit_cast(float, power[i] << 23);
        f16x4 high, low;
#pragma unroll
        for (int t = 0; t < 4; t += 2) {
          f16x2 a, b;
          split_f16(x[i][t], x[i][t + 1], times, a, b);
          high[t] = a[0]; high[t + 1] = a[1];
          low[t] = b[0]; low[t + 1] = b[1];
        }
        *reinterpret_cast<f16x4*>(to + i * 32) = high;
        *reinterpret_cast<f16x4*>(to + i * 32 + 2 * kLgTile) = low;
      }
    };
    fetch(raw[0], 0);
    if (chunks > 1) fetch(raw[1], 1);
    convert(raw[0], 0);
    if (chunks > 2) fetch(raw[0], 2);
    clocks.lap(kPhaseSetup);
    barrier();
    for (int q = 0; q < chunks; q += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (q + u < chunks) {                                          // while chunk q + u is multiplied: the next one
          if (q + u + 1 < chunks) convert(raw[~u & 1], q + u + 1);
          if (q + u + 3 < chunks) fetch(raw[~u & 1], q + u + 3);
          clocks.lap(kPhaseScan);
          barrier();
          clocks.lap(kPhaseBarrier);
        }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (l32 == 0) of_row[first + 2 * i + half] = {127 - power[i], limit[i] > 0.f ? (float)n : -__builtin_inff()};
    barrier();
  }
  // Every wave picks the entries of five or six rows.
  constexpr int NW = kLgWaves + kLgSplitWaves, NP = (kLgRows + NW - 1) / NW;
  int cursor[NP], index[NP];
  auto columns_at = [&](int p) __attribute__((always_inline)) { return column_indices[min(p + lane, nnz - 1)]; };
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    cursor[i] = uniform(bounds[2 * min(wave + NW * i, kLgRows - 1)]);
    index[i] = columns_at(cursor[i]);
  }
  clocks.lap(kPhaseRest);
  barrier();                                                           // the sums are there
  int smalls = 0;
#pragma unroll
  for (int i = 0; i < kLgWaves; ++i) smalls += small_sums[i];
  if (uniform(smalls) > 0) {
    int entries = max(0, bounds[2 * lane + 1] - bounds[2 * lane]);
#pragma unroll
    for (int d = 1; d < kWave; d *= 2) entries += __shfl_xor(entries, d, kWave);
    // (of the block's sums, as many as are stored if these are as small as the others)
    if (uniform((int)((float)smalls * (float)entries * (1.f / (kLgRows * kLgCols)))) >= kLgCount) {
      for (int x = wave; x < kLgRows + kLgCols; x += NW) {
        const bool left = x < kLgRows;
        const int row = left ? i0 + x : c0 + x - kLgRows;
        if (row >= (left ? m : k)) continue;
        RowScale* const of = left ? of_row + x : of_col + x - kLgRows;
        if (uniform((int)(of->lost > 0.f)) == 0) continue;
        const float unit = __builtin_ldexpf(1.f, of->unit);
        const float* const from = (left ? L : R) + (size_t)row * n;
        int lost = 0, j = 4 * lane;
#pragma unroll 8
        for (; j + 4 <= n; j += 4 * kWave) {
          const f32x4 v = *reinterpret_cast<const f32x4_any*>(from + j);
#pragma unroll
          for (int t = 0; t < 4; ++t) lost += scaled_loses(v[t], unit);
        }
        for (; j < n; ++j) lost += scaled_loses(from[j], unit);
#pragma unroll
        for (int d = 1; d < kWave; d *= 2) lost += __shfl_xor(lost, d, kWave);
        if (lane == 0) of->lost = (float)lost;
      }
      barrier();
    }
  }
  // A dot product by the whole wave: what the matrix cores cannot give.  (4096 x 1024 at 10 %, n = 4096, 130 us without any: a row of NaN's worth 250,
  // all results 1360, at the L2s' rate; sums below scaled_floor, 149 us from the same generator: +-1 on both sides 152, log-normal, sigma 1 / 3, 150 / 181,
  // columns 2^20 times the others and zeros 390; one number in a hundred on both sides not zero 272, one in a row 293: 977 and 1372 with nothing counted.)
  auto dot = [&](int row, int column) __attribute__((always_inline)) {
    const float* const l = L + (size_t)(i0 + row) * n;
    const float* const r = R + (size_t)column * n;
    float acc = 0.f;
    int j = 4 * lane;
#pragma unroll 4
    for (; j + 4 <= n; j += 4 * kWave) {
      const f32x4_any x = *reinterpret_cast<const f32x4_any*>(l + j), y = *reinterpret_cast<const f32x4_any*>(r + j);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc = __builtin_fmaf(x[t], y[t], acc);
    }
    for (; j < n; ++j) acc = __builtin_fmaf(l[j], r[j], acc);
#pragma unroll
    for (int d = 1; d < kWave; d *= 2) acc += __shfl_xor(acc, d, kWave);
    return acc;
  };
  unsigned rows_left = 0;
  int stopped = 0;                                                     // lane i: the cursor of row i
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int row = wave + NW * i;
    if (row >= kLgRows) break;
    const int end = uniform(bounds[2 * row + 1]);
    int at = cursor[i];
    int column = index[i];
    const RowScale left = of_row[row];
    while (at < end) {
      const unsigned rel = (unsigned)(column - c0);
      const unsigned long long in = __builtin_amdgcn_ballot_w64(rel < (unsigned)kLgCols) & __builtin_amdgcn_ballot_w64(lane < end - at);
      const int count = in == ~0ull ? 64 : __builtin_ctzll(~in);       // from the first one on without a gap
      const int inside = min(rel, (unsigned)kLgCols - 1);
      const float sum = *reinterpret_cast<const float*>(lds_raw + row * kLgStride + inside * 4);
      const RowScale right = of_col[inside];
      const float v = __builtin_ldexpf(sum, left.unit + right.unit);
      // (sum below scaled_floor of as many products as may be off)
      const bool again = sum * sum < fminf((float)n, left.lost + right.lost) || split_failed(v);
      if (lane < count && !again) sddmm_store<float>(out, scale, at + lane, v);
      unsigned long long fails = __builtin_amdgcn_ballot_w64(lane < count && again);
      for (; fails != 0; fails &= fails - 1) {
        const int e = __builtin_ctzll(fails);
        const float result = dot(row, __builtin_amdgcn_readlane(column, e));
        if (lane == 0) sddmm_store<float>(out, scale, at + e, result);
      }
      at += count;
      if (count < 64) break;
      column = columns_at(at);
    }
    rows_left |= (unsigned)(at < end) << i;
    stopped = lane == i ? at : stopped;
  }
  clocks.lap(kPhaseGather);
  clocks.store(blockIdx.x * NW + wave);
  // What is left of rows that are not ascending.  The ranges that the parts of such a row find may overlap: an entry is its column's part's wherever
  // that part's range holds it, so that the bits do not depend on which workgroup stores last.
  auto bound_of = [&](int begin, int end, int i) __attribute__((always_inline)) {      // as the parts have found them
    const int key = i * kLgCols, window = window_of(begin, end, key);
    const int probe = column_indices[max(0, min(window + lane, nnz - 1))];
    const unsigned long long less = __builtin_amdgcn_ballot_w64(lane < end - window && probe < key);
    const int below = less == ~0ull ? 64 : __builtin_ctzll(~less);
    int lo = window + below, hi = lo;
    if (below == 0 && window > begin) lo = begin;
    if (below == 64) hi = end;
    while (lo < hi) {
      const int mid = (int)(((unsigned)lo + (unsigned)hi) >> 1);
      if (column_indices[mid] < key) lo = mid + 1; else hi = mid;
    }
    return i == 0 ? begin : i == parts ? end : lo;
  };
  for (; rows_left != 0; rows_left &= rows_left - 1) {
    const int i = __builtin_ctz(rows_left), row = wave + NW * i;
    const int begin = uniform(row_offsets[i0 + row]), end = uniform(row_offsets[i0 + row + 1]);
    const int to = uniform(bounds[2 * row + 1]);
    for (int p = __builtin_amdgcn_readlane(stopped, i); p < to; ++p) {
      const int column = uniform(column_indices[p]), home = column / kLgCols;
      if (home != part && p >= uniform(bound_of(begin, end, home)) && p < uniform(bound_of(begin, end, home + 1))) continue;
      const float result = dot(row, column);
      if (lane == 0) sddmm_store<float>(out, scale, p, result);
    }
  }
}

}  // namespace spdl
