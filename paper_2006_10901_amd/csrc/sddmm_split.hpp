// SDDMM of dense sparse matrices on the matrix cores, fp32, dot products of up to 128 columns: whole 64 x 256 blocks of
// L R^T from three-term bf16 products (bf16_split.hpp), of which the entries that A stores are kept.
//
// A workgroup owns 64 sparse rows and a run of steps of 256 columns of A.  Eight waves multiply: the 64 rows of L are
// split into their terms once and stay in LDS, in the order in which the lanes read them as MFMA operands; in a step
// each wave brings in its own 32 rows of R (direct-to-LDS copies of 32 columns at a time, 4 KB, swizzled so
// that neither the copies nor the reads meet in a bank), splits them in registers and multiplies two 32 x 32 tiles:
// twelve MFMA for the 48 vector instructions that split the next sixteen columns, one for four in turn.  The waves share
// nothing up to here, so they wait for nothing.  The block of results then goes to LDS, and four (eight) more waves, on each
// SIMD one (two), pick the stored entries of sixteen (eight) rows each out of it while the others are at the next step: 64 consecutive
// entries of a row at a time, whose column indices were requested a step before.  (Waves that did both waited for
// their stores wherever they waited for a copy.)
//
// What bounds it: at 97 .. 128 columns power.  The multiplying waves keep the matrix cores busy for their part of a step
// (6100 clocks of the 6144 that 2 x 96 MFMA take; 63 % of the whole), the clock falls to 1.5 GHz, and the MFMA alone, with reads
// of L and the splitting, take 104 us in a loop of nothing else.  At up to 64 columns the picking, some 3000 clocks a step.
// 8192 x 10240 at 20 %, 32 / 64 / 96 / 128 columns: 51 / 76 / 98 / 118 us, slab and lane kernels 109 / 109 / 135 / 139; 128 columns
// at 30 %: 128 against 192; at 10 %, 115 against 84, which is why the density decides.  3004 x 2251 at 15 %, 75 columns: 13.2
// against 17.1.
//
// A row's entries are met in stored order by a cursor; entries that the cursor has not passed at the end (rows that
// are not ascending) and results that are not finite are dot products of their own.  The ranges that the parts of such a row
// find may overlap: an entry is its column's part's wherever that part's range holds it, so that the bits do not depend
// on which workgroup stores last.
#pragma once
#include "bf16_split.hpp"

namespace spdl {

constexpr int kSpRows = 64;                              // sparse rows per workgroup
constexpr int kSpCols = 256;                             // columns of A per step, 32 for each multiplying wave
constexpr int kSpWaves = 8;                              // multiplying waves
constexpr int kSpChunk = 32;                             // columns of the dot product per copy
constexpr int kSpStride = (kSpCols + 8) * 4;             // bytes from row to row of the block: four rows on, the other 32 banks
constexpr int kSpBlockBytes = kSpRows * kSpStride;
constexpr int kSpRingBytes = 32 * kSpChunk * 4;          // a wave's rows of R, one chunk
__host__ __device__ __forceinline__ constexpr int sddmm_split_lds_bytes(int ksteps) {
  return (ksteps + 1) / 2 * 12288 + kSpBlockBytes + kSpWaves * kSpRingBytes;
}

// KSTEPS sixteens of columns; AHEAD sixty-fours of a row's entries requested a step ahead.
template <int KSTEPS, int AHEAD, int PICKERS, bool SCALED>
__global__ __launch_bounds__(64 * (kSpWaves + PICKERS)) void sddmm_split_kernel(
    int m, int k, int n, int nnz, int parts, int steps_per_part, const int* __restrict__ row_offsets,
    const int* __restrict__ column_indices, const float* __restrict__ L, const float* __restrict__ R,
    float* __restrict__ out, const float* __restrict__ scale) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int CHUNKS = (KSTEPS + 1) / 2;
  char* const lfrag = lds_raw;
  char* const block = lds_raw + CHUNKS * 12288;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);

  // Workgroup -> (panel, part): each XCD (consecutive ids go round them) gets a run, one part's panels after the other,
  // so that its L2 holds the rows of R that its workgroups stream.
  const int panels = (m + kSpRows - 1) / kSpRows, total = panels * parts;
  const int eighth = (total + 7) >> 3, pos = (blockIdx.x & 7) * eighth + (int)(blockIdx.x >> 3);
  if (pos >= total || (int)(blockIdx.x >> 3) >= eighth) return;        // whole workgroup, before any barrier
  const int part = pos / panels, i0 = (pos - part * panels) * kSpRows;
  const int step0 = part * steps_per_part, step1 = min((k + kSpCols - 1) / kSpCols, step0 + steps_per_part);
  PhaseClocks clocks;
  clocks.start();
  auto barrier = [&]() __attribute__((always_inline)) {                // (no wait for memory)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  if (wave < kSpWaves) {
    const int r = lane & 31, h = lane >> 5;
    char* const ring = block + kSpBlockBytes + wave * kSpRingBytes;
    // Copy q of a chunk fills slots 64 q .. of the wave's ring: slot 8 row + (piece xor (row / 2) % 8).
    const unsigned ring_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)ring;
    auto issue = [&](int step, int chunk) __attribute__((always_inline)) {
      const int row0 = min(step * kSpCols + wave * 32, k - 1);         // (a tile past k copies the last row)
      const char* base = reinterpret_cast<const char*>(R + (size_t)row0 * n);
      const int last = k - 1 - row0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 8 * q + (lane >> 3);
        int col = chunk * kSpChunk + 4 * ((lane & 7) ^ ((row >> 1) & 7));
        col = col < n ? piece_start(col, n, 4) : 0;                    // pieces past the end: L has zeros there
        const unsigned off = ((unsigned)min(row, last) * (unsigned)n + (unsigned)col) * 4u;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(ring_lds + (unsigned)q * 1024u), "v"(off), "s"(base) : "memory", "m0");
      }
    };
    // the chunk after (step, chunk), wherever it is
    auto issue_after = [&](int step, int chunk) __attribute__((always_inline)) {
      if (chunk + 1 < CHUNKS) issue(step, chunk + 1);
      else if (step + 1 < step1) issue(step + 1, 0);
    };
    issue(step0, 0);

    // L: a lane's operand of step j, term t, tile i is 16 bytes at ((3 j + t) * 2 + i) * 1024 + 16 lane.
    for (int task = tid; task < kSpRows * CHUNKS * 4; task += 64 * kSpWaves) {
      const int lrow = task & 63, eight = task >> 6;                   // columns 8 eight .. + 7
      const float* src = L + (size_t)min(i0 + lrow, m - 1) * n;
      float v[8];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int col = 8 * eight + 4 * half;
        const int from = col < n ? piece_start(col, n, 4) : 0;
        float x[4];
        Pack<float, 4>::load(src + from, x);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[4 * half + t] = col < n && from + t >= col ? x[t] : 0.f;
      }
      const Split8 s = split8(v);
      char* dst = lfrag + ((eight >> 1) * 6 + (lrow >> 5)) * 1024 + ((eight & 1) * 32 + (lrow & 31)) * 16;
      *reinterpret_cast<bf16x8*>(dst) = s.high;
      *reinterpret_cast<bf16x8*>(dst + 2048) = s.mid;
      *reinterpret_cast<bf16x8*>(dst + 4096) = s.low;
    }

    float raw[2][8];
    auto arrived = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    auto fetch = [&]() __attribute__((always_inline)) {                // the ring's chunk, once it has arrived
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int piece = 4 * j + 2 * h + half;
          const f32x4 x = *reinterpret_cast<const f32x4*>(ring + (8 * r + (piece ^ ((r >> 1) & 7))) * 16);
#pragma unroll
          for (int t = 0; t < 4; ++t) raw[j][4 * half + t] = x[t];
        }
    };
    auto fetched = [&]() __attribute__((always_inline)) {              // read, so that the ring can be written again
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    arrived();
    barrier();                                                         // the terms of L are there
    fetch();
    fetched();
    issue_after(step0, 0);
    Split8 b = split8(raw[0]);                                         // the terms of the next sixteen columns of R
    clocks.lap(kPhaseSetup);

    for (int step = step0; step < step1; ++step) {
      acc32x32 sum[2], rest[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 16; ++t) sum[i][t] = rest[i][t] = 0.f;
#pragma unroll
      for (int j = 0; j < KSTEPS; ++j) {
        const bool next_chunk = (j & 1) || j + 1 == KSTEPS;            // what comes after is in the ring, not in `raw`
        const Split8 now = b;
        const char* a = lfrag + j * 6144 + lane * 16;
        bf16x8 ah[2], am[2], al[2];
        __builtin_amdgcn_sched_barrier(0);
        if (next_chunk) {
          arrived();
          fetch();
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          ah[i] = *reinterpret_cast<const bf16x8*>(a + i * 1024);
          al[i] = *reinterpret_cast<const bf16x8*>(a + i * 1024 + 4096);
          am[i] = *reinterpret_cast<const bf16x8*>(a + i * 1024 + 2048);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) sum[i] = mfma_bf16(ah[i], now.high, sum[i]);
#pragma unroll
        for (int i = 0; i < 2; ++i) rest[i] = mfma_bf16(ah[i], now.low, rest[i]);
        if (next_chunk) {
          __builtin_amdgcn_sched_barrier(0);
          fetched();
          issue_after(j + 1 < KSTEPS ? step : step + 1, j + 1 < KSTEPS ? (j >> 1) + 1 : 0);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) rest[i] = mfma_bf16(al[i], now.high, rest[i]);
#pragma unroll
        for (int i = 0; i < 2; ++i) rest[i] = mfma_bf16(am[i], now.mid, rest[i]);
#pragma unroll
        for (int i = 0; i < 2; ++i) rest[i] = mfma_bf16(ah[i], now.mid, rest[i]);
#pragma unroll
        for (int i = 0; i < 2; ++i) rest[i] = mfma_bf16(am[i], now.high, rest[i]);
        b = split8(raw[next_chunk ? 0 : 1]);
        if (!next_chunk) {
          __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
          for (int g = 0; g < 12; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
          }
        } else {
#pragma unroll
          for (int g = 0; g < 8; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, 6, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      clocks.lap(kPhaseSteps);
      barrier();                                                       // the entries of the block before have been picked
      clocks.lap(kPhaseBarrier);
      // Register t of lane (r, h) is row 8 (t / 4) + 4 h + t % 4 of the tile, column r.
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        char* rows = block + (32 * i + 4 * h) * kSpStride + (32 * wave + r) * 4;
#pragma unroll
        for (int t = 0; t < 16; ++t)
          *reinterpret_cast<float*>(rows + (8 * (t / 4) + t % 4) * kSpStride) = sum[i][t] + rest[i][t];
      }
      clocks.lap(kPhaseRest);
      barrier();
      clocks.lap(kPhaseBarrier);
    }
  } else {
    // Lane l < NR looks after row l of this wave's: the start of the part's range; lane NR + l after its end.
    constexpr int NR = kSpRows / PICKERS;
    static_assert(2 * NR <= kWave && (NR & (NR - 1)) == 0, "two lanes for each of a wave's rows");
    const int first_row = NR * (wave - kSpWaves);
    const int own_row = i0 + first_row + (lane & (NR - 1));
    const int row_begin = row_offsets[min(own_row, m)], row_end = row_offsets[min(own_row + 1, m)];
    barrier();                                                         // (the terms of L)
    const bool is_end = (lane & NR) != 0;
    auto window_of = [&](int begin, int end, int key) __attribute__((always_inline)) {
      const int guess = begin + (int)((float)(end - begin) * ((float)key / (float)k)) - kWave / 2;
      return max(begin, min(guess, end - kWave));
    };
    int bound;
    int index[NR][AHEAD];                                              // columns of the entries from the cursor on
    // The part's range of each row: the first entries with column step0 * 256 or more, and step1 * 256 (some fixed
    // place in rows that are not ascending).  64 neighbouring entries around the place that evenly spread columns
    // would give, all bounds at a time; if a bound is not among them, by halves.
    {
      const int key = (is_end ? step1 : step0) * kSpCols;
      const int window = window_of(row_begin, row_end, key);
      int probe[2 * NR], below = 0;
#pragma unroll
      for (int i = 0; i < 2 * NR; ++i)
        probe[i] = column_indices[max(0, min(__builtin_amdgcn_readlane(window, i) + lane, nnz - 1))];
#pragma unroll
      for (int i = 0; i < 2 * NR; ++i) {
        const unsigned long long less = __builtin_amdgcn_ballot_w64(
            lane < __builtin_amdgcn_readlane(row_end - window, i) && probe[i] < (i >= NR ? step1 : step0) * kSpCols);
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
      bound = lo;
    }
    int cursor[NR], range_end[NR];
#pragma unroll
    for (int rr = 0; rr < NR; ++rr) {
      cursor[rr] = __builtin_amdgcn_readlane(bound, rr);
      range_end[rr] = __builtin_amdgcn_readlane(bound, NR + rr);
    }
    // (loads past the last entry give 0; stores of lanes without an entry are given an offset past the end and dropped.
    // The range check is on the lane's offset, so all of it is there: nnz < 2^29.)
    const auto column_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(column_indices), 0, nnz * 4, 0x00020000);
    const auto out_rsrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, nnz * 4, 0x00020000);
    const int lane4 = lane * 4;
    auto columns_at = [&](int p0) __attribute__((always_inline)) {               // of entries p0 + lane
      return (int)__builtin_amdgcn_raw_buffer_load_b32(column_rsrc, p0 * 4 + lane4, 0, 0);
    };
    auto look_ahead = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int rr = 0; rr < NR; ++rr)
#pragma unroll
        for (int e = 0; e < AHEAD; ++e) index[rr][e] = columns_at(cursor[rr] + 64 * e);
    };
    const char* const cells = block + first_row * kSpStride;
    auto cell_of = [&](int rr, unsigned rel) __attribute__((always_inline)) {    // (lanes without an entry: any)
      return *reinterpret_cast<const float*>(cells + rr * kSpStride + min(rel, (unsigned)kSpCols - 1) * 4) * kSplitUnscale;
    };
    auto dot = [&](int rr, int column) __attribute__((always_inline)) {
      return split_lane_dot(L + (size_t)(i0 + first_row + rr) * n, R + (size_t)column * n, n);
    };
    // how many of a row's next 64 entries, `left` to its end, lie in the step's columns, from the first one on without a gap
    auto run = [&](int left, unsigned rel) __attribute__((always_inline)) {
      const unsigned long long in = __builtin_amdgcn_ballot_w64(rel < (unsigned)kSpCols) & __builtin_amdgcn_ballot_w64(lane < left);
      return in == ~0ull ? 64 : __builtin_ctzll(~in);
    };
    auto pick = [&](int step) __attribute__((always_inline)) {
      const int c0 = step * kSpCols;
      float value[NR][AHEAD], check = 0.f;
      int before[NR], taken[NR];
      bool more = false;
#pragma unroll
      for (int rr = 0; rr < NR; ++rr)
#pragma unroll
        for (int e = 0; e < AHEAD; ++e) value[rr][e] = cell_of(rr, (unsigned)(index[rr][e] - c0));
#pragma unroll
      for (int rr = 0; rr < NR; ++rr) {
        taken[rr] = 0;
        before[rr] = cursor[rr];
#pragma unroll
        for (int e = 0; e < AHEAD; ++e) {
          int count = run(range_end[rr] - before[rr] - 64 * e, (unsigned)(index[rr][e] - c0));
          if (e > 0) count = taken[rr] == 64 * e ? count : 0;
          float v = value[rr][e];
          check = __builtin_fmaf(v, 0.f, check);                       // NaN once one is not finite
          const int p0 = before[rr] + 64 * e;
          if (SCALED) v *= scale[(unsigned)min(p0 + lane, nnz - 1)];
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), out_rsrc,
                                                lane < count ? p0 * 4 + lane4 : (int)0x80000000, 0, 0);
          taken[rr] += count;
        }
        more |= taken[rr] == 64 * AHEAD;
        cursor[rr] += taken[rr];
      }
      if (__builtin_amdgcn_ballot_w64(check != 0.f) != 0) {            // results that are not finite
#pragma unroll
        for (int rr = 0; rr < NR; ++rr)
          for (int p = before[rr] + lane; p < cursor[rr]; p += 64) {
            const int column = column_indices[p];
            if (split_failed(cell_of(rr, (unsigned)(column - c0))))
              sddmm_store<float>(out, SCALED ? scale : nullptr, p, dot(rr, column));
          }
      }
      bool full[NR];
#pragma unroll
      for (int rr = 0; rr < NR; ++rr) full[rr] = taken[rr] == 64 * AHEAD;
      while (more) {                                                   // entries beyond what was looked ahead for
#pragma unroll
        for (int rr = 0; rr < NR; ++rr)
          if (full[rr]) index[rr][0] = columns_at(cursor[rr]);
        more = false;
#pragma unroll
        for (int rr = 0; rr < NR; ++rr)
          if (full[rr]) {
            const unsigned rel = (unsigned)(index[rr][0] - c0);
            const int count = run(range_end[rr] - cursor[rr], rel);
            const float v = cell_of(rr, rel);
            if (lane < count)
              sddmm_store<float>(out, SCALED ? scale : nullptr, cursor[rr] + lane, split_failed(v) ? dot(rr, index[rr][0]) : v);
            cursor[rr] += count;
            full[rr] = count == 64;
            more |= full[rr];
          }
      }
    };
    look_ahead();
    clocks.lap(kPhaseGather);
    for (int step = step0; step < step1; ++step) {
      barrier();                                                       // the block may be written
      clocks.lap(kPhaseBarrier);
      barrier();                                                       // ... and is there
      clocks.lap(kPhaseBarrier);
      __builtin_amdgcn_s_setprio(3);
      pick(step);
      if (step + 1 < step1) look_ahead();
      __builtin_amdgcn_s_setprio(0);
      clocks.lap(kPhaseScan);
    }
    // What is left of rows that are not ascending.  All the row's bounds, found as above but one at a time, where its results were.
    static_assert(kSpStride >= 4 * (256 + 1), "a bound for each part, of which there are as many as compute units at most");
    const int part_cols = steps_per_part * kSpCols;
    unsigned rows_left = 0;
    int stopped = 0;                                                   // lane l: the cursor of row l
#pragma unroll
    for (int rr = 0; rr < NR; ++rr) {
      rows_left |= (unsigned)(cursor[rr] < range_end[rr]) << rr;
      stopped = lane == rr ? cursor[rr] : stopped;
    }
    for (; rows_left != 0; rows_left &= rows_left - 1) {
      const int rr = __builtin_ctz(rows_left);
      const int from = __builtin_amdgcn_readlane(stopped, rr);
      const int begin = row_offsets[i0 + first_row + rr], end = row_offsets[i0 + first_row + rr + 1];
      volatile int* const bounds = reinterpret_cast<volatile int*>(block + (first_row + rr) * kSpStride);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      for (int i = 0; i <= parts; ++i) {
        const int key = i * part_cols, window = window_of(begin, end, key);
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
        if (lane == 0) bounds[i] = i == 0 ? begin : i == parts ? end : lo;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      for (int p = from + lane; p < bounds[part + 1]; p += 64) {
        const int column = column_indices[p], home = column / part_cols;
        if (home == part || p < bounds[home] || p >= bounds[home + 1])
          sddmm_store<float>(out, SCALED ? scale : nullptr, p, dot(rr, column));
      }
    }
  }
  clocks.store(blockIdx.x * (kSpWaves + PICKERS) + wave);
}

}  // namespace spdl
