// SpMM in mixed precision on the matrix cores (paper Sec. "Mixed Precision": fp16 operands,
// fp32 accumulation).  A panel of 32 sparse rows is expanded into a dense fp16 block in LDS
// (zeros where A stores nothing) and multiplied with MFMA: on this chip the dense fp16 matrix
// rate is some thirty times the fp32 vector rate, so for the moderately sparse matrices of deep
// learning the multiplications by zero cost less than gathering one row of B per stored entry.
// Sparsity still saves the memory and the traffic of A.
//
// A workgroup owns one panel and WAVES tiles of 256 output columns.  The panel
// is expanded once per chunk of up to kMfmaChunk columns of A and shared by the waves.  For a
// step of 16 columns of A, lane (c, h) of a wave loads rows k0+8h .. k0+8h+7 of B, columns
// n0+8c .. n0+8c+7 (eight 16-byte loads; the 32 lanes of a half read 512 contiguous bytes of each
// row), transposes the 8x8 block inside its registers with byte permutes, and so obtains, for
// each j < 8, the second MFMA operand of the 32 output columns n0+8c+j: B needs no staging and
// no transposed copy although the contraction runs over its slow dimension.  The eight
// results of a lane for one row are eight adjacent columns: one 16-byte store.
//
// Rows whose indices are not strictly ascending (duplicates included) cannot be expanded by
// plain stores; they are found while the panel is filled and computed by direct gathers.
//
// A row of B meets zeros of the panel in every sparse row that does not store its column, and 0 * Inf
// is NaN.  With `contain` an output that came out as NaN is looked at again: its row is computed by direct gathers
// for the tile's columns, so that an Inf or NaN of B reaches the rows that store its column and no other.
// Two comparisons for four results on finite data, nothing else.
// Any n from 8 on and any alignment (the lane at a row's end takes the row's last eight columns), k >= 16.
// The row order is not used: dense work is the same for every row.
//
// What bounds it: every MFMA of a panel needs a fresh 1 KB fragment of B, and a CU's
// vector memory path takes 16 clocks for that against the 32 clocks of the MFMA on one of four SIMDs: the
// kernel runs at the rate at which B arrives (1 MB per workgroup), at 1024 x 1024, n = 3136 some 40 bytes per clock
// and compute unit out of L2.  So the memory path has to be kept busy and free of anything else: the
// first loads of B go out before the offsets of the rows are there, ahead of the entries of the panel; steps
// past the end load nothing (with no lane active) instead of something unused; workgroups that share a
// tile's columns of B run on one XCD; and the waves that share a tile each finish their part of its rows.  
// (1024 x 1024 at 10 %, n = 3136: 23.4 us before all of this, 18.3 with it; with B in memory rather than
// in a cache, a quarter more.  Of a wave's time, by clocks inside the kernel: 14 % until the entries are here and the panel
// is clear, 13 to fill it, 54 main loop, 12 to exchange, convert and store, 7 at barriers.)
#pragma once
#include <type_traits>
#include "common.hpp"
#include "sddmm_mfma.hpp"

namespace spdl {

constexpr int kMfmaChunk = 1024;         // columns of A expanded at a time
constexpr int kMfmaSets = 6;             // steps of B rows held in registers per wave
constexpr int kMfmaPad = 8;              // halves of padding per panel row: row stride = 16 mod 128 bytes

// LDS: the panel (reused at the end to exchange the k-parts' sums), the flags of rows that cannot be expanded.
__host__ __device__ __forceinline__ int spmm_mfma_lds_bytes(int k, int waves, int kparts) {
  const int kc = ((k + 15) & ~15) < kMfmaChunk ? ((k + 15) & ~15) : kMfmaChunk;
  const int panel = 32 * (kc + kMfmaPad) * 2, sums = waves * (kparts - 1) * 32 * 64 * 16;
  return (panel > sums ? panel : sums) + 32 * 4;
}

// WAVES tiles of 256 columns per workgroup, and KP waves per tile that split the steps of the
// contraction between them (more loads in flight per CU).  At the end each of the KP waves collects,
// through LDS, the others' sums of 32 / KP of the rows and stores those.
template <int WAVES, int KP, bool CHUNKS, typename I = int>
__global__ __launch_bounds__(64 * WAVES * KP) void spmm_mfma_kernel(
    int m, int k, int n, int tiles_n, const int* __restrict__ row_offsets,
    const I* __restrict__ column_indices, const _Float16* __restrict__ values,
    const _Float16* __restrict__ B, _Float16* __restrict__ C, const _Float16* __restrict__ bias, int relu, int contain) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int NW = WAVES * KP;
  constexpr int NS = kMfmaSets;
  constexpr int RW = 32 / NW;                           // rows of the panel that a wave expands
  constexpr int PRE = 2;                                // sixty-fours of a row fetched ahead
  constexpr int FLAT = 64 / NW;                         // sixty-fours of the panel's entries fetched ahead by a wave
  static_assert(KP == 2 || KP == 4, "a part of the rows for each wave of a tile");
  PhaseClocks clocks;
  clocks.start();
  const int kc_max = min((k + 15) & ~15, kMfmaChunk);
  const int stride = kc_max + kMfmaPad;                 // halves per panel row
  _Float16* panel = reinterpret_cast<_Float16*>(lds_raw);
  int* bad = reinterpret_cast<int*>(lds_raw + spmm_mfma_lds_bytes(k, WAVES, KP) - 32 * 4);   // rows that cannot be expanded

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int tile_w = wave % WAVES;                      // which of the workgroup's tiles
  const int kpart = wave / WAVES;                       // which share of the steps
  const int c = lane & 31;
  const int h = lane >> 5;
  // Consecutive workgroup ids go round-robin to the 8 XCDs; each gets a run of the workgroups, tile after
  // tile, all panels of a tile before the next: an XCD's L2 then holds the columns of B that its
  // workgroups read, where with the panels one after the other every L2 fetched all of B.
  const int panels = (m + 31) >> 5;
  const int eighth = gridDim.x >> 3, xcd = blockIdx.x & 7;
  const int pos = xcd * eighth + min(xcd, (int)(gridDim.x & 7)) + (int)(blockIdx.x >> 3);
  const int tile_group = pos / panels;
  const int i0 = (pos - tile_group * panels) * 32;
  const int tile = tile_group * WAVES + tile_w;
  const bool active = tile < tiles_n;                   // idle waves still take part in the barriers
  const int n0 = tile * 256;
  const bool col_ok = active && n0 + 8 * c < n;
  const int col = col_ok ? piece_start(n0 + 8 * c, n, 8) : 0;      // this lane's eight output columns
  const _Float16* bp = B + col;

  if (CHUNKS && lane < RW) bad[wave + NW * lane] = 0;

  f32x16 acc[8];
  auto clear_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int t = 0; t < 16; ++t) acc[j][t] = 0.f;
  };
  if (CHUNKS) clear_sums();

  // Where each of this wave's rows continues in the next chunk of columns (rows in ascending order:
  // the entries of a chunk follow those of the chunk before).  The first chunk walks whole rows,
  // which is also what finds the rows that are not ascending; later chunks start at the cursor and
  // stop at the first 64 entries that reach past the chunk.
  int cursor[RW];
  for (int kc0 = 0; kc0 < k; kc0 += kMfmaChunk) {
    const int kc = min(k - kc0, kMfmaChunk);
    const int all_steps = (kc + 15) >> 4;
    const int per_part = (all_steps + KP - 1) / KP;
    const int s_begin = min(all_steps, kpart * per_part);
    const int steps = active ? min(all_steps, s_begin + per_part) - s_begin : 0;     // this wave's steps: s_begin ..
    // Second operand source: rows kc0 + 16*(s_begin + s) + 8h + r of B, r < 8: a scalar base that
    // moves with the step, and four rows down for r >= 4, plus this lane's fixed 32-bit byte offset (8h + r%4 rows
    // down, `col` columns in), so a load needs no vector arithmetic and a step little on the scalar unit.  The loads are issued from
    // inline assembly and waited for with explicit counts (they complete in the order issued, and
    // inside the main loop they are the only vector-memory operations): the compiler's own
    // placement of waits made every step wait for all loads in flight, which left one step's
    // loads to cover the whole latency.  A wait names the registers it releases as operands, so
    // that no use of them can be moved above it.  The one step that would reach past the last
    // row of B (k % 16 != 0) is kept out of this pipeline and done at the end with clamped rows
    // (the panel holds zeros there).
    // (rows of B are kept as four 32-bit words each: the byte permutes work on those)
    u32x4 w[NS][8];
    unsigned lane_off[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) lane_off[r] = (unsigned)(((8 * h + r) * n + col) * 2);
    const bool ragged_last = kc0 + 16 * (s_begin + steps) > k && steps > 0;   // this wave's last step is the ragged one
    const int full_steps = steps - (ragged_last ? 1 : 0);
    // The panels of a tile run on one XCD and want the same rows of B: each starts an eighth of its steps after
    // the one before, so that eight times as much of B is on its way from memory at a time.
    const int turn = ((i0 >> 5) & 7) * full_steps >> 3;
    const char* step_rows = reinterpret_cast<const char*>(B + (size_t)(kc0 + 16 * s_begin) * n);
    // A step past this wave's last full one loads with no lane active: nothing is fetched, but the
    // number of loads behind any set is the same at every step and one wait count serves them all.  An idle
    // wave has no steps and loads like that throughout: no path has a load less than another.  That no instruction
    // names a register of `w` while a load into it may be in flight is not left to the compiler, which knows nothing of
    // these loads: the build reads the machine code for it (loads_in_flight.py).
    auto load_rows = [&](int s, u32x4 (&ws)[8]) __attribute__((always_inline)) {
      const int t = s + turn - (s + turn >= full_steps ? full_steps : 0);
      const char* b0 = step_rows + (size_t)t * ((size_t)n * 32);
      const char* b1 = b0 + (size_t)n * 8;
      const int lanes = uniform((s - full_steps) >> 31);               // all ones while s < full_steps
      asm volatile(
          "s_mov_b32 exec_lo, %14\n\t"
          "s_mov_b32 exec_hi, %14\n\t"
          "global_load_dwordx4 %0, %8, %12\n\t"
          "global_load_dwordx4 %1, %9, %12\n\t"
          "global_load_dwordx4 %2, %10, %12\n\t"
          "global_load_dwordx4 %3, %11, %12\n\t"
          "global_load_dwordx4 %4, %8, %13\n\t"
          "global_load_dwordx4 %5, %9, %13\n\t"
          "global_load_dwordx4 %6, %10, %13\n\t"
          "global_load_dwordx4 %7, %11, %13\n\t"
          "s_mov_b64 exec, -1"
          : "=&v"(ws[0]), "=&v"(ws[1]), "=&v"(ws[2]), "=&v"(ws[3]), "=&v"(ws[4]), "=&v"(ws[5]), "=&v"(ws[6]), "=&v"(ws[7])
          : "v"(lane_off[0]), "v"(lane_off[1]), "v"(lane_off[2]), "v"(lane_off[3]), "s"(b0), "s"(b1), "s"(lanes)
          : "memory");
    };
    // the set is complete once only the NS - 1 later sets (8 loads each) are outstanding
    auto await_rows = [&](u32x4 (&ws)[8]) __attribute__((always_inline)) {
      static_assert(NS == 6, "wait count below");
      asm volatile("s_waitcnt vmcnt(40)"
                   : "+v"(ws[0]), "+v"(ws[1]), "+v"(ws[2]), "+v"(ws[3]), "+v"(ws[4]), "+v"(ws[5]), "+v"(ws[6]),
                     "+v"(ws[7])::"memory");
    };
    // keeps a set's registers allocated up to this point (a load into them may still be in flight)
    auto hold_rows = [&](u32x4 (&ws)[8]) __attribute__((always_inline)) {
      asm volatile("" : "+v"(ws[0]), "+v"(ws[1]), "+v"(ws[2]), "+v"(ws[3]), "+v"(ws[4]), "+v"(ws[5]), "+v"(ws[6]),
                   "+v"(ws[7])::"memory");
    };
    if constexpr (!CHUNKS) {
      // Expansion, all columns of A at once: the panel's entries lie one after the other in memory, and
      // each wave takes an equal run of them, 64 at a time, whatever rows they belong to.  The rows of 64
      // entries follow from the row starts among them (lane l holds the offset of row l), one step of
      // scalar work for each.  Nothing but these loads is ahead of the first sets of B.
      // (A wave is alone on its SIMD and issues an instruction every five clocks: all of this is written for
      // few of them.)
      const int first = uniform(row_offsets[i0]), last = uniform(row_offsets[min(i0 + 32, m)]);
      int row_start = row_offsets[min(i0 + min(lane, 32), m)];
      if (row_start >= last) row_start = 0x7fffffff;                     // (also rows without entries at the end)
      const int final_entry = max(last - 1, 0);
      const int share = (last - first + 64 * NW - 1) / (64 * NW);        // sixty-fours of this wave
      const int mine = min(first + wave * share * 64, final_entry);
      const I* my_columns = column_indices + mine;
      const _Float16* my_values = values + mine;
      // lanes past the last entry take it again (to the same place in the panel)
      auto entry = [&](int e) __attribute__((always_inline)) { return (unsigned)min(64 * e + lane, final_entry - mine); };
      int ecol[FLAT];
      _Float16 eval[FLAT];
#pragma unroll
      for (int e = 0; e < FLAT; ++e) {
        ecol[e] = (int)my_columns[entry(e)];
        eval[e] = my_values[entry(e)];
      }
      const int before = mine > first ? (int)column_indices[mine - 1] : -1;
#pragma unroll 8
      for (int o = tid * 16; o < 32 * stride * 2; o += 64 * NW * 16)
        *reinterpret_cast<f32x4*>(lds_raw + o) = f32x4{0.f, 0.f, 0.f, 0.f};
      if (tid < 32) bad[tid] = 0;
      __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt 0: the entries; lgkmcnt is left to the barrier
      load_rows(0, w[0]);
      load_rows(1, w[1]);
      clear_sums();
      clocks.lap(kPhaseSetup);
      __syncthreads();
      clocks.lap(kPhaseBarrier);
      // Ascending rows have ascending places in the panel, across rows too: an entry whose place is not above
      // its predecessor's shows a row that is not ascending.
      int row = __builtin_popcountll(__builtin_amdgcn_ballot_w64(row_start <= mine)) - 1;
      int next = __builtin_amdgcn_readlane(row_start, row + 1);
      int place_before = -1;                             // (the first of a wave's entries: looked at below)
      unsigned long long descending = 0;
      const int row_bytes_lds = stride * 2;
      auto place = [&](int e, int cidx, _Float16 a) __attribute__((always_inline)) {
        const int p0 = mine + 64 * e, p = p0 + lane;
        int at = row * row_bytes_lds;
        while (next <= p0 + 63) {
          ++row;
          at = p >= next ? row * row_bytes_lds : at;
          next = __builtin_amdgcn_readlane(row_start, row + 1);
        }
        at += 2 * (int)min((unsigned)cidx, (unsigned)kc_max);            // a column outside the matrix: padding
        *reinterpret_cast<_Float16*>(lds_raw + at) = a;
        const int prev = __builtin_amdgcn_update_dpp(place_before, at, 0x138, 0xf, 0xf, false);   // the lane below's; lane 0's
        place_before = __builtin_amdgcn_readlane(at, 63);
        descending |= __builtin_amdgcn_ballot_w64(prev >= at && p < last);
      };
#pragma unroll
      for (int e = 0; e < FLAT; e += 4) {
        if (e < share) {
#pragma unroll
          for (int f = 0; f < 4; ++f) place(e + f, ecol[e + f], eval[e + f]);
        }
        // (further sets of B in between: the memory path takes 500 clocks for one of all waves)
        if (2 + e / 4 < NS - 1) load_rows(2 + e / 4, w[2 + e / 4]);
      }
      for (int e0 = FLAT; e0 < share; e0 += 4) {
        int cmore[4];
        _Float16 amore[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          cmore[f] = (int)my_columns[entry(e0 + f)];
          amore[f] = my_values[entry(e0 + f)];
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);              // (no path leaves one of these to be waited for in the main loop)
#pragma unroll
        for (int f = 0; f < 4; ++f) place(e0 + f, cmore[f], amore[f]);
      }
      // which rows they are, and the pair across the start of the run: no need to hurry unless there is one
      const bool head = __builtin_amdgcn_ballot_w64(row_start == mine) != 0;
      if (descending != 0 || (!head && before >= __builtin_amdgcn_readlane(ecol[0], 0))) {
        for (int p = mine + lane; p < min(mine + 64 * share, last); p += 64) {
          int rr = 0, begin = first;
          for (int r = 1; r < 32; ++r) {
            const int at = __builtin_amdgcn_readlane(row_start, r);
            if (p >= at) {
              rr = r;
              begin = at;
            }
          }
          if (p > begin && column_indices[p - 1] >= column_indices[p]) bad[rr] = 1;
        }
      }
    } else {
      // Expansion, a chunk of columns.  A wave takes every fourth row of the panel and its
      // lanes take the row's entries 64 at a time: coalesced loads, no search for the row of an
      // entry, and the loads of each row's first 128 entries are all issued before the panel is
      // even cleared.  Longer rows finish in a loop.  An entry whose column is not above its
      // predecessor's marks the row as not expandable (the predecessor is the lane below, or lane
      // 63 of the previous 64).
      int row_begin[RW], row_end[RW];
      int cfirst[RW][PRE];
      _Float16 afirst[RW][PRE];
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const int rr = wave + NW * i;
        row_begin[i] = uniform(row_offsets[min(i0 + rr, m)]);
        row_end[i] = uniform(row_offsets[min(i0 + rr + 1, m)]);
        if (kc0 > 0) row_begin[i] = cursor[i];
      }
      // half of the sets of B go ahead of the entries: the memory path works on them until the offsets are
      // there and while the panel is filled (more would hold the entries up, which arrive after everything
      // issued before them)
#pragma unroll
      for (int u = 0; u < NS / 2; ++u) load_rows(u, w[u]);
      const int kend = kc0 + kc;
#pragma unroll
      for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int e = 0; e < PRE; ++e) {
          const int p = row_begin[i] + 64 * e + lane;
          cfirst[i][e] = 0;
          afirst[i][e] = (_Float16)0.f;
          if (p < row_end[i]) {
            cfirst[i][e] = (int)column_indices[p];
            afirst[i][e] = values[p];
          }
        }
      if (kc0 > 0) __syncthreads();                        // the previous chunk's reads are done
#pragma unroll
      for (int i = 0; i < RW; ++i)                         // a wave clears the rows that it fills: no barrier in between
        for (int o = lane * 16; o < stride * 2; o += 64 * 16)
          *reinterpret_cast<f32x4*>(lds_raw + (wave + NW * i) * stride * 2 + o) = f32x4{0.f, 0.f, 0.f, 0.f};
      asm volatile("" ::: "memory");
      // (vmcnt 0; the other two counters are left alone.)  No load is in flight while the panel is filled: the
      // compiler, short of registers there, may move some, and does not know which are still to be written.
      __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
      for (int u = 0; u < NS / 2; ++u) hold_rows(w[u]);
      clocks.lap(kPhaseSetup);
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const int rr = wave + NW * i;
        _Float16* prow = panel + rr * stride;
        int below = -1;                                    // column of the previous 64's lane 63
        bool unordered = false;
        int before_end = 0;                                // entries seen whose column lies before the chunk's end
        bool past = false;                                 // some entry seen lies past the chunk
        auto place = [&](int p, int cidx, _Float16 a) __attribute__((always_inline)) {
          const int prev = __builtin_amdgcn_update_dpp(below, cidx, 0x138, 0xf, 0xf, false);   // the lane below's; lane 0: below
          const bool valid = p < row_end[i];
          if (valid) {
            if (prev >= cidx) unordered = true;
            const unsigned rel = (unsigned)(cidx - kc0);
            if (rel < (unsigned)kc) prow[rel] = a;
          }
          const unsigned long long inside = __builtin_amdgcn_ballot_w64(valid && cidx < kend);
          before_end += __builtin_popcountll(inside);
          past = past || __builtin_amdgcn_ballot_w64(valid && cidx >= kend) != 0;
          below = __builtin_amdgcn_readlane(cidx, 63);
        };
#pragma unroll
        for (int e = 0; e < PRE; ++e)
          if (row_begin[i] + 64 * e < row_end[i]) place(row_begin[i] + 64 * e + lane, cfirst[i][e], afirst[i][e]);
        for (int base = row_begin[i] + 64 * PRE; base < row_end[i]; base += 256) {   // long rows: 256 entries per round
          if (kc0 > 0 && past) break;                      // (ascending rows: nothing further belongs to this chunk)
          int cmore[4];
          _Float16 amore[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int q = min(base + 64 * e + lane, row_end[i] - 1);
            cmore[e] = (int)column_indices[q];
            amore[e] = values[q];
          }
          __builtin_amdgcn_s_waitcnt(0x0F70);              // (no path leaves one of these to be waited for in the main loop)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (base + 64 * e < row_end[i]) place(base + 64 * e + lane, cmore[e], amore[e]);
        }
        if (kc0 == 0 && __builtin_amdgcn_ballot_w64(unordered) != 0 && lane == 0) bad[rr] = 1;
        cursor[i] = row_begin[i] + before_end;
      }
#pragma unroll
      for (int u = NS / 2; u < NS - 1; ++u) load_rows(u, w[u]);
    }
    clocks.lap(kPhaseScan);
    __syncthreads();
    clocks.lap(kPhaseBarrier);
    // first operands: rows c of the panel, columns 16*s + 8h .. +7 of the chunk
    const _Float16* ap = panel + c * stride + 8 * h + 16 * s_begin;
    auto fragment = [&](int s) __attribute__((always_inline)) {        // (the ragged step is the last in any order)
      const int t = s >= full_steps ? s : s + turn - (s + turn >= full_steps ? full_steps : 0);
      return *reinterpret_cast<const f16x8*>(ap + 16 * t);
    };
    // (the fragment of a step is read from LDS one step ahead: with one wave per SIMD nothing
    // else would cover the LDS latency)
    f16x8 a_next;
    auto step = [&](int s, const u32x4 (&ws)[8]) __attribute__((always_inline)) {
      const f16x8 a = a_next;
      if (s + 1 < steps) a_next = fragment(s + 1);
      // 8x8 transpose of halves inside the lane: operand j, word q = (ws[2q][j], ws[2q+1][j])
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        u32x4 packed;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const unsigned sel = (j & 1) ? 0x07060302u : 0x05040100u;
          packed[q] = __builtin_amdgcn_perm(ws[2 * q + 1][j / 2], ws[2 * q][j / 2], sel);
        }
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, __builtin_bit_cast(f16x8, packed), acc[j], 0, 0, 0);
      }
    };
    if (steps > 0) a_next = fragment(0);
    for (int s0 = 0; s0 < full_steps; s0 += NS) {
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int s = s0 + u;
        load_rows(s + NS - 1, w[(u + NS - 1) % NS]);
        await_rows(w[u]);
        if (s < full_steps) step(s, w[u]);
      }
    }
    // (every load has landed before its registers serve anything else)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int u = 0; u < NS; ++u) hold_rows(w[u]);
    clocks.lap(kPhaseSteps);
    if (ragged_last) {
      const int k0 = kc0 + 16 * (s_begin + full_steps);
      u32x4 tail[8];
#pragma unroll
      for (int r = 0; r < 8; ++r)
        tail[r] = __builtin_bit_cast(u32x4, (f16x8)*reinterpret_cast<const f16x8_any*>(bp + (size_t)min(k0 + 8 * h + r, k - 1) * n));
      step(full_steps, tail);
    }
    clocks.lap(kPhaseGather);
  }
  // Register t of lane (c, h) in accumulator j is row 8*(t/4) + 4h + t%4, column `col` + j.  Wave `kpart`
  // of a tile finishes the quarters G * kpart .. of t; the others hand it theirs through LDS (the panel
  // is no longer needed), sixteen bytes per access.
  constexpr int G = 4 / KP;
  f32x4* sums = reinterpret_cast<f32x4*>(lds_raw) + (size_t)tile_w * (KP * (KP - 1) * 8 * G * 64) + lane;
  float row_bias[G * 4];                                 // (zeros without bias: no sum is -0)
#pragma unroll
  for (int t = 0; t < G * 4; ++t) {
    const int row = i0 + 8 * (G * kpart + t / 4) + 4 * h + t % 4;
    row_bias[t] = bias && row < m ? (float)bias[row] : 0.f;
  }
  auto hand_over = [&](auto part) __attribute__((always_inline)) {
    constexpr int P = decltype(part)::value;
#pragma unroll
    for (int d = 0; d < KP; ++d)
      if (d != P) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const int t = 4 * (G * d + g);
            sums[(((d * (KP - 1) + (P < d ? P : P - 1)) * 8 + j) * G + g) * 64] =
                f32x4{acc[j][t], acc[j][t + 1], acc[j][t + 2], acc[j][t + 3]};
          }
      }
  };
  unsigned bad_mask = 0;                                 // rows that are computed by gathers
  unsigned nan_mask = 0;                                 // ... those of them in which this wave has met a NaN
  auto finish = [&](auto part) __attribute__((always_inline)) {
    constexpr int P = decltype(part)::value;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      f32x4 total[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int t = 4 * (G * P + g);
        total[j] = f32x4{acc[j][t], acc[j][t + 1], acc[j][t + 2], acc[j][t + 3]};
#pragma unroll
        for (int o = 0; o < KP - 1; ++o) total[j] += sums[(((P * (KP - 1) + o) * 8 + j) * G + g) * 64];
      }
      if (contain) {                                     // (before the bias and a ReLU that would hide it)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
          bool nan = false;
#pragma unroll
          for (int j = 0; j < 8; j += 2) nan |= __builtin_isunordered(total[j][tt], total[j + 1][tt]);
          const unsigned long long lanes = __builtin_amdgcn_ballot_w64(nan && col_ok);
          const unsigned both = ((unsigned)lanes != 0 ? 1u : 0u) | ((unsigned)(lanes >> 32) != 0 ? 16u : 0u);   // h = 0, 1
          nan_mask |= both << (8 * (G * P + g) + tt);
        }
        bad_mask |= nan_mask;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) total[j][tt] += row_bias[4 * g + tt];
      if (relu) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) total[j][tt] = fmaxf(total[j][tt], 0.f);
      }
      const int rr = 8 * (G * P + g) + 4 * h;
      _Float16* out = C + (size_t)(i0 + rr) * n + col;
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = total[j][tt];
        if (col_ok && i0 + rr + tt < m && !((bad_mask >> (rr + tt)) & 1)) Pack<_Float16, 8>::store(out, v);
        out += n;
      }
    }
  };
  clocks.lap(kPhaseRest);
  __syncthreads();
  clocks.lap(kPhaseBarrier);
  if (active) {
    if (kpart == 0) hand_over(std::integral_constant<int, 0>{});
    else if (kpart == 1) hand_over(std::integral_constant<int, 1>{});
    else if (KP > 2 && kpart == 2) hand_over(std::integral_constant<int, KP - 2>{});
    else hand_over(std::integral_constant<int, KP - 1>{});
  }
  clocks.lap(kPhaseRest);
  __syncthreads();
  clocks.lap(kPhaseBarrier);
  if (!active) {
    clocks.store(blockIdx.x * NW + wave);
    return;
  }
  const unsigned unexpanded = (unsigned)__builtin_amdgcn_ballot_w64(lane < 32 && bad[lane & 31] != 0);
  bad_mask = unexpanded;
  if (kpart == 0) finish(std::integral_constant<int, 0>{});
  else if (kpart == 1) finish(std::integral_constant<int, 1>{});
  else if (KP > 2 && kpart == 2) finish(std::integral_constant<int, KP - 2>{});
  else finish(std::integral_constant<int, KP - 1>{});
  // Rows that could not be expanded, left to the first wave of the tile, and rows in which a NaN was met: direct
  // gathers, four columns per lane.  Eight entries at a time; positions past the row's end fetch its last entry
  // again and multiply nothing (0 * Inf).
  unsigned left = (kpart == 0 ? unexpanded : 0u) | (nan_mask & ~unexpanded);
  if (m - i0 < 32) left &= (1u << (m - i0)) - 1u;
  for (; left != 0; left &= left - 1) {
    const int row = i0 + __builtin_ctz(left);
    const bool ok = n0 + 4 * lane < n;
    const int col4 = ok ? piece_start(n0 + 4 * lane, n, 4) : 0;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    const int end = uniform(row_offsets[row + 1]);
    for (int p = uniform(row_offsets[row]); p < end; p += 8) {
      float a[8], b[8][4];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = min(p + u, end - 1);
        a[u] = (float)values[q];
        Pack<_Float16, 4>::load(B + (size_t)(int)column_indices[q] * n + col4, b[u]);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (p + u < end) {
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = __builtin_fmaf(a[u], b[u][j], v[j]);
        }
    }
    spmm_epilogue<_Float16, 4>(v, bias, row, relu);
    if (ok) Pack<_Float16, 4>::store(C + (size_t)row * n + col4, v);
  }
  clocks.lap(kPhaseRest);
  clocks.store(blockIdx.x * NW + wave);
}

}  // namespace spdl
