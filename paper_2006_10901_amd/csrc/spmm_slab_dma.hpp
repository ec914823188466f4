// SpMM, slab family with asynchronous global->LDS copies: same decomposition as the
// producer/consumer slab kernel (64 sparse rows x 64-column tiles per workgroup, B streamed
// through LDS in slabs of S rows, 16-lane groups with DPP-broadcast multiply-adds), but all
// 16 waves compute, one sparse row per 16-lane group, and each wave moves its share of the
// next slab with direct-to-LDS loads (no staging registers, no LDS store instructions).
//
// A wait for sparse elements that were requested after the slab copies also waits for the
// copies, so waits inside a stage are avoided: the kernel works in long rounds of 16*PW*SHARE
// (value, column) pairs per row, the next pairs are requested as soon as the cursor is
// known, before the arithmetic of the current round, and they are first needed in the
// next stage.  The only wait is the one at the end of a stage, for everything (copies and pair
// loads alike have had the stage's arithmetic to complete); no assumption is made about the
// order in which copies and ordinary loads retire.  A row with more than 16*PW*SHARE pairs in a
// slab takes further rounds, each behind a full wait.
//
// What bounds it: the steps' issue rate at the dense end; below 15 % density a stage is held by the vector
// memory path, 64 bytes a clock for the slab (64 KB), the look-ahead of pairs and their instructions alike, and by
// the fill of the step's LDS pipeline per round.  Hence one piece of PW consecutive pairs per lane and array: two
// loads for what took two per sixteen pairs, and one run of steps per round instead of one per sixteen pairs
// (8192 x 10240, n = 128, us per launch, sixteen pairs per load -> pieces: 10 % 90.1 -> 81.5, 13 % 109.6 -> 100.0, 15 %
// 117.4 -> 108, 20 % 143 -> 136, 30 % 201 -> 193; 16384 x 4096 at 10 %: 75.5 -> 70.1).
#pragma once
#include "common.hpp"
#include "spmm_slab.hpp"

namespace spdl {

// RPG = sparse rows per 16-lane group (1 or 2): the workgroup owns 64*RPG rows.  Two rows per
// group halve the traffic of B and the number of stages per unit of work when the output has
// enough tiles to fill the machine anyway.
// PW = consecutive pairs of a row that a lane fetches at once, 1 .. 4 (slab_pairs_per_lane).
// SHARE = lane groups that share a row: group g of a row's SHARE has every SHARE-th piece from the g-th on, and the
// groups' sums are added at the end of a tile.  A workgroup then owns 64 / SHARE rows, so that an output of a half or a
// quarter of the machine's tiles still gives every compute unit a workgroup of sixteen waves, and a row's steps are
// shared out instead of left to one group (before -> after, the former being workgroups of eight waves with 32 rows:
// 3004 x 2251 at 15 %, n = 75: 21.8 us -> 17.5; 8192 x 10240 at 20 %, n = 64: 101.7 -> 87; 2048 x 8000 at 20 %, n = 100:
// 79.7 -> 48.1; 4096 x 8000 at 30 %, n = 50: 103.5 -> 52.9).
// NW = waves per workgroup: 16, or 8 (panels of 32 rows) for small products with few tiles.  One workgroup per CU.
template <int S, int RPG, int PW, int SHARE, int NW = 16>
__global__ __launch_bounds__(64 * NW) void spmm_slab_dma_kernel(
    int m, int k, int n, int nnz, int tiles_n, int tiles_per_wg, int panels,
    const int* __restrict__ row_offsets, const int* __restrict__ column_indices,
    const float* __restrict__ values, const int* __restrict__ row_order, const float* __restrict__ B,
    float* __restrict__ C, const float* __restrict__ bias, int relu, int tiles_first) {
  using T = float;
  static_assert(RPG == 1 || SHARE == 1, "a row shared by lane groups, or several rows to a group");
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int kBufBytes = (S + 1) * kSlabTile * 4;      // S data rows + one all-zero row
  constexpr int kZeroOff = S * kSlabTile * 4;
  constexpr int kCopies = S / (4 * NW);                   // 1 KB direct-to-LDS loads per wave per slab

  PhaseClocks clocks;
  clocks.start();
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int sub = lane >> 4;
  const int l16 = lane & 15;
  const int lane_b = l16 * 16;

  const int groups_n = (tiles_n + tiles_per_wg - 1) / tiles_per_wg;
  int panel, tile_group;
  if (tiles_first ? !slab_wg_map(blockIdx.x, groups_n, panels, tile_group, panel)
                  : !slab_wg_map(blockIdx.x, panels, groups_n, panel, tile_group)) return;
  const int tile_begin = tile_group * tiles_per_wg;
  const int tile_end = min(tiles_n, tile_begin + tiles_per_wg);
  const int nslabs = nnz < PW ? 0 : (k + S - 1) / S;       // (rows that are not walked are gathered at the end)
  const int stages = (tile_end - tile_begin) * nslabs;

  if (tid < 2 * kSlabTile)
    *reinterpret_cast<float*>(lds_raw + (tid >> 6) * kBufBytes + kZeroOff + (tid & 63) * 4) = 0.f;

  // Slab copy: copy i of wave w fills slab rows (i*NW + w)*4 .. +3; lane L brings row L/16 of
  // those, columns 4*(L%16) .. +3, and the hardware places lane L's 16 bytes at M0 + 16*L.
  // The address is a scalar base (start of the slab in B, moved from stage to stage with scalar
  // arithmetic) plus a per-lane byte offset that is the same in every stage except a ragged
  // last slab, whose rows past k are clamped to row k-1, and a ragged last tile, whose columns
  // past n are clamped to the first ones (nothing valid ever reads those) and whose last piece
  // of four starts at n - 4 (piece_start): no address is past B, whatever n and its alignment.
  // (S * n * 4 < 2^31 is checked on the host.)
  unsigned row_off[kCopies], row_off_last[kCopies];
  const int last_rows = k - (nslabs - 1) * S;               // rows of the last slab, 1..S
#pragma unroll
  for (int i = 0; i < kCopies; ++i) {
    const int lrow = (i * NW + wave) * 4 + sub;
    row_off[i] = (unsigned)lrow * (unsigned)n * 4u;
    row_off_last[i] = (unsigned)min(lrow, last_rows - 1) * (unsigned)n * 4u;
  }
  // The copies are issued from inline assembly: the compiler treats its own direct-to-LDS loads
  // as touching both memory paths and then turns every later wait, for LDS reads and for pair
  // loads alike, into a wait for everything.  Their completion is covered by the explicit full
  // wait and barrier that end every stage.  M0 (the LDS destination) is not used by anything
  // the compiler generates in this kernel.
  auto copy_stage = [&](int q) {
    const int t = q / nslabs;
    const int slab = q - t * nslabs;
    const int tile = tile_begin + t;
    const int piece = piece_start(tile * kSlabTile + l16 * 4, n, 4);
    const unsigned col_off = piece < n ? (unsigned)piece * 4u : 0u;
    const char* base = reinterpret_cast<const char*>(B + (size_t)slab * S * n);
    const unsigned dst = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)(lds_raw + (q & 1) * kBufBytes) +
                         (unsigned)wave * (4 * kSlabTile * 4);
    const bool last = slab == nslabs - 1;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      const unsigned voff = (last ? row_off_last[i] : row_off[i]) + col_off;
      const unsigned m0v = dst + (unsigned)i * (NW * 4 * kSlabTile * 4);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(m0v), "v"(voff), "s"(base) : "memory", "m0");
    }
  };

  SlabRow rows[RPG];
#pragma unroll
  for (int j = 0; j < RPG; ++j) {
    // Row binning (paper Sec. "Row Swizzle Load Balancing"): a wave's 4*RPG rows are adjacent
    // in the row order (a bundle of similar lengths), and a workgroup takes every panels-th
    // bundle, so each workgroup gets the same mix of long and short bundles.
    const int slot = SHARE == 1 ? ((wave * panels + panel) * 4 + sub) * RPG + j
                                : (wave * panels + panel) * (4 / SHARE) + sub / SHARE;
    rows[j].row = -1;
    rows[j].p_begin = rows[j].row_end = 0;
    if (slot < m) {
      const int r = row_order ? row_order[slot] : slot;
      rows[j].row = r;
      rows[j].p_begin = row_offsets[r];
      rows[j].row_end = row_offsets[r + 1];
    }
  }
  using Mask = SlabMask<SHARE>;
  // The row's lanes in a wave mask, and the lanes that have met a pair of the slab whose predecessor is not in it: an
  // ascending row has none.  (Pairs are counted, not looked for from the front, which is a third of the scalar work; what
  // was counted of a row with such a pair says nothing, and the row is redone.)
  const unsigned long long row_mask = SHARE == 1 ? 0xffffull << (16 * sub) : SHARE == 2 ? 0xffffffffull << (16 * (sub & 2)) : ~0ull;
  const unsigned row_lo = (unsigned)row_mask, row_hi = (unsigned)(row_mask >> 32);
  unsigned long long strays[RPG];
#pragma unroll
  for (int j = 0; j < RPG; ++j) strays[j] = 0;
  const int lane_pair = (l16 * SHARE + (sub & (SHARE - 1))) * PW;  // this lane's first, from the cursor
  float acc[RPG][4];

  // The next 16 * PW * SHARE pairs of each row from position `at`.  The loaded words are kept
  // raw (no arithmetic on them here): the compiler waits for a load at its first use, and the
  // first use is in the next stage, after the full wait that ends every stage.  32-bit byte
  // offsets from scalar bases (nnz < 2^29 is checked on the host).  A piece that would reach past
  // the arrays' end is loaded from further in front and shifted when it is used (slab_piece_shift).
  int cc[RPG][PW], at[RPG];
  float aa[RPG][PW];
  const int last_start = nnz - PW;
  auto fetch_pairs = [&](int j, int from) {
    at[j] = from;
    const char* cbase = reinterpret_cast<const char*>(column_indices);
    const char* vbase = reinterpret_cast<const char*>(values);
    const unsigned o = (unsigned)min(from + lane_pair, last_start) << 2;
    const SlabPiece<int, PW> c = *reinterpret_cast<const SlabPiece<int, PW>*>(cbase + o);
    const SlabPiece<float, PW> a = *reinterpret_cast<const SlabPiece<float, PW>*>(vbase + o);
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      cc[j][e] = c.v[e];
      aa[j][e] = a.v[e];
    }
  };
  // every vector-memory operation of this wave (pair loads, slab copies) has completed
  auto wait_everything = [&]() { __builtin_amdgcn_s_waitcnt(0); };

  // One long round of row j in the slab starting at slab_start: the fetched pairs that fall into
  // the slab.  Returns true when some row's last one did, i.e. the slab may hold more pairs of that row.
  // `restart`: this is the last slab of a tile and another tile follows, so once the row is done
  // here the next pairs needed are those at the row start again.
  auto long_round = [&](int j, const char* buf, int slab_start, bool restart) -> bool {
    const int first = at[j] + lane_pair, left = rows[j].row_end - first;
    if (__builtin_amdgcn_ballot_w64(first > last_start && left > 0) != 0) slab_piece_shift<PW>(cc[j], aa[j], first - last_start);
    float av[PW];
    int off[PW];
    unsigned long long mk[PW];
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      const unsigned rel = (unsigned)(cc[j][e] - slab_start);
      mk[e] = __builtin_amdgcn_ballot_w64(left > e) & __builtin_amdgcn_ballot_w64(rel < (unsigned)S);
      if (e > 0) strays[j] |= mk[e] & ~mk[e - 1];
      if constexpr (SHARE == 4) rows[j].p += __builtin_popcountll(mk[e]);
      else rows[j].p += __builtin_popcount((unsigned)mk[e] & row_lo) + __builtin_popcount((unsigned)(mk[e] >> 32) & row_hi);
      const bool in = __builtin_amdgcn_inverse_ballot_w64(mk[e]);
      av[e] = in ? aa[j][e] : 0.f;
      off[e] = in ? (int)(rel * (kSlabTile * 4)) : kZeroOff;
    }
    strays[j] |= mk[0] & ~(Mask::lane_before(mk[PW - 1]) | Mask::kFirst);
    unsigned used[PW == 3 ? 3 : 1];
#pragma unroll
    for (int e = 0; e < (PW == 3 ? 3 : 1); ++e) used[e] = Mask::used(mk[e]);
    const bool more = Mask::full(mk[PW - 1]);
    // the next pairs, first needed in the next stage (or in the next long round of this one)
    fetch_pairs(j, (restart && !more) ? rows[j].p_begin : rows[j].p);
    clocks.lap(kPhaseScan);
    if (used[0] != 0) wide_steps<PW>(acc[j], av, off, buf, lane_b, used);
    clocks.lap(kPhaseSteps);
    return more;
  };

  if (nslabs > 0) {
    copy_stage(0);
#pragma unroll
    for (int j = 0; j < RPG; ++j) fetch_pairs(j, rows[j].p_begin);
  }
  wait_everything();
  __builtin_amdgcn_s_barrier();
  clocks.lap(kPhaseSetup);
  int q = 0;
  for (int tile = tile_begin; tile < tile_end; ++tile) {
    const int col = piece_start(tile * kSlabTile + l16 * 4, n, 4);
    const bool col_ok = col < n;
#pragma unroll
    for (int j = 0; j < RPG; ++j) {
      rows[j].p = rows[j].p_begin;          // the pairs at the row start are already in registers
      acc[j][0] = acc[j][1] = acc[j][2] = acc[j][3] = 0.f;
    }
    for (int s = 0; s < nslabs; ++s, ++q) {
      // A use of the youngest pair register before the copies are issued: the compiler places
      // its wait for the pair loads here, where they completed long ago (full wait at the end
      // of the previous stage), instead of after the copies, where it would wait for those too.
      asm volatile("v_mov_b32 %0, %0" : "+v"(aa[RPG - 1][PW - 1]));
      clocks.lap(kPhaseRest);
      if (q + 1 < stages) copy_stage(q + 1);
      clocks.lap(kPhaseIssue);
      const char* buf = lds_raw + (q & 1) * kBufBytes;
#pragma unroll
      for (int j = 0; j < RPG; ++j) {
        const bool restart = s == nslabs - 1 && tile + 1 < tile_end;
        // The first long round stands outside the loop: inside it the compiler would have to
        // wait for the previous iteration's loads, and with them for the copies just issued.
        if (long_round(j, buf, s * S, restart))
          while (long_round(j, buf, s * S, restart)) {}          // more than the fetched pairs in this slab
      }
      wait_everything();
      clocks.lap(kPhaseWait);
      __builtin_amdgcn_s_barrier();
      clocks.lap(kPhaseBarrier);
    }
#pragma unroll
    for (int j = 0; j < RPG; ++j) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {                  // the groups of a row
        if constexpr (SHARE >= 2) acc[j][v] += __shfl_xor(acc[j][v], 16);
        if constexpr (SHARE == 4) acc[j][v] += __shfl_xor(acc[j][v], 32);
      }
      if (rows[j].p != rows[j].row_end || (strays[j] & row_mask) != 0) {
        acc[j][0] = acc[j][1] = acc[j][2] = acc[j][3] = 0.f;
        const T* Bcol = B + (col_ok ? col : 0);
        for (int t = rows[j].p_begin; t < rows[j].row_end; ++t) {
          const float a = (float)values[t];
          float b[4];
          Pack<T, 4>::load(Bcol + (size_t)column_indices[t] * n, b);
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[j][v] = __builtin_fmaf(a, b[v], acc[j][v]);
        }
      }
      if (rows[j].row >= 0 && col_ok && (sub & (SHARE - 1)) == 0) {
        spmm_epilogue<T, 4>(acc[j], bias, rows[j].row, relu);
        Pack<T, 4>::store(C + (size_t)rows[j].row * n + col, acc[j]);
      }
    }
  }
  clocks.lap(kPhaseRest);
  clocks.store(blockIdx.x * NW + wave);
}

}  // namespace spdl
