// SpMM, slab family for wide outputs: the copy-based slab kernel with the loop nest turned
// round.  That kernel walks its output tiles one after the other and, inside a tile, the slabs
// of B; everything it works out about a sparse row and a slab (which of the fetched pairs lie in
// the slab, their LDS offsets, the new cursor) is worked out again for every tile, although it
// depends on the row and the slab only.  Here a workgroup keeps the accumulators of up to TPW
// tiles in registers and walks slab by slab: the pairs of a slab are scanned once, and the TPW
// stages that follow (one per tile: copy of the tile's part of the slab, multiply-adds) reuse the
// masked values and offsets from registers.  The look-ahead for the next slab is requested at the
// scan and has TPW stages to arrive.
//
// The look-ahead holds 16 PW pairs of a row: as one piece of PW consecutive pairs per lane (PIECES), or as PW chunks of sixteen.
// Pieces take two loads instead of 2 PW and one run of steps instead of PW; chunks, with three of which this kernel first ran,
// take fewer registers and bytes than pieces of four (us per launch, chunks / pieces of two, three, four: 1024 x 4096, n = 4096, 10 %
// 123.3 / 132.1 / 124.2 / 123.9, 5 % 92.4 / 87.6 / 89.4 / 91.5; 16384 x 4096 at 10 %, n = 256: 115.4 / 125.5 / 117.1 / 116.3).  So pieces of two
// where 32 pairs hold a row's in a slab (mean and three standard deviations), three chunks where 48 do, pieces of four up to
// 64, where the form that scans for every tile anew ran before (1393 x 5572 at 13 %, n = 3464: 309 -> 277; 7424 x 1856 at 14 %,
// n = 580: 108.7 -> 100.8).
//
// A row with more pairs inside one slab needs further rounds in that slab, 64 pairs at
// a time (16 beside pieces of four), each behind a full wait; they are not kept, every tile's stage fetches and scans them
// again.
#pragma once
#include "common.hpp"
#include "spmm_slab.hpp"

namespace spdl {

template <int S, int RPG, int PW, bool PIECES, int TPW>
__global__ __launch_bounds__(1024) void spmm_slab_tiles_kernel(
    int m, int k, int n, int nnz, int tiles_n, int tiles_per_wg, int panels,
    const int* __restrict__ row_offsets, const int* __restrict__ column_indices,
    const float* __restrict__ values, const int* __restrict__ row_order, const float* __restrict__ B,
    float* __restrict__ C, const float* __restrict__ bias, int relu, int tiles_first) {
  constexpr int NW = 16;
  // pairs per lane and round of a row that has more in a slab than the look-ahead (as many as there are registers for)
  constexpr int kRest = PW == 4 ? 1 : 4;
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int kBufBytes = (S + 1) * kSlabTile * 4;
  constexpr int kZeroOff = S * kSlabTile * 4;
  constexpr int kCopies = S / (4 * NW);

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
  const int ntiles = min(tiles_n, tile_begin + tiles_per_wg) - tile_begin;      // 1 .. TPW
  const int nslabs = nnz < 4 ? 0 : (k + S - 1) / S;       // (rows that are not walked are gathered at the end)
  const int stages = ntiles * nslabs;                       // stage q = (slab q / ntiles, tile q % ntiles)

  if (tid < 2 * kSlabTile)
    *reinterpret_cast<float*>(lds_raw + (tid >> 6) * kBufBytes + kZeroOff + (tid & 63) * 4) = 0.f;

  unsigned row_off[kCopies], row_off_last[kCopies];
  const int last_rows = k - (nslabs - 1) * S;
#pragma unroll
  for (int i = 0; i < kCopies; ++i) {
    const int lrow = (i * NW + wave) * 4 + sub;
    row_off[i] = (unsigned)lrow * (unsigned)n * 4u;
    row_off_last[i] = (unsigned)min(lrow, last_rows - 1) * (unsigned)n * 4u;
  }
  // Slab copies as in the copy-based kernel (issued from assembly, completion covered by the full
  // wait that ends every stage); the stages are copied in order, so source and destination are
  // running scalar state.
  const size_t slab_bytes = (size_t)S * (size_t)n * 4;
  const char* slab_base = reinterpret_cast<const char*>(B);
  int cp_slab = 0, cp_t = 0;
  unsigned cp_dst = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_raw +
                    (unsigned)wave * (4 * kSlabTile * 4);
  unsigned cp_flip = (unsigned)kBufBytes;
  auto copy_stage = [&]() {
    const int piece = piece_start((tile_begin + cp_t) * kSlabTile + l16 * 4, n, 4);
    const unsigned col_off = piece < n ? (unsigned)piece * 4u : 0u;
    const char* base = slab_base;
    const bool last = cp_slab == nslabs - 1;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      const unsigned voff = (last ? row_off_last[i] : row_off[i]) + col_off;
      const unsigned m0v = cp_dst + (unsigned)i * (NW * 4 * kSlabTile * 4);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(m0v), "v"(voff), "s"(base) : "memory", "m0");
    }
    cp_dst += cp_flip;
    cp_flip = 0u - cp_flip;
    if (++cp_t == ntiles) {
      cp_t = 0;
      ++cp_slab;
      slab_base += slab_bytes;
    }
  };

  SlabRow rows[RPG];
#pragma unroll
  for (int j = 0; j < RPG; ++j) {
    const int slot = ((wave * panels + panel) * 4 + sub) * RPG + j;
    rows[j].row = -1;
    rows[j].p_begin = rows[j].row_end = 0;
    if (slot < m) {
      const int r = row_order ? row_order[slot] : slot;
      rows[j].row = r;
      rows[j].p_begin = row_offsets[r];
      rows[j].row_end = row_offsets[r + 1];
    }
    rows[j].p = rows[j].p_begin;
  }
  using Mask = SlabMask<1>;
  // the row's lanes in a wave mask, and the lanes that have met a pair of the slab whose predecessor is not in it
  const unsigned long long row_mask = 0xffffull << (16 * sub);
  const unsigned row_lo = (unsigned)row_mask, row_hi = (unsigned)(row_mask >> 32);
  unsigned long long strays[RPG];
#pragma unroll
  for (int j = 0; j < RPG; ++j) strays[j] = 0;
  float acc[TPW][RPG][4];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < RPG; ++j) acc[t][j][0] = acc[t][j][1] = acc[t][j][2] = acc[t][j][3] = 0.f;

  int cc[RPG][PW];
  float aa[RPG][PW];
  const int last_start = nnz - PW;
  const char* const cbase = reinterpret_cast<const char*>(column_indices);
  const char* const vbase = reinterpret_cast<const char*>(values);
  auto fetch_pairs = [&](int j, int from) {
    if constexpr (PIECES) {
      const unsigned o = (unsigned)min(from + PW * l16, last_start) << 2;
      const SlabPiece<int, PW> c = *reinterpret_cast<const SlabPiece<int, PW>*>(cbase + o);
      const SlabPiece<float, PW> a = *reinterpret_cast<const SlabPiece<float, PW>*>(vbase + o);
#pragma unroll
      for (int e = 0; e < PW; ++e) {
        cc[j][e] = c.v[e];
        aa[j][e] = a.v[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < PW; ++e) {
        const unsigned o = (unsigned)min(from + l16 + 16 * e, nnz - 1) << 2;
        cc[j][e] = *reinterpret_cast<const int*>(cbase + o);
        aa[j][e] = *reinterpret_cast<const float*>(vbase + o);
      }
    }
  };
  auto wait_everything = [&]() { __builtin_amdgcn_s_waitcnt(0); };

  if (nslabs > 0) {
    copy_stage();
#pragma unroll
    for (int j = 0; j < RPG; ++j) fetch_pairs(j, rows[j].p_begin);
  }
  wait_everything();
  __builtin_amdgcn_s_barrier();

  int q = 0;
  for (int s = 0; s < nslabs; ++s) {
    // The scan of the slab: for every row the leading pairs of the look-ahead that lie in it.
    float av[RPG][PW];
    int off[RPG][PW];
    unsigned used[RPG][PW];
    bool over[RPG];                       // wave-uniform
    const int slab_start = s * S;
#pragma unroll
    for (int j = 0; j < RPG; ++j) {
      const int first = rows[j].p + (PIECES ? PW * l16 : l16), left = rows[j].row_end - first;
      if (PIECES && __builtin_amdgcn_ballot_w64(first > last_start && left > 0) != 0)
        slab_piece_shift<PW>(cc[j], aa[j], first - last_start);
      unsigned long long mk[PW];
#pragma unroll
      for (int e = 0; e < PW; ++e) {
        const unsigned rel = (unsigned)(cc[j][e] - slab_start);
        mk[e] = __builtin_amdgcn_ballot_w64(left > (PIECES ? e : 16 * e)) & __builtin_amdgcn_ballot_w64(rel < (unsigned)S);
        if (PIECES && e > 0) strays[j] |= mk[e] & ~mk[e - 1];
        if (!PIECES) strays[j] |= mk[e] & ~(Mask::lane_before(mk[e]) | (e > 0 ? (mk[e - 1] >> 15) & Mask::kFirst : Mask::kFirst));
        rows[j].p += __builtin_popcount((unsigned)mk[e] & row_lo) + __builtin_popcount((unsigned)(mk[e] >> 32) & row_hi);
        used[j][e] = !PIECES || e == 0 ? Mask::used(mk[e]) : 0;
        const bool in = __builtin_amdgcn_inverse_ballot_w64(mk[e]);
        av[j][e] = in ? aa[j][e] : 0.f;
        off[j][e] = in ? (int)(rel * (kSlabTile * 4)) : kZeroOff;
      }
      if (PIECES) strays[j] |= mk[0] & ~(Mask::lane_before(mk[PW - 1]) | Mask::kFirst);
      // every fetched pair of some row lay in the slab: it may hold more of that row
      over[j] = Mask::full(mk[PW - 1]);
      fetch_pairs(j, rows[j].p);
    }
    // One stage per tile: the tile's part of the slab is in LDS, the next part is on its way.
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (t < ntiles) {
        if (q + 1 < stages) copy_stage();
        const char* buf = lds_raw + (q & 1) * kBufBytes;
#pragma unroll
        for (int j = 0; j < RPG; ++j)
          if constexpr (PIECES) {
            const unsigned blocks[1] = {used[j][0]};
            if (blocks[0] != 0) wide_steps<PW>(acc[t][j], av[j], off[j], buf, lane_b, blocks);
          } else {
#pragma unroll
            for (int e = 0; e < PW; ++e)
              if (used[j][e] != 0) slab_steps(acc[t][j], av[j][e], off[j][e], buf, lane_b, 32 - __builtin_clz(used[j][e]));
          }
        // The rare rest of a row that has more pairs in this slab than the look-ahead holds.  (Written out here and in the form
        // with tiles of 128: as a function of both it made the compiler lay out the form with three chunks anew, 1024 x
        // 4096 at 10 %, n = 4096: 113.6 us -> 134.9.)
#pragma unroll
        for (int j = 0; j < RPG; ++j) {
          if (over[j]) {
            int pe = rows[j].p;                 // where the scan stopped (the same in every tile's stage)
            while (true) {
              const int first = pe + kRest * l16, left = rows[j].row_end - first;
              const unsigned o = (unsigned)min(first, nnz - kRest) << 2;
              const SlabPiece<int, kRest> pc = *reinterpret_cast<const SlabPiece<int, kRest>*>(cbase + o);
              const SlabPiece<float, kRest> pa = *reinterpret_cast<const SlabPiece<float, kRest>*>(vbase + o);
              int xc[kRest], xo[kRest];
              float xv[kRest];
#pragma unroll
              for (int e = 0; e < kRest; ++e) {
                xc[e] = pc.v[e];
                xv[e] = pa.v[e];
              }
              if (__builtin_amdgcn_ballot_w64(first > nnz - kRest && left > 0) != 0) slab_piece_shift<kRest>(xc, xv, first - (nnz - kRest));
              unsigned long long mk[kRest];
#pragma unroll
              for (int e = 0; e < kRest; ++e) {
                const unsigned rel = (unsigned)(xc[e] - slab_start);
                mk[e] = __builtin_amdgcn_ballot_w64(left > e) & __builtin_amdgcn_ballot_w64(rel < (unsigned)S);
                if (e > 0) strays[j] |= mk[e] & ~mk[e - 1];
                pe += __builtin_popcount((unsigned)mk[e] & row_lo) + __builtin_popcount((unsigned)(mk[e] >> 32) & row_hi);
                const bool in = __builtin_amdgcn_inverse_ballot_w64(mk[e]);
                xv[e] = in ? xv[e] : 0.f;
                xo[e] = in ? (int)(rel * (kSlabTile * 4)) : kZeroOff;
              }
              strays[j] |= mk[0] & ~(Mask::lane_before(mk[kRest - 1]) | Mask::kFirst);
              const unsigned blocks[1] = {Mask::used(mk[0])};
              if (blocks[0] != 0) wide_steps<kRest>(acc[t][j], xv, xo, buf, lane_b, blocks);
              if (!Mask::full(mk[kRest - 1])) break;
            }
            if (t == ntiles - 1) {              // the slab is done with: the cursor and the look-ahead move on
              rows[j].p = pe;
              fetch_pairs(j, pe);
            }
          }
        }
        wait_everything();
        __builtin_amdgcn_s_barrier();
        ++q;
      }
    }
  }

#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    if (t < ntiles) {
      const int col = piece_start((tile_begin + t) * kSlabTile + l16 * 4, n, 4);
      const bool col_ok = col < n;
#pragma unroll
      for (int j = 0; j < RPG; ++j) {
        if (rows[j].p != rows[j].row_end || (strays[j] & row_mask) != 0)
          slab_gather_row(acc[t][j], rows[j], column_indices, values, B + (col_ok ? col : 0), n);
        if (rows[j].row >= 0 && col_ok) {
          spmm_epilogue<float, 4>(acc[t][j], bias, rows[j].row, relu);
          Pack<float, 4>::store(C + (size_t)rows[j].row * n + col, acc[t][j]);
        }
      }
    }
  }
}

}  // namespace spdl
