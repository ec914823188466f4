// SpMM, slab family for wide outputs, tiles of 128 columns: a lane owns eight of them, 4 l16 .. and 64 + 4 l16 .., so that
// one LDS address serves eight multiply-adds.  Everything else is as in the tile-inner form with tiles of 64: panels of 128
// sparse rows, two rows per 16-lane group, two tiles' accumulators in registers (32 of them), a slab scanned once for
// both; a workgroup may be dealt up to four such pairs, one after the other.  The slab is 128 rows of B by 128 columns, 64 KB as there.
//
// What bounds it: the step (39.6 multiply-adds per clock and CU against 30.8 with four columns per lane, stand-alone) on the
// pairs that the longest of a wave's four rows has in a slab.  Slabs of 128 rows hold half as many, which spreads
// them more (12.8 and 17 at 10 % density, where 256 rows have 25.6 and 32), so blocks are two pairs long instead of four
// and the look-ahead is one, two or four pairs per lane.  4096 x 1024, n = 4096, us per launch, tiles of 64 -> of 128: 10 % 119.7
// -> 118.5, 15 % 181.7 -> 150.4; 3000 x 750 at 15 %, n = 3000: 95.3 -> 84.4; 4804 x 1201 at 23 %, n = 2992: 273 -> 232.  With
// plain multiply-adds on a value that was moved across lanes first: 4 % more at 10 %.
#pragma once
#include "common.hpp"
#include "spmm_slab.hpp"

namespace spdl {

constexpr int kWideTile = 128;
constexpr int kWideRowBytes = kWideTile * 4;
constexpr int kWideS = 128;            // rows of B per slab
constexpr int kWideRows = 128;         // sparse rows per workgroup
constexpr int kWideTiles = 2;          // tiles that a workgroup has in registers at a time (it may be dealt several pairs)
constexpr int kWideLdsBytes = 2 * (kWideS + 1) * kWideRowBytes;

// Two pairs of every 16-lane group: two LDS addresses and four 128-bit reads (columns 4 l16 .. and 64 + 4 l16 ..), then
// sixteen multiply-adds.
template <int PW, int BLOCK>
__device__ __forceinline__ void wide8_load(f32x4 (&bq)[4], const int (&off)[PW], const char* buf, int lane_b) {
  constexpr int P = 2 * BLOCK;
  const char* b0 = buf + __builtin_amdgcn_update_dpp(0, off[(P + 0) % PW], 0x150 + (P + 0) / PW, 0xf, 0xf, false) + lane_b;
  const char* b1 = buf + __builtin_amdgcn_update_dpp(0, off[(P + 1) % PW], 0x150 + (P + 1) / PW, 0xf, 0xf, false) + lane_b;
  bq[0] = *reinterpret_cast<const f32x4*>(b0);
  bq[1] = *reinterpret_cast<const f32x4*>(b0 + 256);
  bq[2] = *reinterpret_cast<const f32x4*>(b1);
  bq[3] = *reinterpret_cast<const f32x4*>(b1 + 256);
}
template <int PW, int BLOCK>
__device__ __forceinline__ void wide8_fma(float (&acc)[8], const float (&av)[PW], const f32x4 (&bq)[4]) {
  constexpr int P = 2 * BLOCK;
#define SPDL_F(ACC, AV, B, LANE) "v_fmac_f32_dpp %" #ACC ", %" #AV ", %" #B " row_newbcast:%" #LANE " row_mask:0xf bank_mask:0xf\n\t"
#define SPDL_F8(AV, B0, B1, B2, B3, B4, B5, B6, B7, LANE)                                                          \
  SPDL_F(0, AV, B0, LANE) SPDL_F(1, AV, B1, LANE) SPDL_F(2, AV, B2, LANE) SPDL_F(3, AV, B3, LANE)                    \
  SPDL_F(4, AV, B4, LANE) SPDL_F(5, AV, B5, LANE) SPDL_F(6, AV, B6, LANE) SPDL_F(7, AV, B7, LANE)
#define SPDL_F16(PRE)                                                                                                \
  asm volatile(PRE SPDL_F8(8, 10, 11, 12, 13, 14, 15, 16, 17, 26) SPDL_F8(9, 18, 19, 20, 21, 22, 23, 24, 25, 27)     \
               : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]),     \
                 "+v"(acc[7])                                                                                        \
               : "v"(av[(P + 0) % PW]), "v"(av[(P + 1) % PW]),                                                       \
                 "v"(bq[0].x), "v"(bq[0].y), "v"(bq[0].z), "v"(bq[0].w), "v"(bq[1].x), "v"(bq[1].y),                 \
                 "v"(bq[1].z), "v"(bq[1].w), "v"(bq[2].x), "v"(bq[2].y), "v"(bq[2].z), "v"(bq[2].w),                 \
                 "v"(bq[3].x), "v"(bq[3].y), "v"(bq[3].z), "v"(bq[3].w), "n"((P + 0) / PW), "n"((P + 1) / PW))
  if constexpr (P < PW) SPDL_F16("s_nop 1\n\t");
  else SPDL_F16("");
#undef SPDL_F16
#undef SPDL_F8
#undef SPDL_F
}
template <int PW, int BLOCK>
__device__ __forceinline__ void wide8_blocks(float (&acc)[8], const float (&av)[PW], const int (&off)[PW], const char* buf,
                                             int lane_b, const unsigned (&used)[(PW + 1) / 2], f32x4 (&now)[4], f32x4 (&next)[4]) {
  constexpr int kBlocks = 8 * PW;
  wide8_fma<PW, BLOCK>(acc, av, now);
  if constexpr (BLOCK + 1 < kBlocks) {
    if ((used[(2 * (BLOCK + 1) % PW) / 2] >> (2 * (BLOCK + 1) / PW)) != 0) {
      if constexpr (BLOCK + 2 < kBlocks) wide8_load<PW, BLOCK + 2>(now, off, buf, lane_b);
      wide8_blocks<PW, BLOCK + 1>(acc, av, off, buf, lane_b, used, next, now);
    }
  }
}
template <int PW>
__device__ __forceinline__ void wide8_steps(float (&acc)[8], const float (&av)[PW], const int (&off)[PW], const char* buf,
                                            int lane_b, const unsigned (&used)[(PW + 1) / 2]) {
  f32x4 bx[4], by[4];
  wide8_load<PW, 0>(bx, off, buf, lane_b);
  wide8_load<PW, 1>(by, off, buf, lane_b);
  wide8_blocks<PW, 0>(acc, av, off, buf, lane_b, used, bx, by);
}

template <int PW>
__global__ __launch_bounds__(1024) void spmm_slab_wide_kernel(
    int m, int k, int n, int nnz, int tiles_n, int tiles_per_wg, int panels,
    const int* __restrict__ row_offsets, const int* __restrict__ column_indices,
    const float* __restrict__ values, const int* __restrict__ row_order, const float* __restrict__ B,
    float* __restrict__ C, const float* __restrict__ bias, int relu, int tiles_first) {
  constexpr int NW = 16, S = kWideS, RPG = kWideRows / 64, TPW = kWideTiles;
  // pairs per lane and round of a row that has more in a slab than the look-ahead (as many as there are registers for)
  constexpr int kRest = PW == 4 ? 1 : 2;
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  constexpr int kBufBytes = (S + 1) * kWideRowBytes;
  constexpr int kZeroOff = S * kWideRowBytes;
  constexpr int kCopies = S / (2 * NW);

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
  int tile_begin = tile_group * tiles_per_wg;
  const int tile_end = min(tiles_n, tile_begin + tiles_per_wg);
  int ntiles = min(tile_end - tile_begin, TPW);             // of the tiles that are being computed
  const int nslabs = nnz < 4 ? 0 : (k + S - 1) / S;       // (rows that are not walked are gathered at the end)
  const int stages = (tile_end - tile_begin) * nslabs;      // by TPW tiles, by slabs, by tiles

  if (tid < 2 * kWideTile)
    *reinterpret_cast<float*>(lds_raw + (tid >> 7) * kBufBytes + kZeroOff + (tid & 127) * 4) = 0.f;

  // Slab copies as in the tile-inner form: copy i of wave w fills slab rows (i*NW + w)*2 and + 1, 32 pieces of a row each.
  unsigned row_off[kCopies], row_off_last[kCopies];
  const int last_rows = k - (nslabs - 1) * S;
#pragma unroll
  for (int i = 0; i < kCopies; ++i) {
    const int lrow = (i * NW + wave) * 2 + (lane >> 5);
    row_off[i] = (unsigned)lrow * (unsigned)n * 4u;
    row_off_last[i] = (unsigned)min(lrow, last_rows - 1) * (unsigned)n * 4u;
  }
  const size_t slab_bytes = (size_t)S * (size_t)n * 4;
  const char* slab_base = reinterpret_cast<const char*>(B);
  int cp_slab = 0, cp_t = 0, cp_begin = tile_begin, cp_tiles = ntiles;
  unsigned cp_dst = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_raw + (unsigned)wave * (2 * kWideRowBytes);
  unsigned cp_flip = (unsigned)kBufBytes;
  auto copy_stage = [&]() {
    const int piece = piece_start((cp_begin + cp_t) * kWideTile + (lane & 31) * 4, n, 4);
    const unsigned col_off = piece < n ? (unsigned)piece * 4u : 0u;
    const char* base = slab_base;
    const bool last = cp_slab == nslabs - 1;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      const unsigned voff = (last ? row_off_last[i] : row_off[i]) + col_off;
      const unsigned m0v = cp_dst + (unsigned)i * (NW * 2 * kWideRowBytes);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(m0v), "v"(voff), "s"(base) : "memory", "m0");
    }
    cp_dst += cp_flip;
    cp_flip = 0u - cp_flip;
    if (++cp_t == cp_tiles) {
      cp_t = 0;
      slab_base += slab_bytes;
      if (++cp_slab == nslabs) {                            // the next tiles' first slab
        cp_slab = 0;
        slab_base = reinterpret_cast<const char*>(B);
        cp_begin += TPW;
        cp_tiles = min(tile_end - cp_begin, TPW);
      }
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
  const int lane_pair = l16 * PW;
  auto of_row = [&](unsigned long long mk) __attribute__((always_inline)) {
    return __builtin_popcount((unsigned)mk & row_lo) + __builtin_popcount((unsigned)(mk >> 32) & row_hi);
  };
  float acc[TPW][RPG][8];

  int cc[RPG][PW];
  float aa[RPG][PW];
  const int last_start = nnz - PW;
  const char* const cbase = reinterpret_cast<const char*>(column_indices);
  const char* const vbase = reinterpret_cast<const char*>(values);
  auto fetch_pairs = [&](int j, int from) {
    const unsigned o = (unsigned)min(from + lane_pair, last_start) << 2;
    const SlabPiece<int, PW> c = *reinterpret_cast<const SlabPiece<int, PW>*>(cbase + o);
    const SlabPiece<float, PW> a = *reinterpret_cast<const SlabPiece<float, PW>*>(vbase + o);
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      cc[j][e] = c.v[e];
      aa[j][e] = a.v[e];
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
  clocks.lap(kPhaseSetup);

  int q = 0;
  for (; tile_begin < tile_end; tile_begin += TPW) {
    ntiles = min(tile_end - tile_begin, TPW);
    const bool again = tile_begin + TPW < tile_end;           // other tiles follow: the rows once more
#pragma unroll
    for (int j = 0; j < RPG; ++j) {
      rows[j].p = rows[j].p_begin;
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int v = 0; v < 8; ++v) acc[t][j][v] = 0.f;
    }
    for (int s = 0; s < nslabs; ++s) {
      float av[RPG][PW];
      int off[RPG][PW];
      unsigned used[RPG][(PW + 1) / 2];
      bool over[RPG];                       // wave-uniform
      const int slab_start = s * S;
      // (a use of the youngest pair register, so that the wait for the pairs is placed here, where it is satisfied)
      asm volatile("v_mov_b32 %0, %0" : "+v"(aa[RPG - 1][PW - 1]));
      if (q + 1 < stages) copy_stage();
      clocks.lap(kPhaseIssue);
#pragma unroll
      for (int j = 0; j < RPG; ++j) {
        const int first = rows[j].p + lane_pair, left = rows[j].row_end - first;
        if (__builtin_amdgcn_ballot_w64(first > last_start && left > 0) != 0) slab_piece_shift<PW>(cc[j], aa[j], first - last_start);
        unsigned long long mk[PW];
#pragma unroll
        for (int e = 0; e < PW; ++e) {
          const unsigned rel = (unsigned)(cc[j][e] - slab_start);
          mk[e] = __builtin_amdgcn_ballot_w64(left > e) & __builtin_amdgcn_ballot_w64(rel < (unsigned)S);
          if (e > 0) strays[j] |= mk[e] & ~mk[e - 1];
          if (e % 2 == 0) used[j][e / 2] = Mask::used(mk[e]);
          rows[j].p += of_row(mk[e]);
          const bool in = __builtin_amdgcn_inverse_ballot_w64(mk[e]);
          av[j][e] = in ? aa[j][e] : 0.f;
          off[j][e] = in ? (int)(rel * kWideRowBytes) : kZeroOff;
        }
        strays[j] |= mk[0] & ~(Mask::lane_before(mk[PW - 1]) | Mask::kFirst);
        over[j] = Mask::full(mk[PW - 1]);
        fetch_pairs(j, again && s == nslabs - 1 && !over[j] ? rows[j].p_begin : rows[j].p);
      }
      clocks.lap(kPhaseScan);
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        if (t < ntiles) {
          if (t > 0 && q + 1 < stages) copy_stage();
          const char* buf = lds_raw + (q & 1) * kBufBytes;
          clocks.lap(kPhaseIssue);
#pragma unroll
          for (int j = 0; j < RPG; ++j)
            if (used[j][0] != 0) wide8_steps<PW>(acc[t][j], av[j], off[j], buf, lane_b, used[j]);
          clocks.lap(kPhaseSteps);
          // The rare rest of a row that has more pairs in this slab than the look-ahead holds.
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
                  pe += of_row(mk[e]);
                  const bool in = __builtin_amdgcn_inverse_ballot_w64(mk[e]);
                  xv[e] = in ? xv[e] : 0.f;
                  xo[e] = in ? (int)(rel * kWideRowBytes) : kZeroOff;
                }
                strays[j] |= mk[0] & ~(Mask::lane_before(mk[kRest - 1]) | Mask::kFirst);
                const unsigned xu[1] = {Mask::used(mk[0])};
                if (xu[0] != 0) wide8_steps<kRest>(acc[t][j], xv, xo, buf, lane_b, xu);
                if (!Mask::full(mk[kRest - 1])) break;
              }
              if (t == ntiles - 1) {              // the slab is done with: the cursor and the look-ahead move on
                rows[j].p = pe;
                fetch_pairs(j, again && s == nslabs - 1 ? rows[j].p_begin : pe);
              }
            }
          }
          wait_everything();
          clocks.lap(kPhaseWait);
          __builtin_amdgcn_s_barrier();
          clocks.lap(kPhaseBarrier);
          ++q;
        }
      }
    }

#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (t < ntiles) {
#pragma unroll
        for (int j = 0; j < RPG; ++j) {
          const bool redo = rows[j].p != rows[j].row_end || (strays[j] & row_mask) != 0;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int col = piece_start((tile_begin + t) * kWideTile + h * 64 + l16 * 4, n, 4);
            const bool col_ok = col < n;
            float sum[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[v] = acc[t][j][4 * h + v];
            if (redo) slab_gather_row(sum, rows[j], column_indices, values, B + (col_ok ? col : 0), n);
            if (rows[j].row >= 0 && col_ok) {
              spmm_epilogue<float, 4>(sum, bias, rows[j].row, relu);
              Pack<float, 4>::store(C + (size_t)rows[j].row * n + col, sum);
            }
          }
        }
      }
    }
  }
  clocks.lap(kPhaseRest);
  clocks.store(blockIdx.x * NW + wave);
}

}  // namespace spdl
