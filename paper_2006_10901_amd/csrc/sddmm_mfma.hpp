// SDDMM in mixed precision on the matrix cores (paper Sec. "Mixed Precision": fp16 operands,
// fp32 accumulation).  On this chip the dense fp16 matrix rate is some thirty times the fp32
// vector rate, so for the moderately sparse matrices of deep learning it is cheaper to compute
// a whole 32x32 block of L R^T with MFMA and keep only the entries A stores there than to
// gather one row of R per stored entry.  The contraction runs over n, which is the contiguous
// dimension of both row-major operands.
//
// A workgroup owns one 64x64 block of A's index space.  Which stored entries fall into the
// block: for each of its 64 rows a binary search gives the first entry with column >= c0 and
// the first with column >= c0 + 64.  Whatever the column order inside a row, the ranges of
// consecutive blocks cover the row (the first block starts at the row start, the last ends at
// the row end), and every entry of a range is produced by the workgroup that owns the range: from
// the block if its column lies inside it, else (rows that are not ascending) by a plain dot
// product.  Dense work is the same for every block, so row lengths do not unbalance anything.
//
// Any n from 8 on and any alignment (see the two forms below).
#pragma once
#include "common.hpp"

namespace spdl {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Dot product of two rows of length n by one lane (entries whose column lies outside the block
// that owns their range; only rows that are not ascending have them).
__device__ __attribute__((noinline)) float sddmm_lane_dot(const _Float16* __restrict__ l,
                                                          const _Float16* __restrict__ r, int n) {
  float acc = 0.f;
  int j = 0;
  for (; j + 8 <= n; j += 8) {
    float a[8], b[8];
    Pack<_Float16, 8>::load(l + j, a);
    Pack<_Float16, 8>::load(r + j, b);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc = __builtin_fmaf(a[t], b[t], acc);
  }
  for (; j < n; ++j) acc = __builtin_fmaf((float)l[j], (float)r[j], acc);
  return acc;
}

constexpr int kSmPieces = 16;                          // pieces of 8 columns of L and R resident per stage
constexpr int kSmRing = 4;                             // stages resident in LDS (three being fetched)
constexpr int kSmOperandBytes = 64 * kSmPieces * 16;   // 64 rows of one operand
constexpr int kSmStageBytes = 2 * kSmOperandBytes;     // L rows, then R rows
constexpr int kSmThreads = 576;                        // waves 0-3 multiply, 4-7 copy, 8 looks for the entries
constexpr int kSmAhead = 16;                           // column indices of a row fetched ahead
constexpr int kSmPartBytes = 4 * 64 * 65 * 4;          // the waves' partial blocks, in the ring's place; ranges and indices behind
constexpr int kSddmmMfmaLdsBytes = kSmRing * kSmStageBytes;

// Block id -> (tile_i, tile_c).  Consecutive workgroup ids go round-robin to the 8 XCDs, each with its
// own L2; the workgroups that an XCD has at work at a time advance through n together and share the
// rows of L and R they stream.  XCD x gets half x/4 of the rows and quarter x%4 of the columns of the
// block grid if those are no more blocks than it has compute units (all at work at once: the fewer
// different rows the better).  Otherwise every XCD gets an equal run of the blocks, in strips walked from
// top to bottom, a strip a quarter of the columns wide, but no wider than what keeps its rows of R in half of an
// L2 meanwhile: halves and quarters leave XCDs without work where the grid does not come out even (41 by
// 5 blocks, n = 965: 20 us against 11), and wide ones fetch R again for every row of blocks (5053 x 7246, n = 1968:
// 445 us against 395).
__host__ __device__ __forceinline__ int sddmm_mfma_region(int tiles_m, int tiles_k) {   // blocks of an XCD, 0: runs
  const int TI = (tiles_m + 1) >> 1, TC = (tiles_k + 3) >> 2;
  return TI <= 32 && TC <= 32 && TI * TC <= 32 ? TI * TC : 0;
}
__host__ __device__ __forceinline__ int sddmm_mfma_grid(int tiles_m, int tiles_k) {
  const int region = sddmm_mfma_region(tiles_m, tiles_k);
  return 8 * (region ? region : (tiles_m * tiles_k + 7) / 8);
}
__device__ __forceinline__ bool sddmm_mfma_tile(int bid, int tiles_m, int tiles_k, int n, int& tile_i, int& tile_c) {
  const int xcd = bid & 7, local = bid >> 3;
  const int TC = (tiles_k + 3) >> 2;
  if (sddmm_mfma_region(tiles_m, tiles_k)) {
    tile_i = (xcd >> 2) * ((tiles_m + 1) >> 1) + local / TC;
    tile_c = (xcd & 3) * TC + local % TC;
    return tile_i < tiles_m && tile_c < tiles_k;
  }
  const int blocks = tiles_m * tiles_k;
  const int pos = xcd * ((blocks + 7) >> 3) + local;
  if (pos >= blocks) return false;
  const int strip_width = min(TC, max(4, (1 << 14) / n));      // 2 MB of rows of R
  const int strip = pos / (strip_width * tiles_m), at = pos - strip * strip_width * tiles_m;
  const int width = min(strip_width, tiles_k - strip_width * strip);
  tile_i = at / width;
  tile_c = strip_width * strip + at - tile_i * width;
  return true;
}

// One workgroup owns one 64x64 block of A's index space.  The contraction runs over n, 128 columns
// per stage.  Waves 4-7 bring the 64 rows of L and of R of the block in by direct-to-LDS loads:
// sixteen lanes read the 256 contiguous bytes of one row, and each lane fetches the piece that belongs
// at its place in a swizzled layout (piece p of row r at slot p xor (r mod 16)), so that the sixteen
// lanes of an operand read, which want the same piece of sixteen rows, hit sixteen different bank
// groups.  Three stages are in flight while waves 0-3 multiply one; one barrier per stage.  Every
// multiplying wave accumulates the whole 64x64 block over its quarter of each stage: every byte of a
// stage is then read from LDS once, by one wave, where a split of the block into four 32x32 tiles reads
// it twice (LDS reads and the copies' LDS writes share one port).  Wave 8 finds the block's entries
// meanwhile, one step of its binary searches in every other stage.  At the end the partial blocks go to
// LDS and the threads pick out the positions A stores.
//
// What bounds it is not established.  A CU's vector memory path takes 16 clocks or a little more for a copy of 1 KB, some
// 0.27 us for the 32 KB of a stage, against 0.13 us of MFMA and 0.25 us of LDS reads and writes; the 25 stages of
// n = 3136 are 6.7 us on that path, of the 14 that the launch takes.  When the
// waves that multiply issue the copies as well (as this kernel did), they stand in that queue first and
// read and multiply after it, with the memory path idle (1024 x 1024, n = 3136:
// 20.1 us instead of 15.6).  Clocks inside the kernel: the copying waves hand over copies 50 % of their time, wait for the
// oldest stage 17 % and for the multiplying waves to release one 28 %; the multiplying waves multiply 37 % and wait 55 %.
// (Measured and dropped: operands loaded from memory straight into the registers of 16x16x32 MFMAs,
// without LDS: sixteen consecutive lanes then read sixteen rows, which the memory path takes one by
// one, 64 clocks per load instead of 16: 31 us.)
//
// ODD = false: every row starts at an address that is a multiple of four, what a copy needs: n is even
// and so are the operands' first addresses, in elements.  The last n % 8 columns, which fill no piece,
// are one more MFMA step at the end, its operands loaded element by element.  ODD = true, anything else: a row that starts two
// bytes past a multiple of four is copied from there, one element early, and the fragments are moved
// into place when they are read, the last element from the piece that follows.  The stages then
// overlap by one piece (120 columns each), and the last 8 .. 15 columns are the step at the end.
template <bool ODD>
__global__ __launch_bounds__(kSmThreads) void sddmm_mfma_kernel(
    int m, int k, int n, int tiles_k, const int* __restrict__ row_offsets,
    const int* __restrict__ column_indices, const _Float16* __restrict__ L, const _Float16* __restrict__ R,
    _Float16* __restrict__ out, const _Float16* __restrict__ scale) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  float (*part)[64][65] = reinterpret_cast<float (*)[64][65]>(lds_raw);           // [wave][row][column], after the loop
  int (*bound)[64] = reinterpret_cast<int (*)[64]>(lds_raw + kSmPartBytes);              // [0]: range start, [1]: end
  int (*ahead)[64] = reinterpret_cast<int (*)[64]>(lds_raw + kSmPartBytes + 2 * 64 * 4); // [entry][row]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  int tile_i, tile_c;
  if (!sddmm_mfma_tile(blockIdx.x, (m + 63) >> 6, tiles_k, n, tile_i, tile_c)) return;   // whole workgroup, before any barrier
  const int i0 = tile_i * 64;
  const int c0 = tile_c * 64;
  PhaseClocks clocks;
  clocks.start();

  constexpr int kAdvance = ODD ? kSmPieces - 1 : kSmPieces;         // pieces from stage to stage
  const int pieces = ODD ? max(0, n / 8 - 1) : n / 8;               // multiplied in stages; the rest at the end
  const int stages = (pieces + kAdvance - 1) / kAdvance;

  if (wave < 4) {
    const int r = lane & 31;
    const int half = lane >> 5;
    const _Float16* lrow[2];
    const _Float16* rrow[2];
    bool lodd = false, rodd = false;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      lrow[i] = L + (size_t)min(i0 + 32 * i + r, m - 1) * n;
      rrow[i] = R + (size_t)min(c0 + 32 * i + r, k - 1) * n;
    }
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[i][j][t] = 0.f;
    // the columns past the last piece: fetched now, multiplied after the loop, by one of the waves
    f16x8 at[2], bt[2];
    const bool tail = wave == 0 && 8 * pieces < n;
    if (tail) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int col = 8 * pieces + 8 * half + t;
          at[i][t] = col < n ? lrow[i][col] : (_Float16)0.f;
          bt[i][t] = col < n ? rrow[i][col] : (_Float16)0.f;
        }
    }
    if (ODD) {                                         // (rows 32 apart, or clamped: the same parity or never looked at)
      lodd = ((uintptr_t)(L + (size_t)(i0 + r) * n) & 2) != 0;
      rodd = ((uintptr_t)(R + (size_t)(c0 + r) * n) & 2) != 0;
    }
    const unsigned lshift = lodd ? 16u : 0u, rshift = rodd ? 16u : 0u;
    // operand fragments: lane (r, half) reads piece 4*wave + 2*step + half of rows r and 32 + r of L
    // and of R, from their swizzled slots (rows r and 32 + r share r % 16)
    const int a_row_off = r * (kSmPieces * 16), b_row_off = kSmOperandBytes + r * (kSmPieces * 16);
    constexpr int kBlock = 32 * kSmPieces * 16;
    auto fragment = [&](const char* row, int slot, int next, unsigned shift) __attribute__((always_inline)) {
      const u32x4 w = *reinterpret_cast<const u32x4*>(row + slot);
      u32x4 v = w;
      if (ODD) {
        const unsigned after = *reinterpret_cast<const unsigned*>(row + next);
        const unsigned w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
        v[0] = __builtin_amdgcn_alignbit(w1, w0, shift);
        v[1] = __builtin_amdgcn_alignbit(w2, w1, shift);
        v[2] = __builtin_amdgcn_alignbit(w3, w2, shift);
        v[3] = __builtin_amdgcn_alignbit(after, w3, shift);
      }
      return v;
    };
    clocks.lap(kPhaseSetup);
    for (int s = 0; s < stages; ++s) {
      __syncthreads();                                 // stage s has arrived
      clocks.lap(kPhaseBarrier);
      const char* buf = lds_raw + (s % kSmRing) * kSmStageBytes;
      const bool ragged = (s + 1) * kAdvance > pieces;
#pragma unroll
      for (int step = 0; step < 2; ++step) {
        const int p = 4 * wave + 2 * step + half;
        const int slot = (p ^ (r & 15)) << 4, next = ((p + 1) ^ (r & 15)) << 4 & (kSmPieces * 16 - 1);
        u32x4 a0 = fragment(buf + a_row_off, slot, next, lshift);
        u32x4 a1 = fragment(buf + a_row_off + kBlock, slot, next, lshift);
        u32x4 b0 = fragment(buf + b_row_off, slot, next, rshift);
        u32x4 b1 = fragment(buf + b_row_off + kBlock, slot, next, rshift);
        // pieces past the last, and the one that overlaps the next stage (both operands: 0 * Inf)
        if ((ragged && s * kAdvance + p >= pieces) || (ODD && p == kAdvance))
          a0 = a1 = b0 = b1 = u32x4{0u, 0u, 0u, 0u};
        const f16x8 x0 = __builtin_bit_cast(f16x8, a0), x1 = __builtin_bit_cast(f16x8, a1);
        const f16x8 y0 = __builtin_bit_cast(f16x8, b0), y1 = __builtin_bit_cast(f16x8, b1);
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0, y0, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0, y1, acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1, y0, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1, y1, acc[1][1], 0, 0, 0);
      }
      clocks.lap(kPhaseSteps);
    }
    if (tail) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(at[i], bt[j], acc[i][j], 0, 0, 0);
    }
    clocks.lap(kPhaseRest);
    __syncthreads();                                   // the ring is free: it now holds the four partial blocks
    clocks.lap(kPhaseBarrier);
    // Register t of lane (r, half) in acc[i][j] is element (32*i + 8*(t/4) + 4*half + t%4, 32*j + r).
    float (*mine)[65] = part[wave];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < 16; ++t) mine[32 * i + 8 * (t / 4) + 4 * half + (t % 4)][32 * j + r] = acc[i][j][t];
  } else if (wave < 8) {
    // A stage is 32 copies of 1 KB (4 rows each): waves 4 and 5 bring L, 6 and 7 bring R.  Copy j of a
    // wave fills rows 4*(8*(w%2) + j) .. +3 of its operand; lane t brings row t/16 of those, the piece
    // (t%16) xor (row%16), to slot t%16.  Rows past the end of either matrix are clamped (their results
    // are never looked at), pieces past the last become the stage's first (zeroed when they are read).
    // The copies are issued from inline assembly and waited for with explicit counts: they are the only
    // vector-memory operations of these waves and complete in the order issued.
    const _Float16* operand = wave < 6 ? L : R;
    const int row_base = wave < 6 ? i0 : c0, row_limit = (wave < 6 ? m : k) - 1 - row_base;
    const int fetched = ODD ? pieces + 1 : pieces;
    const char* first = reinterpret_cast<const char*>(operand + (size_t)row_base * n);
    unsigned voff[8];
    int vpiece[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int row = 4 * (8 * (wave & 1) + j) + (lane >> 4);
      vpiece[j] = (lane & 15) ^ (row & 15);
      voff[j] = (unsigned)min(row, row_limit) * (unsigned)n * 2u;
      if (ODD) voff[j] += 2u - ((unsigned)((uintptr_t)first + voff[j]) & 2u);
    }
    if (ODD) first -= 2;
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_raw +
                              (unsigned)(((wave - 4) >> 1) * kSmOperandBytes + (wave & 1) * (kSmOperandBytes / 2));
    auto issue_stage = [&](int s) __attribute__((always_inline)) {
      const char* base = first + (size_t)s * (kAdvance * 16);
      const unsigned dst = lds_base + (unsigned)((s % kSmRing) * kSmStageBytes);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bool in = s * kAdvance + vpiece[j] < fetched;
        const unsigned off = voff[j] + (in ? (unsigned)vpiece[j] * 16u : 0u);
        const unsigned m0v = dst + (unsigned)j * 1024u;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(m0v), "v"(off), "s"(base) : "memory", "m0");
      }
    };
    clocks.lap(kPhaseSetup);
#pragma unroll
    for (int s = 0; s < kSmRing - 1; ++s)
      if (s < stages) issue_stage(s);
    clocks.lap(kPhaseIssue);
    for (int s = 0; s < stages; ++s) {
      // stage s has arrived when at most the copies of the (up to two) later stages are outstanding
      if (s + 2 < stages) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
      else if (s + 1 < stages) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      clocks.lap(kPhaseWait);
      __syncthreads();                                 // ... and stage s-1 is consumed
      clocks.lap(kPhaseBarrier);
      if (s + kSmRing - 1 < stages) issue_stage(s + kSmRing - 1);
      clocks.lap(kPhaseIssue);
    }
    __syncthreads();
    clocks.lap(kPhaseBarrier);
  } else {
    // Range of row i0 + lane that this block owns, and its first column indices: one step of the searches
    // for both ends in every other stage (a chain of dependent loads), what is left after the loop.
    // (Steps that look at seven places instead of one: the chain is shorter, but each of the loads takes the
    // memory path 64 clocks, a row per lane: 0.3 .. 1 us slower where few stages hide it.)
    const int row = i0 + lane;
    int rs = 0, re = 0;
    if (row < m) {
      rs = row_offsets[row];
      re = row_offsets[row + 1];
    }
    int lo[2] = {rs, rs}, hi[2] = {re, re}, probe[2] = {0, 0};
    auto look = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int w = 0; w < 2; ++w)
        if (lo[w] < hi[w]) probe[w] = column_indices[(lo[w] + hi[w]) >> 1];
    };
    auto halve = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int w = 0; w < 2; ++w)
        if (lo[w] < hi[w]) {
          const int mid = (lo[w] + hi[w]) >> 1;
          if (probe[w] < c0 + 64 * w) lo[w] = mid + 1; else hi[w] = mid;
        }
    };
    auto searching = [&]() { return __builtin_amdgcn_ballot_w64(lo[0] < hi[0] || lo[1] < hi[1]) != 0; };
    look();
    clocks.lap(kPhaseSetup);
    for (int s = 0; s < stages; ++s) {
      __syncthreads();
      clocks.lap(kPhaseBarrier);
      if ((s & 1) && searching()) {
        halve();
        look();
      }
      clocks.lap(kPhaseScan);
    }
    while (searching()) {
      halve();
      look();
    }
    if (tile_c == 0) lo[0] = rs;
    if (tile_c == tiles_k - 1) lo[1] = re;
    int pre[kSmAhead];
#pragma unroll
    for (int e = 0; e < kSmAhead; ++e) pre[e] = lo[0] + e < lo[1] ? column_indices[lo[0] + e] : 0;
    clocks.lap(kPhaseScan);
    __syncthreads();
    clocks.lap(kPhaseBarrier);
    bound[0][lane] = lo[0];
    bound[1][lane] = lo[1];
#pragma unroll
    for (int e = 0; e < kSmAhead; ++e) ahead[e][lane] = pre[e];
  }
  clocks.lap(kPhaseRest);
  __syncthreads();
  clocks.lap(kPhaseBarrier);
  if (tid >= 512) {
    clocks.store(blockIdx.x * (kSmThreads / 64) + wave);
    return;
  }

  // Eight threads per row take alternate entries of its range.
  const int rr = tid >> 3;
  const int row = i0 + rr;
  const int b0 = bound[0][rr], b1 = max(b0, bound[1][rr]);
  for (int p = b0 + (tid & 7); p < b1; p += 8) {
    const int c = p - b0 < kSmAhead ? ahead[p - b0][rr] : column_indices[p];
    const unsigned cc = (unsigned)(c - c0);
    float val;
    if (cc < 64u) val = (part[0][rr][cc] + part[1][rr][cc]) + (part[2][rr][cc] + part[3][rr][cc]);
    else val = sddmm_lane_dot(L + (size_t)row * n, R + (size_t)c * n, n);
    sddmm_store<_Float16>(out, scale, p, val);
  }
  clocks.lap(kPhaseRest);
  clocks.store(blockIdx.x * (kSmThreads / 64) + wave);
}

}  // namespace spdl
