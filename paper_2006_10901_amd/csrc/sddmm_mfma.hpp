// SDDMM in mixed precision on the matrix cores (paper Sec. "Mixed Precision": fp16 operands,
// fp32 accumulation).  On this chip the dense fp16 matrix rate is some thirty times the fp32
// vector rate, so for the moderately sparse matrices of deep learning it is cheaper to compute
// a whole 32x32 block of L R^T with MFMA and keep only the entries A stores there than to
// gather one row of R per stored entry.  The contraction runs over n, which is the contiguous
// dimension of both row-major operands.
//
// A workgroup owns one block of A's index space, 64x64 or smaller (SmBlock).  Which stored entries fall into the
// block: for each of its rows a binary search gives the first entry with column >= c0 and
// the first with column >= c0 + the block's width.  Whatever the column order inside a row, the ranges of
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

constexpr int kSmThreads = 576;                        // waves 0-3 multiply, 4-7 copy, 8 looks for the entries
constexpr int kSmAhead = 16;                           // column indices of a row fetched ahead

// A block of BM sparse rows and BN columns of A, P pieces of 8 columns of L and R per stage.
template <int BM, int BN, int P>
struct SmBlock {
  static constexpr int kStageBytes = (BM + BN) * P * 16;               // L rows, then R rows
  static constexpr int kCopies = (BM + BN) * P / 256, kCopiesL = BM * P / 256;   // copies of 1 KB per copying wave and stage, of L among them
  static constexpr int kRing = 147456 / kStageBytes;   // stages resident in LDS (all but one being fetched)
  static constexpr int kPartBytes = 4 * BM * (BN + 1) * 4;             // the waves' partial blocks, in the ring's place; ranges and indices behind
  static constexpr int kLdsBytes = kRing * kStageBytes;
  static_assert(kPartBytes + (2 + kSmAhead) * BM * 4 <= kLdsBytes && kRing >= 3, "LDS");
};

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

// The contraction runs over n, P pieces of eight columns per
// stage.  Waves 4-7 bring the block's rows of L and of R in by direct-to-LDS loads:
// P lanes read the contiguous bytes of one row, and each lane fetches the piece that belongs
// at its place in a swizzled layout (piece p of row r at slot p xor (r mod 16)), so that the sixteen
// lanes of an operand read, which want the same piece of sixteen rows, hit sixteen different bank
// groups.  All stages of the ring but one are in flight while waves 0-3 multiply that one; one barrier per stage.  Every
// multiplying wave accumulates the whole block over its quarter of each stage: every byte of a
// stage is then read from LDS once, by one wave, where a split of a 64x64 block into four 32x32 tiles reads
// it twice (LDS reads and the copies' LDS writes share one port).  Wave 8 finds the block's entries
// meanwhile, one or two steps of its binary searches in every other stage.  At the end the partial blocks go to
// LDS and the threads pick out the positions A stores.
//
// What bounds it: 3 to 4 us of set-up, first copies, searches and sampling, and the stages: what is in flight, 96 KB, takes 1.2 .. 1.6 us
// to come, and a stage costs 0.13 us whatever its size.  (A CU's vector memory path takes 16 clocks or a little more for a copy of 1 KB, some
// 0.27 us for 32 KB.)  Hence long stages, 256 columns, where the block's rows are few enough for a ring of them, and small blocks where that
// many workgroups find a compute unit each.  (us: 304 x 744, n = 2880, 32x32 blocks, stages of 64 / 128 / 256 columns 12.2 / 11.1 / 9.8; 894 x 407, n =
// 2544, 64x32, 128 / 256: 13.8 / 12.7; before, in 64x64 blocks with single search steps, 13.3 and 15.9.  64x64 in a ring of nine stages of 64: 15.8 us
// for 1024 x 1024, n = 3136, 14.9 in one of four of 128.  Eight multiplying waves in place of four: 5 .. 10 % slower throughout.)
// When the waves that multiply issue the copies as well (as this kernel did), they stand in that queue first and
// read and multiply after it, with the memory path idle (1024 x 1024, n = 3136: 20.1 us instead of 15.6).
// (Measured and dropped: operands loaded from memory straight into the registers of 16x16x32 MFMAs,
// without LDS: sixteen consecutive lanes then read sixteen rows, which the memory path takes one by
// one, 64 clocks per load instead of 16: 31 us.)
//
// ODD = false: every row starts at an address that is a multiple of four, what a copy needs: n is even
// and so are the operands' first addresses, in elements.  The last n % 8 columns, which fill no piece,
// are one more MFMA step at the end, its operands loaded element by element.  ODD = true, anything else: a row that starts two
// bytes past a multiple of four is copied from there, one element early, and the fragments are moved
// into place when they are read, the last element from the piece that follows.  The stages then
// overlap by one piece (P - 1 pieces each), and the last 8 .. 15 columns are the step at the end.
template <bool ODD, int BM, int BN, int P>
__global__ __launch_bounds__(kSmThreads) void sddmm_mfma_kernel(
    int m, int k, int n, int tiles_k, const int* __restrict__ row_offsets,
    const int* __restrict__ column_indices, const _Float16* __restrict__ L, const _Float16* __restrict__ R,
    _Float16* __restrict__ out, const _Float16* __restrict__ scale) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  using Block = SmBlock<BM, BN, P>;
  constexpr int kRing = Block::kRing, kStageBytes = Block::kStageBytes, TM = BM / 32, TN = BN / 32;
  float (*part)[BM][BN + 1] = reinterpret_cast<float (*)[BM][BN + 1]>(lds_raw);   // [wave][row][column], after the loop
  int (*bound)[BM] = reinterpret_cast<int (*)[BM]>(lds_raw + Block::kPartBytes);              // [0]: range start, [1]: end
  int (*ahead)[BM] = reinterpret_cast<int (*)[BM]>(lds_raw + Block::kPartBytes + 2 * BM * 4); // [entry][row]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  int tile_i, tile_c;
  if (!sddmm_mfma_tile(blockIdx.x, (m + BM - 1) / BM, tiles_k, n, tile_i, tile_c)) return;   // whole workgroup, before any barrier
  const int i0 = tile_i * BM;
  const int c0 = tile_c * BN;
  PhaseClocks clocks;
  clocks.start();

  constexpr int kAdvance = ODD ? P - 1 : P;         // pieces from stage to stage
  const int pieces = ODD ? max(0, n / 8 - 1) : n / 8;               // multiplied in stages; the rest at the end
  const int stages = (pieces + kAdvance - 1) / kAdvance;

  if (wave < 4) {
    const int r = lane & 31;
    const int half = lane >> 5;
    const _Float16* lrow[TM];
    const _Float16* rrow[TN];
    bool lodd = false, rodd = false;
#pragma unroll
    for (int i = 0; i < TM; ++i) lrow[i] = L + (size_t)min(i0 + 32 * i + r, m - 1) * n;
#pragma unroll
    for (int j = 0; j < TN; ++j) rrow[j] = R + (size_t)min(c0 + 32 * j + r, k - 1) * n;
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[i][j][t] = 0.f;
    // the columns past the last piece: fetched now, multiplied after the loop, by one of the waves
    f16x8 at[TM], bt[TN];
    const bool tail = wave == 0 && 8 * pieces < n;
    if (tail) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int col = 8 * pieces + 8 * half + t;
#pragma unroll
        for (int i = 0; i < TM; ++i) at[i][t] = col < n ? lrow[i][col] : (_Float16)0.f;
#pragma unroll
        for (int j = 0; j < TN; ++j) bt[j][t] = col < n ? rrow[j][col] : (_Float16)0.f;
      }
    }
    if (ODD) {                                         // (rows 32 apart, or clamped: the same parity or never looked at)
      lodd = ((uintptr_t)(L + (size_t)(i0 + r) * n) & 2) != 0;
      rodd = ((uintptr_t)(R + (size_t)(c0 + r) * n) & 2) != 0;
    }
    const unsigned lshift = lodd ? 16u : 0u, rshift = rodd ? 16u : 0u;
    // operand fragments: lane (r, half) reads pieces P / 4 * wave + 2 * step + half of rows r, 32 + r .. of L
    // and of R, from their swizzled slots (rows r and 32 + r have the same)
    const int a_row_off = r * (P * 16), b_row_off = (BM + r) * (P * 16);
    constexpr int kBlock = 32 * P * 16;
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
    int place = 0;                                     // of stage s in the ring
    for (int s = 0; s < stages; ++s) {
      __syncthreads();                                 // stage s has arrived
      clocks.lap(kPhaseBarrier);
      const char* buf = lds_raw + place * kStageBytes;
      place = place == kRing - 1 ? 0 : place + 1;
      const bool ragged = (s + 1) * kAdvance > pieces;
#pragma unroll
      for (int step = 0; step < P / 8; ++step) {
        const int p = P / 4 * wave + 2 * step + half;
        const int slot = (p ^ (r & 15)) << 4, next = (((p + 1) & (P - 1)) ^ (r & 15)) << 4;
        u32x4 a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = fragment(buf + a_row_off + i * kBlock, slot, next, lshift);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = fragment(buf + b_row_off + j * kBlock, slot, next, rshift);
        // pieces past the last, and the one that overlaps the next stage (both operands: 0 * Inf)
        if ((ragged && s * kAdvance + p >= pieces) || (ODD && p == kAdvance)) {
#pragma unroll
          for (int i = 0; i < TM; ++i) a[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int j = 0; j < TN; ++j) b[j] = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a[i]), __builtin_bit_cast(f16x8, b[j]), acc[i][j], 0, 0, 0);
      }
      clocks.lap(kPhaseSteps);
    }
    if (tail) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(at[i], bt[j], acc[i][j], 0, 0, 0);
    }
    clocks.lap(kPhaseRest);
    __syncthreads();                                   // the ring is free: it now holds the four partial blocks
    clocks.lap(kPhaseBarrier);
    // Register t of lane (r, half) in acc[i][j] is element (32*i + 8*(t/4) + 4*half + t%4, 32*j + r).
    float (*mine)[BN + 1] = part[wave];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int t = 0; t < 16; ++t) mine[32 * i + 8 * (t / 4) + 4 * half + (t % 4)][32 * j + r] = acc[i][j][t];
  } else if (wave < 8) {
    // Copy 4 j + w of wave w of these, of 1 KB, fills rows 64 / P (4 j + w) .. of the stage (L's, then R's); lane t brings of row t / P of those
    // the piece (t % P) xor (row % 16), to slot t % P.  Rows past the end of either matrix are clamped (their results
    // are never looked at), pieces past the last become the stage's first (zeroed when they are read).
    // The copies are issued from inline assembly and waited for with explicit counts: they are the only
    // vector-memory operations of these waves and complete in the order issued.
    constexpr int C = Block::kCopies;
    const int fetched = ODD ? pieces + 1 : pieces;
    const char* first[2] = {reinterpret_cast<const char*>(L + (size_t)i0 * n), reinterpret_cast<const char*>(R + (size_t)c0 * n)};
    unsigned voff[C];
    int vpiece[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const bool of_r = j >= Block::kCopiesL;
      const int row = 64 / P * (4 * (of_r ? j - Block::kCopiesL : j) + wave - 4) + lane / P;
      vpiece[j] = (lane & (P - 1)) ^ (row & 15);
      voff[j] = (unsigned)min(row, of_r ? k - 1 - c0 : m - 1 - i0) * (unsigned)n * 2u;
      if (ODD) voff[j] += 2u - ((unsigned)((uintptr_t)first[of_r] + voff[j]) & 2u);
    }
    if (ODD) {
      first[0] -= 2;
      first[1] -= 2;
    }
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_raw + (unsigned)(wave - 4) * 1024u;
    int place = 0;
    auto issue_stage = [&](int s) __attribute__((always_inline)) {
      const unsigned dst = lds_base + (unsigned)(place * kStageBytes);
      place = place == kRing - 1 ? 0 : place + 1;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const bool in = s * kAdvance + vpiece[j] < fetched;
        const unsigned off = voff[j] + (in ? (unsigned)vpiece[j] * 16u : 0u);
        const unsigned m0v = dst + (unsigned)j * 4096u;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(m0v), "v"(off), "s"(first[j >= Block::kCopiesL] + (size_t)s * (kAdvance * 16)) : "memory", "m0");
      }
    };
    clocks.lap(kPhaseSetup);
#pragma unroll
    for (int s = 0; s < kRing - 1; ++s)
      if (s < stages) issue_stage(s);
    clocks.lap(kPhaseIssue);
    for (int s = 0; s < stages; ++s) {
      // stage s has arrived when at most the copies of the later stages are outstanding (or of fewer, near the end)
      constexpr int kLater = kRing - 2;
      const int later = stages - 1 - s;
      if (later >= kLater) asm volatile("s_waitcnt vmcnt(%0)" :: "i"(kLater * C) : "memory");
      else if (later >= kLater / 2) asm volatile("s_waitcnt vmcnt(%0)" :: "i"(kLater / 2 * C) : "memory");
      else if (later >= 2) asm volatile("s_waitcnt vmcnt(%0)" :: "i"(2 * C) : "memory");
      else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" :: "i"(C) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      clocks.lap(kPhaseWait);
      __syncthreads();                                 // ... and stage s-1 is consumed
      clocks.lap(kPhaseBarrier);
      if (s + kRing - 1 < stages) issue_stage(s + kRing - 1);
      clocks.lap(kPhaseIssue);
    }
    __syncthreads();
    clocks.lap(kPhaseBarrier);
  } else {
    // Range of row i0 + lane that this block owns, and its first column indices: a step of the searches
    // for both ends in every other stage (a chain of dependent loads), what is left after the loop.
    // (Two halvings per step, three places instead of one, unless there are stages enough: 0.2 .. 0.7 us faster; with 25 stages 0.7 slower.  Three, seven places: each of the loads takes the
    // memory path 64 clocks, a row per lane, 0.3 .. 1 us slower where few stages hide it.)
    const int row = i0 + lane;
    int rs = 0, re = 0;
    if (row < m && lane < BM) {
      rs = row_offsets[row];
      re = row_offsets[row + 1];
    }
    const bool two = stages < 20;
    int lo[2] = {rs, rs}, hi[2] = {re, re}, probe[2][3] = {};
    auto look = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int w = 0; w < 2; ++w)
        if (lo[w] < hi[w]) {
          const int mid = (lo[w] + hi[w]) >> 1;
          probe[w][0] = column_indices[mid];
          if (!two) continue;
          probe[w][1] = column_indices[(lo[w] + mid) >> 1];
          probe[w][2] = column_indices[min((mid + 1 + hi[w]) >> 1, hi[w] - 1)];
        }
    };
    auto halve = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const int key = c0 + BN * w;
        if (lo[w] < hi[w]) {
          const int mid = (lo[w] + hi[w]) >> 1;
          const bool right = probe[w][0] < key;
          if (right) lo[w] = mid + 1; else hi[w] = mid;
          if (two && lo[w] < hi[w]) {
            const int then = (lo[w] + hi[w]) >> 1;
            if (probe[w][right ? 2 : 1] < key) lo[w] = then + 1; else hi[w] = then;
          }
        }
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
    if (lane < BM) {
      bound[0][lane] = lo[0];
      bound[1][lane] = lo[1];
#pragma unroll
      for (int e = 0; e < kSmAhead; ++e) ahead[e][lane] = pre[e];
    }
  }
  clocks.lap(kPhaseRest);
  __syncthreads();
  clocks.lap(kPhaseBarrier);
  if (tid >= 512) {
    clocks.store(blockIdx.x * (kSmThreads / 64) + wave);
    return;
  }

  // Eight or sixteen threads per row take entries of its range in turn.
  constexpr int T = 512 / BM;
  const int rr = tid / T;
  const int row = i0 + rr;
  const int b0 = bound[0][rr], b1 = max(b0, bound[1][rr]);
  for (int p = b0 + (tid & (T - 1)); p < b1; p += T) {
    const int c = p - b0 < kSmAhead ? ahead[p - b0][rr] : column_indices[p];
    const unsigned cc = (unsigned)(c - c0);
    float val;
    if (cc < (unsigned)BN) val = (part[0][rr][cc] + part[1][rr][cc]) + (part[2][rr][cc] + part[3][rr][cc]);
    else val = sddmm_lane_dot(L + (size_t)row * n, R + (size_t)c * n, n);
    sddmm_store<_Float16>(out, scale, p, val);
  }
  clocks.lap(kPhaseRest);
  clocks.store(blockIdx.x * (kSmThreads / 64) + wave);
}

}  // namespace spdl
