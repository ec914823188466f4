// SpMM of dense sparse matrices on the matrix cores, fp32: whole blocks of A, zeros included, times B, from three-term bf16
// products (bf16_split.hpp).
//
// A workgroup owns 64 sparse rows and 64 columns of C and walks A's columns in stages of 128.  Eight waves scatter: sixteen lanes to
// a row, they find the row's entries of the stage by a cursor, take each apart into its terms and write these into a block of
// zeros in LDS, in the order in which the lanes read them as MFMA operands.  Eight waves multiply: each has 32 of the 64 columns and a
// quarter of the stage's columns of A, brings in its rows of B straight into registers (a lane's operand is eight rows of its column),
// splits them there, one step of sixteen ahead, and multiplies them with both 32-row tiles of the block; the quarters are
// added at the end.  Three blocks: one is multiplied, the next one written, the one before cleared, a barrier per stage, which
// a multiplying wave reaches with what it still needs of the block in registers, so that half a step of products lies behind it.
//
// One accumulator, not two as in the SDDMM: a sum is four chains, and 6 k / 64 roundings each leave a smaller error than one
// chain of the row's entries, if these are enough: against the slab kernel, 2-norm of the error, normally distributed values, rows of 10 % / 20 %
// / 30 % of 10240 columns 0.90 / 0.79 / 0.72 of it, of 1025 columns 0.995 / 0.85 / 0.73.  With fewer entries the six roundings for each of
// them count (2.0 times the error for rows of two, 1.3 for 20 of 1025, 1.06 for 205 of 10240): such rows are gathered (spmm_split_entries).  What
// is left out of a product is below 2^-24 of it: the terms of both operands are rounded.  (A's cut off, up to 2.9 times that: 1.01 .. 1.04
// times the error, and the same time.  6765 x 2169 at 28 %, n = 120: 30 us; every other row of 40 entries: 34.8, gathered 43.4, slab kernel 66.)
//
// What bounds it: the issue of vector instructions beside the MFMA.  A stage is 48 MFMA of 32 clocks on each SIMD, 240 vector
// instructions of the multiplying waves and 120 (10 %) to 230 (30 %) of the scattering ones; it takes 3000 .. 3400 clocks, the sum of
// both.  Without scattered stores 10 .. 25 us less of 146 at 30 %, without loads of B 10, without the splitting 13, reading A back costs
// nothing; rows of B requested two steps further ahead, half a stage between the two multiplying waves of a SIMD, 64 columns and an
// eighth of the stage per wave, splitting by dot products of bf16 pairs (fewer instructions, but none beside an MFMA) gain nothing.
// 8192 x 10240, n = 128, slab kernel -> here, inputs in turn: 20 % 142 us -> 136, 30 % 202 -> 148 (188 -> 144 on a faster card); 6765 x 2169 at
// 28 %, n = 120: 41.0 -> 30.4; 5923 x 6704 at 42 %, n = 128: 157 -> 94; at 10 % 84 us -> 116, which is why the density decides.
//
// Rows that are not ascending, or hold a column twice, are noticed (an entry that does not come right after a smaller column of the
// same stage; a cursor short of the row's end) and gathered at the end (split_gather), as is what is not finite: a zero of the
// block times an infinity of B must not reach the result.
#pragma once
#include "bf16_split.hpp"

namespace spdl {

constexpr int kDsRows = 64;                              // sparse rows per workgroup
constexpr int kDsCols = 64;                              // columns of C per workgroup
constexpr int kDsS = 128;                                // columns of A per stage
constexpr int kDsGroup = kDsRows * 16 + 16;              // bytes of eight columns, one term: the next eight lie four banks on
constexpr int kDsPlane = kDsS / 8 * kDsGroup;            // one term of a stage's block of A
constexpr int kDsBuf = 3 * kDsPlane;
constexpr int kDsLdsBytes = 3 * kDsBuf + kDsRows * 4;
constexpr int kDsMulWaves = 8, kDsScatterWaves = 8;
constexpr int kDsThreads = 64 * (kDsMulWaves + kDsScatterWaves);

// Lane i gets the place of the (i + 1)-th one of `set`.  (Lanes beyond the last one: those of the zeros.)
__device__ __forceinline__ int nth_one(unsigned long long set) {
  const int lane = threadIdx.x & 63;
  const int before = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(set >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)set, 0u));
  const int to = (set >> lane & 1) ? before : __builtin_popcountll(set) + lane - before;
  return __builtin_amdgcn_ds_permute(to * 4, lane);
}

// Results that the matrix cores cannot give, from the rows of B themselves: row i of the workgroup (bit i of `rows`) in the fours of
// columns that lane i's `mask` names.  All threads of the workgroup share out the rows, and a row's among the fours of columns that any
// row needs and parts of the row's entries, sixteen of them in flight for each thread: a single row waits for a few gathers, not for
// as many as it has sixteens, and where all rows need four columns (an infinity in B) no lane idles.  A part whose sums are
// all NaN already is done.  (8192 x 10240 at 30 %, n = 128, 143 us with nothing to gather; by the thread that has the result, eight entries in
// flight -> here: one infinity in B 727 us -> 286, a row of them 2960 -> 692, B all NaN 121, one NaN in A 364 -> 149, one row
// in 64 not ascending 342 -> 151, none 2970 -> 694.)
__device__ __forceinline__ void split_gather(unsigned long long rows, unsigned mask, int i0, int j0, int m, int n,
                                             const int* __restrict__ row_offsets, const int* __restrict__ column_indices,
                                             const float* __restrict__ values, const float* __restrict__ B, float* __restrict__ C,
                                             const float* __restrict__ bias, int relu, char* lds) {
  const int tid = threadIdx.x;
  unsigned any = mask;
#pragma unroll
  for (int d = 1; d < kWave; d *= 2) any |= (unsigned)__shfl_xor((int)any, d, kWave);
  const int nrows = __builtin_popcountll(rows), nfours = __builtin_popcount(any);
  const int row_bits = nrows > 1 ? 32 - __builtin_clz(nrows - 1) : 0, four_bits = nfours > 1 ? 32 - __builtin_clz(nfours - 1) : 0;
  const int per_row = kDsThreads >> row_bits, mine = tid & (per_row - 1), index = tid / per_row;
  const int part = mine >> four_bits, parts = min(per_row >> four_bits, 64);
  const int local = __shfl(nth_one(rows), index, kWave), four = __shfl(nth_one(any), mine & ((1 << four_bits) - 1), kWave);
  const unsigned wanted = (unsigned)__shfl((int)mask, local, kWave);
  const bool on = index < nrows && (mine & ((1 << four_bits) - 1)) < nfours && (wanted >> four & 1) && part < parts;
  const int row = i0 + local, first = j0 + 4 * four, col = min(first, n - 4);               // (the last four columns of B's row at its end)
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
  f32x4* const sums = reinterpret_cast<f32x4*>(lds);                   // (the products' sums before have been read)
  sums[tid] = f32x4{v[0], v[1], v[2], v[3]};
  __syncthreads();
  if (!on || part > 0) return;
#pragma unroll 4
  for (int i = 1; i < parts; ++i) {
    const f32x4 x = sums[tid + (i << four_bits)];
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] += x[t];
  }
  spmm_epilogue<float, 4>(v, bias, row, relu);
  float* const c = C + (size_t)row * n + col;
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (col + t >= first) c[t] = v[t];
}

// Entries from which on a row's sum on the matrix cores is no less exact than a chain of multiply-adds.  (It is as exact at 100 entries of
// 1025 columns, 155 of 2169, 290 of 5120, 460 of 10240.)
__host__ __device__ constexpr int spmm_split_entries(int k) { return 72 + k / 24; }

// NC sixteens of a row's entries fetched a stage ahead.  (k >= 16, 0 < nnz < 2^28.)
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
  int* const redo = reinterpret_cast<int*>(lds_raw + 3 * kDsBuf);       // rows to be gathered
  auto barrier = [&]() __attribute__((always_inline)) {                // (no wait for memory)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < (3 * kDsBuf + 16 * kDsThreads - 1) / (16 * kDsThreads); ++i)
      if ((i * kDsThreads + tid) * 16 < 3 * kDsBuf) *reinterpret_cast<f32x4*>(lds_raw + (i * kDsThreads + tid) * 16) = zero;
  }
  barrier();

  if (wave < kDsMulWaves) {
    const int r = lane & 31, h = lane >> 5, quarter = wave & 3, half = wave >> 2;
    const int col = tile * kDsCols + half * 32 + r;                    // (columns past n: the last one again, not stored)
    const unsigned row_bytes = (unsigned)n * 4u;
    const unsigned lane_off = (unsigned)(8 * h) * row_bytes + (unsigned)min(col, n - 1) * 4u;
    float raw[2][8];
    // Rows of the wave's columns: step 2 q + s is columns 128 q + 32 quarter + 16 s .. of A.  The sixteen that k ends in, and steps
    // past it, take A's last sixteen: an entry of theirs is scattered to where its row of B then comes.
    auto load_b = [&](float (&x)[8], int step) __attribute__((always_inline)) {
      const int k0 = uniform(min((step >> 1) * kDsS + quarter * 32 + (step & 1) * 16, k - 16));
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B) + (size_t)k0 * (unsigned)n, 0, 0x7fffffff, 0x00020000);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)lane_off, (int)((unsigned)e * row_bytes), 0));
    };
    // A lane's operand of a term, eight columns of row 32 i + r: 16 bytes at group * kDsGroup + 512 i + 16 r.
    unsigned a_off[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) a_off[s] = (unsigned)((2 * (2 * quarter + s) + h) * kDsGroup + (r << 4));
    bf16x8 high[2], mid[2], low[2];
    auto load_a = [&](bf16x8 (&x)[2], const char* p) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = *reinterpret_cast<const bf16x8*>(p + i * 512);
    };
    acc32x32 sum[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int x = 0; x < 16; ++x) sum[i][x] = 0.f;
    auto two = [&](const bf16x8 (&x)[2], const bf16x8& y) __attribute__((always_inline)) {
      sum[0] = mfma_bf16(x[0], y, sum[0]);
      sum[1] = mfma_bf16(x[1], y, sum[1]);
    };
#pragma unroll
    for (int i = 0; i < 2; ++i) load_b(raw[i], i);
    barrier();                                                         // the first stage's block is there
    load_a(high, lds_raw + a_off[0]);
    load_a(mid, lds_raw + a_off[0] + kDsPlane);
    load_a(low, lds_raw + a_off[0] + 2 * kDsPlane);
    Split8 b = split8(raw[0]);
    clocks.lap(kPhaseSetup);
    char* const clear = lds_raw + wave * (kDsBuf / kDsMulWaves) + lane * 16;
    static_assert(kDsBuf / kDsGroup % kDsMulWaves == 0, "whole groups for a wave");
    // One step of sixteen columns; `next` is where the next one's operands are, each read as soon as its registers are done
    // with.  `last` of a stage: half of the products need nothing of the stage's block that is not in registers.
    auto step = [&](const char* next, int at, bool last, int before, float (&now)[8], float (&after)[8])
                    __attribute__((always_inline)) {
      load_b(now, at + 2);
      const Split8 c = split8(after);
      two(high, b.low);
      two(high, b.mid);
      two(high, b.high);
#pragma unroll
      for (int g = 0; g < 6; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 5, 0);
      }
      if (last) {
        clocks.lap(kPhaseSteps);
        __builtin_amdgcn_sched_barrier(0);
        barrier();                                                     // this block may be cleared; the next one is there
        clocks.lap(kPhaseBarrier);
      }
      __builtin_amdgcn_sched_barrier(0);
      load_a(high, next);
      if (!last) {
        const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < kDsBuf / kDsGroup / kDsMulWaves; ++i) *reinterpret_cast<u32x4*>(clear + before * kDsBuf + i * kDsGroup) = zero;
      }
      two(mid, b.mid);
      two(mid, b.high);
      load_a(mid, next + kDsPlane);
      two(low, b.high);
      load_a(low, next + 2 * kDsPlane);
      b = c;
      __builtin_amdgcn_sched_barrier(0);
    };
    int x = 0, before = 2;
    for (int q = 0; q < nst; ++q) {
      const int next = x == 2 ? 0 : x + 1;
      step(lds_raw + x * kDsBuf + a_off[1], 2 * q, false, before, raw[0], raw[1]);
      step(lds_raw + next * kDsBuf + a_off[0], 2 * q + 1, true, before, raw[1], raw[0]);
      before = x;
      x = next;
    }
    barrier();
    // This wave's sums.  Register t of lane (r, h) is row 8 (t / 4) + 4 h + t % 4 of the tile, column r.
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int row = 32 * i + 8 * (t / 4) + 4 * h + t % 4;
        *reinterpret_cast<float*>(lds_raw + quarter * (kDsRows * kDsCols * 4) + row * (kDsCols * 4) + (half * 32 + r) * 4) = sum[i][t];
      }
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
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int local = first_row + 4 * j + sub, row = min(i0 + local, m);
      at[j] = (row_offsets[row] + l16) * 4;
#pragma unroll
      for (int e = 0; e < NC; ++e) row_end[j][e] = row_offsets[min(row + 1, m)] * 4 - 64 * e;
      row_base[j] = (unsigned)((local >> 5) * 512 + ((local & 31) << 4));
      strays[j] = 0;
    }
    auto fetch = [&](int j) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < NC; ++e) cc[j][e] = (int)__builtin_amdgcn_raw_buffer_load_b32(column_rsrc, at[j] + 64 * e, 0, 0);
#pragma unroll
      for (int e = 0; e < NC; ++e)
        aa[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(value_rsrc, at[j] + 64 * e, 0, 0));
    };
    auto term = [](float x) __attribute__((always_inline)) {           // x rounded to its first term, in the upper half
      return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{0.f, x}), bf16x2));
    };
    const int shift16 = 16 * (sub & 1);
    const bool upper = sub >= 2;
    unsigned last = 0;                                                 // the last column of the round before, in a group's first lane
    // The fetched entries of row j in the stage's columns; whether there may be more of them.  What is fetched is used up
    // before the next fetch, which then has the same registers: the compiler copies nothing, and so waits for nothing, before the next stage.
    auto round = [&](int j, char* block, int start, bool again) __attribute__((always_inline)) -> bool {
      unsigned long long mk[NC];
      unsigned rel[NC];
      float v[NC];
      unsigned count = 0;
#pragma unroll
      for (int e = 0; e < NC; ++e) {
        rel[e] = (unsigned)(cc[j][e] - start);
        v[e] = aa[j][e] * kSplitScale;
        mk[e] = __builtin_amdgcn_ballot_w64(at[j] < row_end[j][e]) & __builtin_amdgcn_ballot_w64(rel[e] < (unsigned)kDsS);
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
          typedef __attribute__((address_space(3))) unsigned short LdsHalf;
          LdsHalf* const to = (LdsHalf*)(uintptr_t)d;
          const unsigned x = term(v[e]);
          const float rest = v[e] - __builtin_bit_cast(float, x);
          const unsigned y = term(rest), z = __builtin_bit_cast(unsigned, rest - __builtin_bit_cast(float, y));      // (eight bits at most are left)
          to[0] = (unsigned short)(x >> 16);
          to[kDsPlane / 2] = (unsigned short)(y >> 16);
          to[kDsPlane] = (unsigned short)(z >> 16);
        }
      }
      const bool more = (mk[NC - 1] & (kFirst << 15)) != 0;
      if (more) last = (unsigned)__builtin_amdgcn_mov_dpp((int)rel[NC - 1], 0x121, 0xf, 0xf, true);
      return more;
    };
    // (ahead of the multiplying waves, which have the MFMA to wait for: 30 %, 157 us -> 147; 42 %, 111 -> 96)
    __builtin_amdgcn_s_setprio(1);
    auto fill = [&](int q, int x) __attribute__((always_inline)) {
      char* block = lds_raw + x * kDsBuf;
#pragma unroll
      for (int j = 0; j < NR; ++j)
        if (round(j, block, q * kDsS, false))
          while (round(j, block, q * kDsS, true)) {}
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
      if (l16 == 0)
        redo[local] = at[j] != row_end[j][0] || (strays[j] & mine) != 0 || (entries > 0 && entries < spmm_split_entries(k));
    }
  }
  clocks.lap(kPhaseRest);
  clocks.store(blockIdx.x * (kDsMulWaves + kDsScatterWaves) + wave);
  barrier();
  // The four sums of each result; four columns to a thread.
  static_assert(kDsThreads * 4 == kDsRows * kDsCols, "a thread for every four results");
  const int local = tid >> 4, c4 = (tid & 15) * 4, row = i0 + local, col = tile * kDsCols + c4;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(lds_raw + w * (kDsRows * kDsCols * 4) + local * (kDsCols * 4) + c4 * 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] += x[t];
  }
  const int count = row < m ? min(4, n - col) : 0;
  bool failed = redo[local] != 0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    v[t] *= kSplitUnscale;
    failed |= split_failed(v[t]);
  }
  failed &= count > 0;
  const unsigned long long fails = __builtin_amdgcn_ballot_w64(failed);
  if ((tid & 15) == 0) redo[local] = (int)((unsigned)(fails >> (lane & 48)) & 0xffffu);      // (fours of columns to be gathered)
  if (!failed) {
    if (count > 0) spmm_epilogue<float, 4>(v, bias, row, relu);
    float* c = C + (size_t)row * n + col;
    if (count >= 4) {
      Pack<float, 4>::store(c, v);
    } else {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t < count) c[t] = v[t];
    }
  }
  barrier();
  const unsigned mask = (unsigned)redo[lane];
  const unsigned long long rows = __builtin_amdgcn_ballot_w64(mask != 0);
  if (rows == 0) return;
  split_gather(rows, mask, i0, tile * kDsCols, m, n, row_offsets, column_indices, values, B, C, bias, relu, lds_raw);
}

}  // namespace spdl
