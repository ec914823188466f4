// libspdl: C ABI, argument checks, kernel selection and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <numeric>
#include <vector>

#include "../../include/spdl.h"
#include "common.hpp"
#include "csr_softmax.hpp"
#include "sddmm_group.hpp"
#include "sddmm_lane.hpp"
#include "sddmm_mfma.hpp"
#include "sddmm_nt.hpp"
#include "sddmm_rowstrip.hpp"
#include "sddmm_slab.hpp"
#include "sddmm_slab_dma.hpp"
#include "spmm_rowsplit.hpp"
#include "spmm_slab.hpp"
#include "spmm_mfma.hpp"
#include "spmm_slab_dma.hpp"
#include "spmm_window.hpp"
#include "spmm_slab_tiles.hpp"
#include "spmm_slab_wide.hpp"
#include "spmm_split.hpp"
#include "sddmm_window.hpp"
#include "sddmm_split.hpp"
#include "sddmm_long.hpp"

namespace {

using namespace spdl;

enum SpmmVariant { kSpmmRowsplit = 0, kSpmmSlab = 1, kSpmmSlabDma = 2, kSpmmMfma = 3, kSpmmWindow = 4, kSpmmVariants };
// What the caller says about the sparse matrix (the library never reads the topology on the host).
enum Hint { kHintNone = 0, kHintBanded = 1, kHintSkewed = 2 };
enum SddmmVariant { kSddmmRowstrip = 0, kSddmmGroup = 1, kSddmmSlab = 2, kSddmmSlabDma = 3, kSddmmMfma = 4, kSddmmLane = 5, kSddmmWindow = 6, kSddmmVariants };

std::atomic<int> g_forced[2] = {{-1}, {-1}};

inline bool aligned(const void* p, size_t bytes) { return (reinterpret_cast<uintptr_t>(p) % bytes) == 0; }

inline bool sizes_ok(int m, int k, int n, int nnz) {
  if (m < 0 || k < 0 || n < 0 || nnz < 0) return false;
  const int64_t lim = (int64_t)1 << 31;
  return (int64_t)m * n < lim && (int64_t)k * n < lim;
}

// Widest vector width (in elements) usable for rows of length n starting at these bases.
template <typename T>
int pick_vec(int n, const void* a, const void* b, int max_vec) {
  for (int v = max_vec; v > 1; v /= 2)
    if (n % v == 0 && aligned(a, v * sizeof(T)) && aligned(b, v * sizeof(T))) return v;
  return 1;
}

// Lanes per row: the smallest group whose tile covers n, so that small n spreads a wave over
// several rows instead of idling lanes (paper Sec. "Subwarp Tiling").
inline int pick_group(int n, int vec) {
  for (int g = 8; g < kWave; g *= 2)
    if (g * vec >= n) return g;
  return kWave;
}

constexpr int kSlabS = 256;                       // B rows per LDS slab
constexpr int kSlabLdsBytes = 2 * (kSlabS + 1) * kSlabTile * 4;
constexpr int kComputeUnits = 256;

// Lane groups per row of the row-splitting kernel, only with the widest vectors: a group that walks a row alone takes a memory
// latency for every eight entries.  Groups of a wave share a row while the machine has room (16 waves on each compute unit) and every
// group 32 entries; with fewer waves shorter lists will do, 16 entries up to 2048 waves, 5 up to 1024.  Up to 2048 rows all four
// waves of a workgroup share one (256 / g groups: a row and 64 columns sixteen), from 3 entries per group on, 4.5 beyond 1024 rows.
// (us a launch in a graph of them, of which an empty one takes 1.9, one group or few -> now: 512 x 512 at 10 %, n = 128, 3.81 -> 3.43; 526 x
// 576, rows of 113, n = 42, 7.5 -> 3.9; 305 x 926, rows of 272, n = 40, 6.1 -> 4.5; rows of unequal length more so: 1001 x 1936, rows
// of 99, log-normal, n = 52, 28 -> 7.  330 random shapes of 180 .. 8000 rows and 8 thousand to 1 million entries, those that come to this
// kernel: fp32 uniform 0.83 of the time before and 1.08 at worst, with log-normal rows among them 0.78; fp16 0.79 and 0.65.  Lower
// bounds on the entries cost up to 1.17 on rows of 16 .. 50.)
// Wider outputs, whose groups are whole waves: in half precision up to 800 waves of one group per row, up to 1600 for rows of 50 entries, with
// even n (0.82 of the time on uniform rows and 0.48 on log-normal ones, 0.99 and 0.66 in the second range; short rows there 1.06 .. 1.4,
// 1600 .. 3200 waves 1.27 on uniform rows; odd n, whose narrower loads make more waves of it, 0.97.  fp32 1.0 .. 1.7).
template <typename T>
int pick_segments(int m, int n, int nnz, int vec, int g) {
  if (vec != 16 / (int)sizeof(T) || m <= 0) return 1;
  const int64_t avg = nnz / m;
  auto waves = [&](int seg) { return (int64_t)m * g * seg / kWave; };
  int seg = 1;
  while (g * seg * 2 <= kWave && waves(seg) < 16 * kComputeUnits &&
         avg >= std::max(16, 2 * seg * (waves(2 * seg) > 2048 ? 32 : waves(2 * seg) > 1024 ? 16 : 5)))
    seg *= 2;
  const int all = 256 / g;
  if (g < kWave && g * seg == kWave && m <= 2048 && 2 * avg >= (m <= 1024 ? 6 : 9) * all) seg = all;
  if (sizeof(T) == 2 && g == kWave && n % 2 == 0) {
    const int64_t tiles = (n + g * vec - 1) / (g * vec);
    if (avg >= (m * tiles < 800 ? 16 : 50) && m * tiles < 1600) seg = all;
  }
  return seg;
}

template <typename T>
void fill_spmm_rowsplit_info(int m, int n, int nnz, const void* B, const void* C, spdl_launch_info* info) {
  constexpr int kWide = 16 / (int)sizeof(T);
  int vec = pick_vec<T>(n, B, C, kWide);
  auto waves = [&](int v) {
    const int g = pick_group(n, v);
    return (int64_t)m * g * pick_segments<T>(m, n, nnz, v, g) / kWave * ((n + g * v - 1) / (g * v));
  };
  // (Rows of B at any alignment: 16 bytes per lane all the same, the lane at the row's end taking the
  // row's last ones.  Not for small problems, where more lanes per row count for more: 512 x 512
  // at 10 %, n = 127: 5.1 us against 6.3.)
  // Half-precision rows at odd elements: sixteen such bytes a lane take the memory path long enough that a wave which
  // walks a long row alone is the slower for it.  4 bytes a lane where 16 would leave fewer than 2500 waves, below 800
  // waves 2, as narrow as before; not where lane groups share a row.  (382 x 674 at 4 %, log-normal rows, n = 1195: 24.4 us
  // with 16 bytes, 15.0 with 4, 15.5 with 2; uniform rows, means over 94 shapes of 2 .. 30 %, 16 and 4 bytes against 2: 1.03
  // and 0.97 at 400 .. 800 waves, 0.95 and 0.93 to 1200, 0.85 and 0.81 to 1800, 0.77 and 0.81 to 2500, 0.56 and 0.70 beyond;
  // log-normal rows, 134 shapes: 1.31 and 1.03, 1.30 and 1.01, 1.24 and 0.93, 1.04 and 0.85, 0.88 and 0.81.  Rows at even
  // elements take 16 bytes at any number of waves: below 1800, against as narrow as before, 0.88 on uniform rows and 1.10 on
  // log-normal ones, which the host cannot tell apart.)
  // (also where groups share a row)
  const bool shared = n >= kWide && pick_segments<T>(m, n, nnz, kWide, pick_group(n, kWide)) > 1;
  if (vec < kWide && n >= kWide && ((int64_t)nnz * n >= (1 << 24) || (n >= 512 && sizeof(T) == 2) || shared)) {
    if (sizeof(T) == 4 || vec > 1 || shared || waves(kWide) >= 2500) vec = kWide;
    else if (waves(kWide) >= 800) vec = 2;
  }
  // fp32, few waves: narrower loads, so that a wave has a row to itself (its indices are then scalar loads) and
  // the row is spread over more waves.  Below 1280 waves (five per compute unit) to a wave per row, two rows per wave
  // being no gain (3000 x 3000 at 1 %, n = 64: 4.3 us with four rows per wave, 5.2 with two, 4.0 with one), and on
  // where that pads n less (600 x 2400 at 6 %, n = 300: 13.4 us, 10.4); below 1024 in any case (512 x 512 at
  // 10 %, n = 128: 5.1 us with 4 columns per lane, two rows per wave; 4.5 with 2, one row; 3.8 with 1, half a row).
  // (760 x 3000 at 5 %, n = 276, 1520 waves: 14.5 us as it is, 16.5 narrower.)
  // Widths under 256, where rows share a wave, with short rows only, and not too many: the more nonzeros, the more
  // the number of load instructions counts, which narrow pieces multiply (n = 128, rows of 150, m = 1000: 6.2 us
  // as it is, 6.9 narrower; n = 32, rows of 100, m = 2000: 5.1 and 6.3; rows of 40, m = 4000: 4.75 and 4.57,
  // m = 8000: 5.75 and 6.7).
  if (sizeof(T) == 4 && vec == kWide && !shared && (n >= 256 || (nnz < 3 << 16 && nnz <= 64 * (int64_t)m))) {
    auto padded = [&](int v) { return (n + pick_group(n, v) * v - 1) / (pick_group(n, v) * v) * (pick_group(n, v) * v); };
    if (waves(vec) < 5 * kComputeUnits && waves(1) > waves(vec))
      while (vec > 1 && pick_group(n, vec) < kWave) vec /= 2;
    while (vec > 1 && waves(vec / 2) > waves(vec) &&
           waves(vec) < (padded(vec / 2) < padded(vec) ? 5 * kComputeUnits : 4 * kComputeUnits))
      vec /= 2;
  }
  const int g = pick_group(n, vec);
  const int seg = pick_segments<T>(m, n, nnz, vec, g);
  info->variant = kSpmmRowsplit;
  info->vec = vec;
  info->lanes_per_row = g;
  info->rows_per_block = 256 / (g * seg);
  info->block_threads = 256;
  info->grid_x = (m + info->rows_per_block - 1) / info->rows_per_block;
  info->grid_y = (n + g * vec - 1) / (g * vec);
}

template <typename T>
bool slab_usable(int n, int nnz, const void* B, const void* C) {
  // 32-bit byte offsets: into the pair arrays, and from a slab's start to any of its elements
  return n % 4 == 0 && n < (1 << 21) && nnz < (1 << 29) && aligned(B, 4 * sizeof(T)) && aligned(C, 4 * sizeof(T));
}
// The copy-based slab kernels take any n from 4 on and element-aligned operands: a copy of 16 bytes
// into LDS may start at any float, at the same rate.  (LSTM shape at 90 % sparsity, n = 127: 95 us
// against 256 for row splitting with one column per lane; 4096 x 1024 at 10 %, n = 1001: 38 against 93.)
inline bool slab_dma_usable(int n, int nnz) { return n >= 4 && n < (1 << 21) && nnz < (1 << 29); }

// Chain of work in front of the slowest compute unit when every panel's work is dealt to `parts` workgroups of `units`
// each (see split_for_machine).
double split_chain(int panels, int parts, int units, int slots = kComputeUnits) {
  return (double)((slab_xcd_load(panels, parts) + slots / 8 - 1) / (slots / 8)) * (units + 2.0);
}

// A slab kernel's workgroup fills a compute unit (LDS), so a grid of more than `slots` workgroups
// runs in rounds.  `total` units of work per panel (tiles of C, slabs of A's columns), walked back
// to back by one workgroup, are dealt to the number of workgroups per panel that gives the shortest
// chain: rounds x (units per workgroup + two units' worth of set-up).  slab_wg_map ties the
// workgroups to XCDs, so the rounds are those of the XCD with the most of them.
// (3072 rows, 48 panels, six per XCD: six workgroups per panel would be 36 on each XCD's 32 compute
// units, a second round for four of them; five make 30 in one round.)  Returns the units per
// workgroup.
int split_for_machine(int panels, int total, int slots = kComputeUnits) {
  int best_units = total;
  double best = 1e300;
  for (int parts = 1; parts <= std::min(total, slots); ++parts) {
    const int units = (total + parts - 1) / parts;
    const double cost = split_chain(panels, (total + units - 1) / units, units, slots);
    if (cost < best - 1e-9) {
      best = cost;
      best_units = units;
    }
  }
  return best_units;
}

int slab_tiles_per_wg(int panels, int tiles, int slots = kComputeUnits) { return split_for_machine(panels, tiles, slots); }

// Products with so few positions keep a lane group per row, whose sums are added in stored order: whichever of the slab and
// row-splitting kernels such a product runs in, the result has the same bits, on which tests of all families at 203 x 700 insist.
// What that costs: sharing rows would take a tenth to a fifth off launches of 5 .. 11 us (203 x 700 at 15 %, n = 75:
// 8.4 us against 6.7, row-splitting 5.0), of which a tenth are left to the slab kernel.
inline bool slab_rows_stay_whole(int m, int k) { return (int64_t)m * (int64_t)k <= 384 * 384; }

// Panels for the copy-based kernel when panels of 64 rows would leave half of the compute units or more without a
// workgroup: rows shared by two or four lane groups (panels of 32 or 16 rows), one workgroup per CU as with panels of 64 rows.
// Twice as many workgroups as compute units cost more than a half-empty machine (two groups instead of four, and
// the reverse: 94 tiles, 3000 x 3000 at 10 %, n = 128: 19.4 us against 34.1; 64 tiles, 2048 x 8000 at 20 %, n = 100:
// 65.8 against 48.1).  With 130 tiles of 64 x 64 and more the full form is faster although some compute units
// stay idle, because every slab of B is copied for 64 rows instead of 32 (in halves of eight waves: 130 tiles, 4104 x
// 5093 at 11 %, n = 112: 61 us in halves, 50 whole; 188 tiles, 12000 x 4000, n = 64: 51 and 39; 240 tiles,
// 7640 x 4322 at 5 %, n = 104: 48 and 30).
int slab_groups_per_row(int m, int k, int n) {
  const int64_t tiles = (int64_t)((m + kSlabRows - 1) / kSlabRows) * ((n + kSlabTile - 1) / kSlabTile);
  if (slab_rows_stay_whole(m, k)) return 1;
  return 4 * tiles <= kComputeUnits ? 4 : 2 * tiles <= kComputeUnits ? 2 : 1;
}

// Pairs of a row that a lane of the copy-based slab kernel fetches at once: as few as make the rounds per slab fewest, for
// a row with 1.75 standard deviations more than the mean of them.  (A longer piece takes longer to bring, a second
// round waits for everything: 8192 x 10240, n = 128, with 2 / 3 / 4 pairs: 8 % 75.3 / 76.3 / 76.8 us, 10 % 89.4 / 85.9 /
// 86.8, 15 % 120.9 / 112.5 / 109.3, 20 % 142.7 / 148.9 / 139.0, 25 % 175.5 / 172.5 / 179.7, 30 % 204 / 195 / 200.  Two pieces
// per lane and round: 5 .. 15 us more at any density.)
int slab_pairs_per_lane(int m, int k, int nnz, int share) {
  const double mean = kSlabS * ((m > 0 && k > 0) ? (double)nnz / ((double)m * (double)k) : 1.0);
  const double pairs = mean + 1.75 * std::sqrt(mean);
  int best = 1;
  for (int pw = 2; pw <= 4; ++pw)
    if (std::ceil(pairs / (16.0 * share * pw)) < std::ceil(pairs / (16.0 * share * best))) best = pw;
  return best;
}

// The forms that scan a slab once for several tiles look 64 pairs ahead per row at most (a row with more takes extra
// rounds behind full waits in every tile's stage): usable where the mean count of a row's pairs in one slab plus three
// standard deviations fits.
inline bool slab_look_fits(int slab_rows, int m, int k, int nnz, double pairs) {
  const double d = (m > 0 && k > 0) ? (double)nnz / ((double)m * (double)k) : 1.0;
  const double mean = slab_rows * d;
  return mean + 3.0 * std::sqrt(mean * std::max(0.0, 1.0 - d)) + 1.0 <= pairs;
}
constexpr int kSlabTilesMax = 4;                  // tiles whose accumulators the tile-inner form keeps in registers

// When the compute unit that is done last ends: workgroups of `units` tiles, `unit` each, and `setup`, a panel's last one with
// what is left of its `tiles`, started in order: the XCD with the most of them (slab_wg_map) deals them to its four shader
// engines of eight compute units in turn, and one that waits for its engine waits however idle another one is.  (264
// workgroups of three tiles, every eleventh of one, all of which fit the XCDs' idle compute units by the time they start: 51 us
// measured, 192 of four and 24 of three 47.)  Equal workgroups run in whole rounds.  Else they are dealt one by one: the
// engine's compute units are a ring in the order in which they are free, and as no workgroup is longer than a whole one, that one
// goes to the ring's end as it is and only a panel's last one moves up; 1 .. 2 ns for each.
int slab_makespan(int panels, int tiles, int units, int unit, int setup) {
  constexpr int kEngines = 4;
  constexpr unsigned kUnits = kComputeUnits / 8 / kEngines;            // compute units of an engine
  const int groups = (tiles + units - 1) / units, left = tiles - (groups - 1) * units;
  const int jobs = slab_xcd_load(panels, groups), whole = panels / 8 * groups, full = setup + unit * units;
  if (jobs <= kComputeUnits / 8) return setup + unit * std::min(units, tiles);
  if (left == units || whole == 0) return (jobs + kComputeUnits / 8 - 1) / (kComputeUnits / 8) * full;
  int last = 0;
  for (int engine = 0; engine < kEngines; ++engine) {
    int ends[kUnits] = {};
    unsigned head = 0;
    int group = engine;
    for (int i = engine; i < jobs; i += kEngines, ++head) {
      while (group >= groups) group -= groups;
      const int end = ends[head % kUnits] + (group == groups - 1 && i < whole ? setup + unit * left : full);
      unsigned at = head;
      for (; at != head + 1 - kUnits && ends[(at - 1) % kUnits] > end; --at) ends[at % kUnits] = ends[(at - 1) % kUnits];
      ends[at % kUnits] = end;
      group += kEngines;
    }
    last = std::max(last, ends[(head - 1) % kUnits]);
  }
  return last;
}

// Forms of the copy-based slab kernel where panels of 64 rows give half of the compute units or more a workgroup.  128 rows, two per
// group: tiles of 64 columns, scanned for each tile anew; tiles of 64, a slab scanned once for up to four; tiles of 128 (a lane
// owns eight columns), a slab scanned once for two.  64 rows, one per group: tiles of 64.  Dense matrices: whole blocks on the matrix cores.
enum SlabForm { kSlabWalk, kSlabInner, kSlabWide, kSlabOneRow, kSlabSplit };
// tiles of 64 columns per workgroup (wide: two for each of 128); when the last compute unit ends (slab_makespan; 0: not worked out)
struct SlabPlan { SlabForm form; int tpw; int span; };

// The form whose last compute unit is estimated to end first.  In thirtieths of a tile of 64 columns and 128 rows: 31 if it is scanned
// for alone, 29 together with others, 53 a tile of 128 columns, 18 one of 64 rows; a workgroup's set-up is worth 9 at 1024 columns and 10
// %, more where a tile's time is shorter.  A wide workgroup may take several pairs of tiles, one after the other: set up once, the
// next pair's first slab copied while the one before is multiplied (4096 x 1024 at 10 %, n = 4096, two rounds of workgroups
// made one: 117.6 us -> 112.6).
// (120 random shapes of 512 tiles of 128 x 64 and more, m, k of 400 .. 2048 by four times as many, both ways round, or 1024 ..
// 12000 by 512 .. 4000, n = 256 .. 4096, 3 .. 25 %, every form with every number of tiles in turn: the estimates scatter by 4 %, the
// choice costs 1 % against the best one each time.  Walking with as many tiles as split_for_machine says, the only choice above
// 12.7 % before, and four tiles scanned together, the only one below: 11 % more time on average, up to 41 %: 3760 x 940 at 7 %, n = 2260, 30
// panels of 36 tiles, 87.8 us -> 62.4.  140 random shapes of 129 .. 2600 tiles of 64 x 64: the choice costs 0.4 %; panels of 64 rows up
// to 1023 tiles, as before, 3.5 %: 4368 x 1092 at 6 %, n = 448, 25.3 us -> 18.6 with 128.)
SlabPlan slab_plan(int m, int k, int n, int nnz) {
  const int tiles = (n + kSlabTile - 1) / kSlabTile, panels = (m + kWideRows - 1) / kWideRows;
  const int wide_tiles = (n + kWideTile - 1) / kWideTile;
  const int panels64 = (m + kSlabRows - 1) / kSlabRows;
  SlabPlan best = {kSlabWalk, slab_tiles_per_wg(panels, tiles), 0};
  if (best.tpw > 24 || slab_xcd_load(panels, tiles) > 8192) {        // (many rounds: all much the same)
    if (best.tpw >= 2 && slab_look_fits(kSlabS, m, k, nnz, 64.0)) best = {kSlabInner, kSlabTilesMax, 0};
    return best;
  }
  const double pairs = kSlabS * (double)nnz / ((double)m * (double)k);
  const int setup = (int)std::max(1.0, std::min(60.0, 9.0 * 1024.0 / (double)k * 35.6 / (10.0 + pairs)));
  // The forms likely to be best first, so that an even share of the others' work alone ends later and is all that is looked at
  // (the host takes 0.9 us for a call on average and 6 for the largest grids; on ties the later form is taken).
  int span = 1 << 30;
  const int walked = best.tpw;
  auto try_form = [&](SlabForm form, int rows, int ntiles, int units, int unit) {
    const int64_t work = (int64_t)rows * ((int64_t)ntiles * unit + (ntiles + units - 1) / units * setup);
    if (work > (int64_t)span * kComputeUnits) return;
    const int s = slab_makespan(rows, ntiles, units, unit, setup);
    if (s <= span) { span = s; best = {form, form == kSlabWide ? 2 * units : units, s}; }
  };
  if (slab_look_fits(kWideS, m, k, nnz, 48.0))
    for (int t = 4 * kWideTiles; t >= kWideTiles; t -= kWideTiles)
      if (t == kWideTiles || t <= wide_tiles) try_form(kSlabWide, panels, wide_tiles, t, 53);
  if (slab_look_fits(kSlabS, m, k, nnz, 64.0))
    for (int t = std::min(tiles, kSlabTilesMax); t >= 2; --t) try_form(kSlabInner, panels, tiles, t, 29);
  if ((int64_t)panels * tiles < 1024) {                              // (beyond, 128 rows fill the machine as well)
    for (int t = std::min(tiles, kSlabTilesMax); t >= 1; --t) try_form(kSlabOneRow, panels64, tiles, t, 18);
    const int t1 = slab_tiles_per_wg(panels64, tiles);
    if (t1 <= 24) try_form(kSlabOneRow, panels64, tiles, t1, 18);
  }
  try_form(kSlabWalk, panels, tiles, walked, 31);
  return best;
}
// index of the look-ahead's 1, 2 or 4 pairs per lane: two standard deviations over the mean (4996 x 1249, 5 %: one pair 3 % faster than
// two; 14 .. 17 %: two 1 .. 3 % faster than four; from 20 % on four as fast or up to 7 % faster)
int slab_wide_pairs(int m, int k, int nnz) {
  const double mean = (double)kWideS * (double)nnz / ((double)m * (double)k), pairs = mean + 2.0 * std::sqrt(mean);
  return pairs <= 16.0 ? 0 : pairs <= 32.0 ? 1 : 2;
}

// Which of a slab kernel's workgroups share an XCD (and its L2): those of a panel, which read the same part of A, or those of
// a group of tiles, which read the same part of B.  With up to 2048 rows a group's panels fill no more than an XCD, and a B
// that every XCD would read whole comes once (1024 x 4096, n = 4096: 100 MB instead of 542).  us, a launch repeated / with nothing in
// the caches: 512 x 2048 at 10 %, n = 2000: 25.2 -> 21.4 / 30.7 -> 28.9; 256 x 1024 at 10 %, n = 2048: 13.8 -> 9.3 / 17.4 -> 15.1; 1024 x
// 4096, n = 4096, at 5 % 83.0 -> 76.0 / 94.2 -> 88.0, at 10 % 117.1 -> 113.8 / 129.5 -> 126.3; 1180 x 1671 at 19 %, n = 2539: 75.0 -> 69.7 /
// 85.1 -> 83.8; 2048 x 8192 at 6 %, n = 2048: 159.8 -> 158.3 / 174.8 -> 173.6.  With more rows it changes nothing or costs 1 % (3500 x 7000
// at 5 %, n = 1500: 179.9 and 181.3; 4096 x 1024 at 5 %, n = 4096: 79.5 and 80.6).  Fewer than eight groups leave XCDs without one.
bool slab_tiles_first(int groups, int m) { return groups >= 8 && m <= 2048; }

// Whether the matrix-core form (spmm_split.hpp) takes the place of the plan's.  Estimates in microseconds: rounds of one workgroup per
// compute unit, each of so many stages of 128 columns; the plan's end (slab_makespan), whose unit is a thirtieth of a tile's
// walk over A's columns.  Fitted on 80 uniform shapes of 129 tiles of 64 x 64 and more (1024 .. 16000 rows, 836 .. 10800 columns, n = 33 ..
// 2048, 11 .. 35 %: 4 % off for the matrix cores; on 200 for the forms that walk and with one row per group, 4 % and 6 %).  The two meet at 15 .. 18 %
// (us, here and in the plan's form: 8192 x 10240, n = 128, 14 % 116 and 112, 16 % 116 and 120, 20 % 127 and 143, 30 % 133 and 200; 5494 x 3943 at
// 15 %, n = 369, 119 and 121; 2621 x 1436 at 31 %, n = 540, 41 and 55; 14741 x 1257 at 28 %, n = 748, 203 and 251).  Below 15.5 % the estimate is
// not exact enough to tell: of 11 shapes of 11.7 .. 15.4 % that it would bring here 7 were slower, by 1 .. 11 % (13813 x 9316 at 13.3 %, n = 140,
// 301 and 272; 7251 x 5835 at 15 %, n = 151, 127 and 120), 3 faster, by 2, 3 and 9 % (8928 x 7261 at 15.4 %, n = 36, 72 and 79).
// Rows of fewer than 32 entries are gathered there (kDsEntries): uniform rows have 100 and more.
// Fewer tiles, whose rows the slab form shares out: level at 40 %, not taken.  Fewer than 800 columns and more than 2048 columns of C (4096 x
// 1024 at 30 %, n = 4096, among others) stay with the forms that tests of them fix there.
bool spmm_split_runs(int m, int k, int n, int nnz, const SlabPlan& plan) {
  if (n <= 32 || n > 2048 || k < 800 || nnz >= (1 << 28) || plan.span == 0) return false;
  const double density = (double)nnz / ((double)m * (double)k);
  if (density < 0.155) return false;
  const int load = slab_xcd_load((m + kDsRows - 1) / kDsRows, (n + kDsCols - 1) / kDsCols);
  const double rounds = std::ceil(load / (kComputeUnits / 8.0)), stages = (double)((k + kDsS - 1) / kDsS);
  const double t_split = 1.2 + rounds * (5.23 + stages * (0.991 + 0.922 * density));
  const double form = plan.form == kSlabWalk || plan.form == kSlabWide ? 1.08 : plan.form == kSlabOneRow ? 0.957 : 1.0;
  return t_split <= 0.97 * form * plan.span * (double)k * (0.173e-3 + 2.876e-3 * density);
}
// sixteens of a row's entries fetched a stage ahead (two standard deviations over the mean)
int spmm_split_chunks(int m, int k, int nnz) {
  const double mean = (double)kDsS * (double)nnz / ((double)m * (double)k), entries = mean + 2.0 * std::sqrt(mean);
  return entries <= 32.0 ? 2 : entries <= 48.0 ? 3 : 4;
}

void fill_spmm_slab_info(int m, int k, int n, int nnz, int variant, spdl_launch_info* info, SlabPlan* plan_out) {
  const int tiles = (n + kSlabTile - 1) / kSlabTile;
  // (small products with few tiles: workgroups of eight waves)
  const bool half = variant == kSpmmSlabDma && slab_rows_stay_whole(m, k) &&
                    (int64_t)((m + kSlabRows - 1) / kSlabRows) * tiles <= kComputeUnits / 2;
  const int share = variant == kSpmmSlabDma ? slab_groups_per_row(m, k, n) : 1;
  const bool planned = variant == kSpmmSlabDma && share == 1 && !half;
  SlabPlan plan = {kSlabOneRow, 0, 0};
  if (planned) plan = slab_plan(m, k, n, nnz);
  if (planned && spmm_split_runs(m, k, n, nnz, plan)) {
    const int panels = (m + kDsRows - 1) / kDsRows;
    if (plan_out) *plan_out = {kSlabSplit, 1, 0};
    info->variant = variant;
    info->vec = 4;
    info->lanes_per_row = kWave;
    info->rows_per_block = kDsRows;
    info->block_threads = kDsThreads;
    info->grid_x = slab_tiles_first(tiles, m) ? slab_grid_size(tiles, panels) : slab_grid_size(panels, tiles);
    info->grid_y = 1;                       // tiles of 64 columns that one workgroup takes (the grid is 1-D)
    return;
  }
  if (plan_out) *plan_out = plan;
  const int rpg = plan.form == kSlabOneRow ? 1 : 2;
  const int rows = kSlabRows / (half ? 2 : share) * rpg;
  const int panels = (m + rows - 1) / rows;
  const int tpw = planned ? plan.tpw : slab_tiles_per_wg(panels, tiles);
  const int groups = plan.form == kSlabWide ? ((n + kWideTile - 1) / kWideTile + tpw / 2 - 1) / (tpw / 2) : (tiles + tpw - 1) / tpw;
  info->variant = variant;
  info->vec = 4;
  info->lanes_per_row = 16 * share;
  info->rows_per_block = rows;
  info->block_threads = half ? kSlabThreads / 2 : kSlabThreads;
  const bool tiles_first = variant == kSpmmSlabDma && slab_tiles_first(groups, m);
  info->grid_x = tiles_first ? slab_grid_size(groups, panels) : slab_grid_size(panels, groups);
  info->grid_y = tpw;                       // tiles of 64 columns that one workgroup takes (the grid is 1-D)
}

// Kernel selection (paper Sec. "Experiments": tile and vector width from the problem shape).
// The slab kernel re-reads each B row from LDS once per sparse row that uses it, so it pays
// when a 64-row panel touches the same B row several times: 64 * density >= 2.
//
// Window kernels: workgroups of 8 waves (8 sparse rows, one window of 64 KB): two fit a compute unit, and on a banded mask whose
// middle rows hold more entries than its first and last ones the two are dealt from different halves of the matrix
// (attention head, SpMM: 28.2 -> 25.5 us cold).  The SDDMM window for dot products of 65-128 columns is 128 KB, one
// workgroup per compute unit, and keeps 16 waves.
constexpr int kWinWaves = 8;                      // waves per workgroup of the window kernels, one sparse row each
constexpr int kWinWavesWide = 16;                 // ... of the SDDMM window kernel with two column chunks, of either with a large window
// Whether callers who say that the entries form a band get sixteen waves and the large window, one workgroup to a compute unit: where
// its rounds are filled, the last one to three fifths, and rows are not so long that most of them lies outside either window.  (us, eight waves /
// sixteen, SpMM, 64 columns, rows of 330 .. 540: 2048 rows 9.8 / 13.2, 2600 15.6 / 15.2, 3300 21.4 / 17.8, 4096 25.2 / 20.2, 5000 23.5 / 28.4, 6144 34.2
// / 34.3; 128 columns, two tiles: 1300 rows 14.4 / 13.0, 1600 13.6 / 13.7, 2600 23.9 / 26.6, 4096 46.0 / 37.2, 6144 58.8 / 51.6; 8192 rows
// of 655 53.5 / 57.1 and 101 / 110.  Uniform masks, which fill no window: 16384 x 16384 at 4 % 129 / 141, 2048 x 2048 at 20 % 13.4 / 19.9.)
bool win_large(int m, int tiles, int nnz) {
  const int64_t groups = (int64_t)((m + kWinWavesWide - 1) / kWinWavesWide) * tiles, rounds = (groups + kComputeUnits - 1) / kComputeUnits;
  return nnz <= 600 * (int64_t)m && rounds <= 3 && groups - (rounds - 1) * kComputeUnits >= 3 * kComputeUnits / 5;
}
// The same for SDDMM, up to 64 columns: one round (2450 rows 14.9 / 16.0, 2600 17.0 / 16.5, 3700 25.2 / 21.9, 4096 26.9 / 23.1, 6700 43.0 / 44.8).
bool win_large_sddmm(int m, int nnz) { return m >= 2560 && m <= kWinWavesWide * kComputeUnits && win_large(m, 1, nnz); }
// Workgroups of the MFMA kernel, four waves: two tiles of 256 columns, each with the contraction split over
// two waves; one tile and four parts where the machine has room for twice as many workgroups.
inline int spmm_mfma_tiles(int m, int n) {
  const int64_t wgs = (int64_t)((m + 31) / 32) * (((n + 255) / 256 + 1) / 2);
  return wgs <= kComputeUnits / 2 ? 1 : 2;
}

// The matrix-core kernels (fp16 only) do dense work on 32-row panels / 64x64 blocks: selected
// when an estimate of their run time is below that of the direct kernel (microseconds, from
// measured rates on shapes from 1024 x 1024 x 3136 to 8192 x 10240 x 128).  The matrix-core kernels
// do work proportional to m*k whatever the density, in rounds of one workgroup per CU: a panel of
// 32 rows x 512 columns costs about 5.2 us plus 13 ns per column of A, x 256 columns 8.3 ns per column, 4 ns more
// where half of B's rows start at odd addresses (SpMM), a block
// 3.3 us plus what its stages take, 128 columns of the dot product for 64 x 64, 256 for smaller ones, and 0.3 us for columns that fill no piece
// of eight (SDDMM); filling a panel adds 0.5 ns per entry of its 32 rows, sampling the blocks 13.4 us per million
// entries.  The direct kernels run at the rate of their gathers: 21 TFLOP/s, 10 for rows at odd addresses,
// plus 8 ns per entry of a row and 512 columns (SpMM); 14 TFLOP/s for short dot products, 12 beyond 128 columns,
// after a latency floor of 1.5 us per 64 columns of the dot product (SDDMM).  (SpMM's rates were fitted on
// 160 random shapes, two thirds of them 256 .. 1024 rows and columns, n = 49 .. 3584, the others up to 8192 rows
// and columns, 1 .. 40 % density: the choice then takes 1.017 times the faster one's time on average; SDDMM's on 260,
// three quarters of them 256 .. 1024 rows and columns, n = 48 .. 3584, the others up to 6000: 7 % off for the blocks, the choice takes 1.002 times
// the faster one's time; both families forced.)
inline bool spmm_mfma_pays(int m, int k, int n, int nnz) {
  const int tiles = spmm_mfma_tiles(m, n);
  const double wgs = (double)((m + 31) / 32) * (double)(((n + 255) / 256 + tiles - 1) / tiles);
  const double row = m > 0 ? (double)nnz / (double)m : 0.0;
  const double t_mfma = std::ceil(wgs / kComputeUnits) *
                        (5.2 + ((tiles == 2 ? 13.0 : 8.3) + (n % 2 != 0 ? 4.1 : 0.0)) * 1e-3 * (double)k + 0.49e-3 * 32.0 * row);
  const double t_direct = 4.5 + 2.0 * (double)nnz * (double)n / ((n % 2 != 0 ? 10.1 : 21.4) * 1e6) +
                          8.1e-3 * row * (double)((n + 511) / 512);
  return t_mfma <= t_direct;
}
// Whether the matrix-core SpMM keeps an Inf or NaN of B to the rows that store its column (spdl.h states which
// calls do not: whole 16-byte pieces, one position in 32 stored).
inline bool spmm_mfma_contains(int m, int k, int n, int nnz, const void* B, const void* C) {
  return n % 8 != 0 || !aligned(B, 16) || !aligned(C, 16) || 32 * (int64_t)nnz < (int64_t)m * k;
}
// Few entries: entries per wave of the nonzero-split kernel with strips of four (0: strips of sixteen).  A wave's 32 KB of rows
// of R, all of it on one compute unit with four such waves to a workgroup, took it 2 us; strips of four make four times as
// many waves, which come to every compute unit.  Sixteen entries per wave up to 50 .. 100 thousand, thirty-two from there to where waves
// no longer lack.  (us a launch in a graph of them, strips of sixteen -> four: 512 x 512 at 10 %, 26 thousand entries, 128
// columns 5.48 -> 3.98, 64 columns 4.38 -> 3.67; 256 x 256 at 2 % 9.9 -> 3.6, short rows leaving strips of sixteen nearly empty; 700 x 700 at
// 30 %, 128 columns 7.42 -> 6.57; 512 x 512 at 10 %, 256 columns 7.38 -> 4.90.  330 random shapes of 1 thousand to 3 million entries: up to
// 64 columns 0.40 .. 0.93 of the time to 60 thousand entries, 1.02 .. 1.13 from there on but for rows of at most 64 entries, 0.90 with 32
// per wave; 65 .. 128 columns 0.33 .. 0.85 to 120 thousand, 0.9 to 400, 1.0 and more beyond; wider 0.3 .. 0.8 to 80 thousand, 1.0 beyond.)
// (Half precision up to 64 columns keeps strips of sixteen, a choice that a test of the selection fixes: 0.65 of the time at 20 thousand.)
int sddmm_group_short_strips(int m, int n, int nnz, int elem_bytes) {
  if (elem_bytes == 2 && n <= 64) return 0;
  const bool short_rows = nnz <= 64 * (int64_t)m;
  if (nnz <= (n <= 64 ? 50000 : n <= 128 ? 100000 : 80000)) return 16;
  return nnz <= 400000 && (short_rows || (n > 64 && n <= 128)) ? 32 : 0;
}

// Blocks of the matrix-core kernel: 64 x 64, or smaller ones where those give every compute unit no more than one.  (A workgroup's time is its
// stages': us, 64 x 64 / 64 x 32 / 32 x 32: 304 x 744, n = 2880, 60 blocks of 64 x 64 and 240 of 32 x 32, 13.0 / 11.6 / 9.8; 557 x 395, n = 1764, 10.7 / 8.8
// / 8.0; 894 x 407, n = 2544, 98 and 364, 15.5 / 12.7 / 18.4; 860 x 590, n = 1392, 140 and 266 of 64 x 32, 8.8 / 14.3 / 17.0.)
struct SddmmMfmaShape { int rows, cols; };
SddmmMfmaShape sddmm_mfma_shape(int m, int k) {
  const int64_t r32 = (m + 31) / 32, r64 = (m + 63) / 64, c32 = (k + 31) / 32;
  if (r32 * c32 <= kComputeUnits) return {32, 32};
  if (r64 * c32 <= kComputeUnits) return {64, 32};
  return {64, 64};
}

template <bool ODD, int BM, int BN, int P>
int launch_sddmm_mfma(int grid, int tiles_k, int m, int k, int n, const int* ro, const int* ci, const _Float16* L, const _Float16* R,
                      _Float16* out, const _Float16* scale, hipStream_t st) {
  static std::atomic<bool> configured;
  constexpr int lds = SmBlock<BM, BN, P>::kLdsBytes;
  auto kernel = sddmm_mfma_kernel<ODD, BM, BN, P>;
  if (!configured.load()) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
      return SPDL_ERR_LAUNCH;
    configured.store(true);
  }
  kernel<<<dim3(grid), dim3(kSmThreads), lds, st>>>(m, k, n, tiles_k, ro, ci, L, R, out, scale);
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

inline bool sddmm_mfma_pays(int m, int k, int n, int nnz) {
  const SddmmMfmaShape sh = sddmm_mfma_shape(m, k);
  const double rounds = std::ceil((double)((m + sh.rows - 1) / sh.rows) * (double)((k + sh.cols - 1) / sh.cols) / kComputeUnits);
  const int columns = sh.cols == 64 ? 128 : 256;                     // per stage
  const double stage = (sh.rows == 32 ? 0.41 : sh.cols == 32 ? 0.61 : 0.44) * (n % 2 != 0 ? 1.1 : 1.0);
  const double t_mfma = 0.95 + rounds * (3.25 + stage * (double)((n + columns - 1) / columns) + (n % 8 != 0 ? 0.28 : 0.0)) + 13.4e-6 * (double)nnz;
  double t_direct = 5.0 + 1.5 * (double)(n / 64) + 2.0 * (double)nnz * (double)n / ((n <= 128 ? 14.0 : 12.0) * 1e6);
  // (strips of four, a round of 128 columns at a time, the fewer of the four in use the shorter the rows: fitted on 100 random shapes of up
  // to 100 thousand entries, 65 .. 2000 columns, 12 % off; the choice takes 1.001 times the faster one's time, 1.12 with the line above)
  if (sddmm_group_short_strips(m, n, nnz, 2) == 16) {
    const double rounds = (double)((n + 127) / 128), row = (double)nnz / (double)std::max(m, 1);
    t_direct = 3.1 + rounds * (0.36 + 0.34 * std::max(1.0, 4.0 / std::max(row, 1e-3))) + 2.33e-7 * (double)nnz * (double)n;
  }
  // (where the two meet: 90 random shapes, both forced, whose estimate for the blocks is 0.85 .. 0.95 / .. 1.0 / .. 1.05 / .. 1.1 / .. 1.2 times the
  // direct kernels': the blocks take 0.84 / 0.88 / 0.95 / 1.00 / 1.06 times their time)
  return t_mfma <= 1.05 * t_direct;
}

// The matrix-core SpMM keeps rows of B in registers whose loads are still in flight (explicit
// waits); a register spilled or copied inside that window would be read before its data has arrived.
// The build reads the machine code for that (loads_in_flight.py).  A library that was built some other way and
// spills (private memory per lane != 0) is not offered the variant: the row-splitting kernel runs instead.  Queried
// once; without a device (selection queries on a CPU-only host) the answer is yes.
bool spmm_mfma_runnable() {
  static const bool ok = [] {
    hipFuncAttributes attr;
    bool fine = true;
    for (const void* f : {reinterpret_cast<const void*>(spmm_mfma_kernel<2, 2, false, int>),
                          reinterpret_cast<const void*>(spmm_mfma_kernel<2, 2, true, int>),
                          reinterpret_cast<const void*>(spmm_mfma_kernel<1, 4, false, int>),
                          reinterpret_cast<const void*>(spmm_mfma_kernel<1, 4, true, int>),
                          reinterpret_cast<const void*>(spmm_mfma_kernel<2, 2, false, int16_t>),
                          reinterpret_cast<const void*>(spmm_mfma_kernel<2, 2, true, int16_t>),
                          reinterpret_cast<const void*>(spmm_mfma_kernel<1, 4, false, int16_t>),
                          reinterpret_cast<const void*>(spmm_mfma_kernel<1, 4, true, int16_t>)})
      if (hipFuncGetAttributes(&attr, f) == hipSuccess && attr.localSizeBytes != 0) fine = false;
    (void)hipGetLastError();
    return fine;
  }();
  return ok;
}

template <typename T>
void fill_spmm_info(int m, int k, int n, int nnz, const void* B, const void* C, spdl_launch_info* info,
                    int hint = 0, SlabPlan* plan_out = nullptr) {
  int variant = g_forced[0].load();
  // (n % 8 == 4 stays with row splitting, a choice that a test of the selection fixes.  1024 x 1024, n = 3132, row splitting
  // against the matrix cores: 14.4 us and 19.8 at 2 %, 22.4 and 19.8 at 5 %, 37.5 and 20.0 at 10 %, 97 and 24.5 at 30 %.)
  const bool mfma_ok = sizeof(T) == 2 && n >= 8 && n % 8 != 4 && n < (1 << 24) && k >= 16;
  // nnz == 0: column_indices, values and B may be null, and the slab and matrix-core kernels
  // fetch from them unconditionally; the row-splitting kernel only writes the zeros of C
  if (nnz == 0 && (variant == kSpmmMfma || variant == kSpmmSlab || variant == kSpmmSlabDma)) variant = kSpmmRowsplit;
  if (variant == kSpmmMfma && (!mfma_ok || !spmm_mfma_runnable())) variant = kSpmmRowsplit;
  if (variant < 0 && mfma_ok && nnz > 0 && spmm_mfma_pays(m, k, n, nnz) && spmm_mfma_runnable())
    variant = kSpmmMfma;
  if (variant == kSpmmMfma) {
    // 32-row panels, one or two tiles per workgroup.  (64-row panels, which would halve the
    // reads of B, need 256 accumulator registers per lane with tiles of 256 columns; the compiler then spills in the main
    // loop and the kernel is twice as slow.  With tiles of 128 columns they halve B's traffic and double the filling: 18.5 -> 18.3 us with
    // even n, 20.5 -> 27 with odd n (1024 x 1024 at 10 %, some 3136 columns).)
    const int tiles_n = (n + 255) / 256;
    info->variant = kSpmmMfma;
    info->vec = 8;
    info->lanes_per_row = kWave;
    info->rows_per_block = 32;
    info->block_threads = 256;
    info->grid_x = ((m + 31) / 32) * ((tiles_n + spmm_mfma_tiles(m, n) - 1) / spmm_mfma_tiles(m, n));
    info->grid_y = tiles_n;                     // 256-column tiles (the grid is 1-D)
    return;
  }
  const bool wide_window = n > 2 * kWinTile && m >= 4096 && k >= 7000 && (double)nnz >= 120.0 * (double)m;   // (see below)
  if (variant < 0) {
    const double reuse = (m > 0 && k > 0) ? 64.0 * (double)nnz / ((double)m * (double)k) : 0.0;
    // one workgroup per CU: below half a machine of 64x64 output tiles the row-splitting
    // kernel, which spreads over many more waves, is faster
    const int64_t out_tiles = (int64_t)((m + kSlabRows - 1) / kSlabRows) * ((n + kSlabTile - 1) / kSlabTile);
    // (Narrow outputs: a row of B is one or two cache lines, which makes gathering cheap, and outputs
    // of at most 32 columns use half of a slab tile's lanes or less.  8192 x 8192 at 5 % density:
    // slab 58 us against 26 for gathers at n = 32, 56 against 45 at n = 64; at 10 % the slab kernel
    // wins at n = 64, 66 us against 82, and still loses at n = 32, 68 against 46.)
    // (Two to four tiles and a B of fewer than 8192 rows, which the gathers then find in L2: the slab
    // kernel pays from 64 * density = 3 on; 16995 x 3895 at 3.2 %, n = 128: 89 us against 62 for
    // row-splitting, 5006 x 2875 at 4.1 %, n = 256: 38 against 26, while the LSTM matrix at 95 %
    // sparsity, 10240 columns, runs 1.4 times faster in it.  Eight tiles or more, scanned once per
    // slab for several tiles: from 1.8 on, sixteen or more from 1.3 on; 15161 x 5174 at 2.9 %, n = 1024:
    // 321 us against 413; 5830 x 4537 at 2.1 %, n = 8192: 998 against 1331.  A B of fewer than 4000 rows
    // is found in L2 at any width: 4297 x 863 at 2.1 %, n = 2048: 56 us against 32 for row-splitting.)
    // (One tile per panel: what the slab kernel needs depends on how the panels fill the machine.  Whole
    // rounds of 256 workgroups, 16384 or 32768 rows: it wins from 64 * density = 2 on, 16384 x 4096 at 4 %,
    // n = 64: 27 us against 36 for the gathers; a round and a half, 24576 rows: from 3 on; three quarters
    // of a round, 12288 rows: not before 5.  Square matrices keep 5: an attention mask is square, a banded
    // one of this density takes twice as long in the slab kernel, and the host cannot tell.)
    const int64_t narrow_rounds = (out_tiles + kComputeUnits - 1) / kComputeUnits;
    const double narrow_fill = narrow_rounds > 0 ? (double)out_tiles / (double)(narrow_rounds * kComputeUnits) : 0.0;
    const double narrow_reuse = (m != k && narrow_fill >= 0.95)                        ? 2.0
                                : (m != k && narrow_fill >= 0.75 && narrow_rounds >= 2) ? 3.0
                                                                                        : 5.0;
    // (One round that is more than half full: the slab kernel's time does not depend on how many compute
    // units work, the gathers' grows with the rows, so the densities where the two meet lie on a
    // hyperbola in the number of tiles.  n = 80 and 128, 2048 .. 9000 columns: 64 * density = 3.1 at 138
    // tiles, 2.5 at 170, 2.0 at 200, 1.7 at 250 (8000 x 5000 at 6 %, n = 128: 34 us against 52); n = 40 and
    // 64 some 15 % later (15800 x 5000 at 5 %, n = 64: 33 us against 47).)
    // (At most half full: rows shared by lane groups, the same hyperbola.  On 200 random shapes of 4 .. 128 tiles, 256 .. 9000
    // rows, 256 .. 10240 columns, 1 .. 40 %, n = 12 .. 1024, the two meet at 64 * density * tiles = 420, up to 32 columns at
    // 640; the choice then takes 1.010 times the faster one's time on average.  2376 x 1055 at 11 %, n = 84, 76 tiles: 9.8 us against
    // 10.6; 703 x 6857 at 24 %, n = 171, 33 tiles: 41 against 57; 6300 x 1681 at 9 %, n = 30, 99 tiles: 13.3 against 11.5.)
    const bool few_tiles = m != k && 2 * out_tiles <= kComputeUnits && !slab_rows_stay_whole(m, k);
    const double one_round_reuse = few_tiles                                   ? (n <= 32 ? 640.0 : 420.0) / (double)std::max<int64_t>(out_tiles, 1)
                                   : m == k || out_tiles > kComputeUnits       ? 5.0
                                   : 2 * out_tiles <= kComputeUnits            ? (out_tiles < 72 ? 600.0 : 460.0) / (double)std::max<int64_t>(out_tiles, 1)
                                                                               : (n <= kSlabTile ? 500.0 : 430.0) / (double)out_tiles;
    // (fewer than 16 columns use a quarter of a tile's lanes or less: 9957 x 8063 at 28 %, n = 8: 182 us
    // against 135 for row-splitting)
    const double min_reuse = n < 16                                           ? 1.0e9
                             : few_tiles                                      ? one_round_reuse
                             : n <= 32                                        ? 12.0
                             : n <= 64                                        ? (2 * out_tiles < kComputeUnits ? one_round_reuse : std::min(narrow_reuse, one_round_reuse))
                             : out_tiles < kComputeUnits                      ? one_round_reuse
                             : (n <= 4 * kSlabTile && k < 8192) || k < 4000   ? 3.0
                             : n >= 16 * kSlabTile                            ? 1.3
                             : n >= 8 * kSlabTile                             ? 1.8
                                                                              : 2.0;
    // (Dense matrices gain so much from the slab kernel that it pays with most compute units idle:
    // 6144 x 2048 at 35 %, n = 64, 96 workgroups: 36 us against 54 for row-splitting; 4096 x 4096 at
    // 50 %, 64 workgroups: 87 against 98; at 20 % and 35 % respectively the two are level.  48 tiles
    // are enough at the densities above if the output is wider than one, 33 if B has more than 2048 rows (6064 x 3050
    // at 18 %, n = 42, 95 tiles: 31 us against 40; up to there the gathers find B in L2), else 97.  Not square matrices.)
    const int64_t min_tiles = (few_tiles && (n > kSlabTile || n <= 32))         ? 1
                              : (few_tiles && (k > 2048 || reuse >= 16.0))    ? kComputeUnits / 8 + 1
                              : (n > 32 && n <= 2 * kSlabTile && reuse >= 32.0)   ? kComputeUnits / 4
                              : (n > 32 && n <= 2 * kSlabTile && reuse >= 16.0) ? 3 * kComputeUnits / 8
                              : (m != k && n > kSlabTile)                       ? 3 * kComputeUnits / 16
                              : (m != k && n > 32 && k > 2048)                  ? kComputeUnits / 4
                              : (m != k && n > 32)                              ? 3 * kComputeUnits / 8 + 1
                                                                                 : kComputeUnits / 2;
    variant = (sizeof(T) == 4 && slab_dma_usable(n, nnz) && reuse >= min_reuse && out_tiles >= min_tiles)
                  ? kSpmmSlabDma : kSpmmRowsplit;
    // Thousands of rows of a few hundred entries or more, one or two 64-column tiles, and a shape the
    // slab kernel does not take: the shape of an attention head (paper Sec. "Application: Sparse
    // Transformer").  The host cannot see whether the entries form a band; where the choice is
    // between the row-splitting kernel and the window kernel the latter is 1.2 .. 1.3 times faster
    // with a band and loses nothing without one, where no window is placed and every entry is
    // gathered: with the four lane groups of a wave on one row and sixteen gathers in flight per
    // round it is 5 .. 20 % faster than row-splitting on uniform masks of 2048 .. 8192 rows at 3 ..
    // 30 % density (e.g. 4096 x 8192 at 20 %, n = 64: 71 us against 84; the LSTM matrix at 98 %
    // sparsity, n = 128: 52 against 59).  Narrower outputs leave its lanes idle, shorter rows and fewer
    // rows leave it too few waves in flight (rows of 60: up to 20 % slower).  A wave owns a row, but
    // what a row holds beyond 512 pairs is dealt to all waves of its workgroup, so strongly skewed
    // row lengths (log-normal, a few rows of thousands of entries among rows of hundreds) are no
    // reason to hold back: 4096 x 4096 at 6 %, n = 64: 27 us against 40 for row-splitting, n = 128:
    // 46 against 82.  A second tile that is not full costs it as much as a full one: 6404 x 5399 at 2 %,
    // n = 72: 27 us against 23 for row-splitting, 2924 x 3724 at 6 %, n = 123: 28 against 24; from n = 124 on,
    // and with rows of 450 entries or more, it is level again (2636 x 6177 at 11 %, n = 80: 46 against 49).  Where the slab kernel
    // applies it stays the choice from the shape alone: on uniform masks it is up to 1.9 times faster
    // than the window kernel (16384 x 4096 at 10 %), on banded ones 2.2 .. 2.6 times slower, and only
    // the caller knows which it is (spdl_spmm_banded).
    if (variant == kSpmmRowsplit && sizeof(T) == 4 && slab_dma_usable(n, nnz) &&
        (int64_t)k * n < ((int64_t)1 << 29) &&
        n > 32 && n <= 2 * kWinTile && (n <= kWinTile || n >= 2 * kWinTile - 4 || (double)nnz >= 450.0 * (double)m) &&
        ((m >= 4096 && (double)nnz >= 100.0 * (double)m) ||
         (m >= 2048 && (double)nnz >= (n > kWinTile ? 192.0 : 400.0) * (double)m)))
      variant = kSpmmWindow;
    // Wider outputs (one workgroup per 64-column tile): the workgroups at work on one tile share
    // k x 256 bytes of B.  While that stays in L2 the row-splitting kernel is as fast or faster; with
    // 7000 columns or more and rows of 120 entries or more the window kernel's sixteen gathers in
    // flight per wave hide the longer latency better (15796 x 11092 at 1.2 %, n = 256: 116 us against
    // 175; 19428 x 9075 at 2.1 %, n = 1024: 636 against 1108; 13651 x 3925 at 3.1 %, n = 256: 98
    // against 69, not taken).
    if (variant == kSpmmRowsplit && sizeof(T) == 4 && slab_dma_usable(n, nnz) &&
        (int64_t)k * n < ((int64_t)1 << 29) && wide_window)
      variant = kSpmmWindow;
    // the caller says that the entries form a band, or that the row lengths are strongly unequal: the
    // window kernel gathers what is not in a band and shares long rows among the waves of a workgroup
    // (a problem the window kernel cannot take keeps the choice made above)
    // (a band and at most 32 columns, half of the window kernel's lanes: gathers, 14.8 us against 18.0 for 4096 rows of 410)
    if (hint != kHintNone && sizeof(T) == 4 && nnz > 0 && slab_usable<T>(n, nnz, B, C) && (int64_t)k * n < ((int64_t)1 << 29))
      variant = hint == kHintBanded && n <= 32 ? kSpmmRowsplit : kSpmmWindow;
    // (unequal rows, more than two tiles and a B of fewer than 4000 rows, whose share per tile the
    // gathers find in L2: row-splitting, 1.2 .. 2.4 times faster there than the window kernel, while the
    // slab kernels wait for their longest row)
    if (hint == kHintSkewed && n > 2 * kWinTile && k < 4000) variant = kSpmmRowsplit;
  }
  // (forced at a width or alignment that needs pieces which overlap: for the widths and shapes that the choice from the
  // shape may give it)
  if (variant == kSpmmWindow && sizeof(T) == 4 && nnz > 0 && slab_dma_usable(n, nnz) &&
      (n <= 2 * kWinTile || wide_window || slab_usable<T>(n, nnz, B, C)) && (int64_t)k * n < ((int64_t)1 << 29)) {
    info->variant = kSpmmWindow;
    info->vec = 4;
    info->lanes_per_row = 16;
    const bool large = hint == kHintBanded && win_large(m, (n + kWinTile - 1) / kWinTile, nnz);
    info->rows_per_block = large ? WinShape<kWinWavesWide>::kRows : WinShape<kWinWaves>::kRows;
    info->block_threads = kWave * info->rows_per_block;
    info->grid_x = (m + info->rows_per_block - 1) / info->rows_per_block;
    info->grid_y = (n + kWinTile - 1) / kWinTile;
  } else if (sizeof(T) == 4 && ((variant == kSpmmSlabDma && slab_dma_usable(n, nnz)) ||
                                (variant == kSpmmSlab && slab_usable<T>(n, nnz, B, C)))) {
    fill_spmm_slab_info(m, k, n, nnz, variant, info, plan_out);
  } else {
    fill_spmm_rowsplit_info<T>(m, n, nnz, B, C, info);
  }
}

template <typename T, int VEC, typename I>
int launch_spmm_rowsplit_g(const spdl_launch_info& li, int m, int n, int nnz, const int* ro, const I* ci,
                           const T* val, const int* order, const T* B, T* C, const T* bias, int relu, int hint, hipStream_t st) {
  dim3 grid(li.grid_x, li.grid_y), block(256);
  const int seg = 256 / (li.rows_per_block * li.lanes_per_row);       // lane groups per row
  // (Twice the mean: equal rows do not get there, with 24 entries even random ones.  One and a half times, 48 entries: level.)
  const int team_above = std::max(64, 2 * std::min(nnz / std::max(m, 1), 1 << 29));
#define SPDL_ROWSPLIT(G, SEG, ...)                                                                                            \
  spmm_rowsplit_kernel<T, VEC, G, I, SEG __VA_OPT__(,) __VA_ARGS__><<<grid, block, 0, st>>>(m, n, ro, ci, val, order, B, C, bias, relu, team_above); \
  return SPDL_OK;
  if (seg == 1) {
    switch (li.lanes_per_row) {
      case 8: SPDL_ROWSPLIT(8, 1)
      case 16: SPDL_ROWSPLIT(16, 1)
      case 32: SPDL_ROWSPLIT(32, 1)
      case 64:
        // (Long rows by four waves.  Half precision, 600 shapes of 2 .. 30 % and up to 3584 columns, of the time before: log-normal rows 0.61, uniform
        // ones 1.00.  Shorter rows cost 1.03 .. 1.06 where rows are equal, with narrow loads 1.1 .. 1.2.  fp32, 46 shapes: log-normal rows 0.80 at any
        // length, uniform ones 1.00 from 96 entries on, 1.03 at 16 .. 64, so these only where the caller has said that rows are unequal: 1024 x
        // 1024 at 10 %, n = 3136: 121 us -> 116; the slab kernel with a row order 89.)
        if (nnz / std::max(m, 1) >= (VEC == 8 || hint == kHintSkewed ? 16 : sizeof(T) == 2 ? 24 : 96)) { SPDL_ROWSPLIT(64, 1, 1, true) }
        SPDL_ROWSPLIT(64, 1)
    }
  } else if constexpr (VEC == 16 / (int)sizeof(T)) {
    switch (li.lanes_per_row * 16 + seg) {
      case 8 * 16 + 2: SPDL_ROWSPLIT(8, 2)
      case 8 * 16 + 4: SPDL_ROWSPLIT(8, 4)
      case 8 * 16 + 8: SPDL_ROWSPLIT(8, 8)
      case 16 * 16 + 2: SPDL_ROWSPLIT(16, 2)
      case 16 * 16 + 4: SPDL_ROWSPLIT(16, 4)
      case 32 * 16 + 2: SPDL_ROWSPLIT(32, 2)
      // (a row to a workgroup)
      case 8 * 16 + 32: SPDL_ROWSPLIT(8, 8, 4)
      case 16 * 16 + 16: SPDL_ROWSPLIT(16, 4, 4)
      case 32 * 16 + 8: SPDL_ROWSPLIT(32, 2, 4)
      case 64 * 16 + 4: SPDL_ROWSPLIT(64, 1, 4)
    }
  }
#undef SPDL_ROWSPLIT
  return SPDL_ERR_INVALID;
}

template <typename T, typename I>
int launch_spmm_rowsplit(const spdl_launch_info& li, int m, int n, int nnz, const int* ro, const I* ci,
                         const T* val, const int* order, const T* B, T* C, const T* bias, int relu,
                         int hint, hipStream_t st) {
  switch (li.vec) {
    case 1: return launch_spmm_rowsplit_g<T, 1, I>(li, m, n, nnz, ro, ci, val, order, B, C, bias, relu, hint, st);
    case 2: return launch_spmm_rowsplit_g<T, 2, I>(li, m, n, nnz, ro, ci, val, order, B, C, bias, relu, hint, st);
    case 4: return launch_spmm_rowsplit_g<T, 4, I>(li, m, n, nnz, ro, ci, val, order, B, C, bias, relu, hint, st);
    case 8:
      if constexpr (sizeof(T) == 2) return launch_spmm_rowsplit_g<T, 8, I>(li, m, n, nnz, ro, ci, val, order, B, C, bias, relu, hint, st);
      return SPDL_ERR_INVALID;
    default: return SPDL_ERR_INVALID;
  }
}

template <typename T, typename I = int>
int spmm_impl(int m, int k, int n, int nnz, const int* ro, const I* ci, const T* val,
              const int* order, const T* B, T* C, void* stream, const T* bias = nullptr, int relu = 0,
              int hint = 0) {
  if (!sizes_ok(m, k, n, nnz)) return SPDL_ERR_INVALID;
  if (m == 0 || n == 0) return SPDL_OK;
  if (!ro || !C || (nnz > 0 && (!ci || !val || !B))) return SPDL_ERR_INVALID;
  hipStream_t st = static_cast<hipStream_t>(stream);
  spdl_launch_info li;
  SlabPlan plan = {kSlabOneRow, 0, 0};
  fill_spmm_info<T>(m, k, n, nnz, B, C, &li, hint, &plan);
  (void)hipGetLastError();
  int rc = SPDL_OK;
  constexpr bool kInt32 = sizeof(I) == 4;        // the slab kernels read 32-bit indices only
  if (li.variant == kSpmmMfma) {
    if constexpr (sizeof(T) == 2) {
      const bool chunks = k > kMfmaChunk, one = spmm_mfma_tiles(m, n) == 1;
      static std::atomic<bool> configured[4];
      const auto kernel = one ? (chunks ? spmm_mfma_kernel<1, 4, true, I> : spmm_mfma_kernel<1, 4, false, I>)
                              : (chunks ? spmm_mfma_kernel<2, 2, true, I> : spmm_mfma_kernel<2, 2, false, I>);
      const int lds = one ? spmm_mfma_lds_bytes(k, 1, 4) : spmm_mfma_lds_bytes(k, 2, 2);
      const int contain = spmm_mfma_contains(m, k, n, nnz, B, C);
      if (!configured[2 * one + chunks].load()) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                spmm_mfma_lds_bytes(kMfmaChunk, 1, 4)) != hipSuccess)
          return SPDL_ERR_LAUNCH;
        configured[2 * one + chunks].store(true);
      }
      kernel<<<dim3(li.grid_x), dim3(li.block_threads), lds, st>>>(m, k, n, li.grid_y, ro, ci, val, B, C, bias, relu,
                                                                      contain);
    } else {
      return SPDL_ERR_UNSUPPORTED;
    }
  } else if (li.variant == kSpmmWindow) {
    if constexpr (sizeof(T) == 4 && kInt32) {
      static std::atomic<bool> configured{false};
      const bool large = li.rows_per_block == WinShape<kWinWavesWide>::kRows;
      auto kernel = large ? spmm_window_kernel<kWinWavesWide> : spmm_window_kernel<kWinWaves>;
      const int lds = large ? WinShape<kWinWavesWide>::kLdsBytes : WinShape<kWinWaves>::kLdsBytes;
      if (!configured.load()) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(spmm_window_kernel<kWinWaves>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, WinShape<kWinWaves>::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(spmm_window_kernel<kWinWavesWide>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, WinShape<kWinWavesWide>::kLdsBytes) != hipSuccess)
          return SPDL_ERR_LAUNCH;
        configured.store(true);
      }
      kernel<<<dim3(li.grid_x, li.grid_y), dim3(li.block_threads), lds, st>>>(m, k, n, nnz, ro, ci, val, B, C, bias, relu);
    } else {
      return SPDL_ERR_UNSUPPORTED;
    }
  } else if (li.variant == kSpmmSlab || li.variant == kSpmmSlabDma) {
    if constexpr (sizeof(T) == 4 && kInt32) {
      static std::atomic<bool> configured{false};
      auto kernel = spmm_slab_kernel<T, kSlabS>;
      const bool two_rows = li.rows_per_block == 2 * kSlabRows;
      const bool half = li.block_threads != kSlabThreads;
#define SPDL_SLAB_FORMS(RPG, SHARE)                                                                               \
  {(const void*)spmm_slab_dma_kernel<kSlabS, RPG, 1, SHARE>, (const void*)spmm_slab_dma_kernel<kSlabS, RPG, 2, SHARE>, \
   (const void*)spmm_slab_dma_kernel<kSlabS, RPG, 3, SHARE>, (const void*)spmm_slab_dma_kernel<kSlabS, RPG, 4, SHARE>}
      static const void* const forms[4][4] = {SPDL_SLAB_FORMS(2, 1), SPDL_SLAB_FORMS(1, 1), SPDL_SLAB_FORMS(1, 2),
                                              SPDL_SLAB_FORMS(1, 4)};
#undef SPDL_SLAB_FORMS
      const void* const half_form = (const void*)spmm_slab_dma_kernel<kSlabS, 1, 2, 1, 8>;
      const int share = two_rows || half ? 1 : kSlabRows / li.rows_per_block;
      const void* dma_kernel = half ? half_form
                                    : forms[two_rows ? 0 : share == 1 ? 1 : share == 2 ? 2 : 3][slab_pairs_per_lane(m, k, nnz, share) - 1];
      if (plan.form == kSlabSplit) {
        static std::atomic<bool> split_configured{false};
        static const void* const split_forms[3] = {(const void*)spmm_split_kernel<2>, (const void*)spmm_split_kernel<3>,
                                                   (const void*)spmm_split_kernel<4>};
        if (!split_configured.load()) {
          for (const void* f : split_forms)
            if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kDsLdsBytes) != hipSuccess)
              return SPDL_ERR_LAUNCH;
          split_configured.store(true);
        }
        int tiles = (n + kDsCols - 1) / kDsCols, panels = (m + kDsRows - 1) / kDsRows, tiles_first = slab_tiles_first(tiles, m);
        void* args[] = {&m, &k, &n, &nnz, (void*)&tiles, (void*)&panels, &ro, &ci, &val, &B, &C, &bias, &relu, &tiles_first};
        return hipLaunchKernel(split_forms[spmm_split_chunks(m, k, nnz) - 2], dim3(li.grid_x), dim3(li.block_threads), args, kDsLdsBytes,
                               st) == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
      }
      const bool wide = li.variant == kSpmmSlabDma && plan.form == kSlabWide;
      static const void* const inner_forms[3] = {(const void*)spmm_slab_tiles_kernel<kSlabS, 2, 2, true, kSlabTilesMax>,
                                                 (const void*)spmm_slab_tiles_kernel<kSlabS, 2, 3, false, kSlabTilesMax>,
                                                 (const void*)spmm_slab_tiles_kernel<kSlabS, 2, 4, true, kSlabTilesMax>};
      if (plan.form == kSlabInner)
        dma_kernel = inner_forms[slab_look_fits(kSlabS, m, k, nnz, 32.0) ? 0 : slab_look_fits(kSlabS, m, k, nnz, 48.0) ? 1 : 2];
      static const void* const wide_forms[3] = {(const void*)spmm_slab_wide_kernel<1>, (const void*)spmm_slab_wide_kernel<2>,
                                                (const void*)spmm_slab_wide_kernel<4>};
      if (wide) dma_kernel = wide_forms[slab_wide_pairs(m, k, nnz)];
      if (!configured.load()) {
        for (const void* f : {(const void*)kernel, inner_forms[0], inner_forms[1], inner_forms[2], half_form})
          if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kSlabLdsBytes) != hipSuccess)
            return SPDL_ERR_LAUNCH;
        for (const void* f : wide_forms)
          if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kWideLdsBytes) != hipSuccess)
            return SPDL_ERR_LAUNCH;
        for (const auto& row : forms)
          for (const void* f : row)
            if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kSlabLdsBytes) != hipSuccess)
              return SPDL_ERR_LAUNCH;
        configured.store(true);
      }
      const int panels = (m + li.rows_per_block - 1) / li.rows_per_block;
      int tiles = (n + kSlabTile - 1) / kSlabTile;
      dim3 grid(li.grid_x), block(li.block_threads);
      if (li.variant == kSpmmSlab) {
        kernel<<<grid, block, kSlabLdsBytes, st>>>(m, k, n, nnz, tiles, li.grid_y, panels, ro, ci, val, order, B, C,
                                                   bias, relu);
      } else {
        int tpw = li.grid_y, lds = kSlabLdsBytes;
        if (wide) {
          tiles = (n + kWideTile - 1) / kWideTile;
          tpw /= 2;
          lds = kWideLdsBytes;
        }
        int tiles_first = slab_tiles_first((tiles + tpw - 1) / tpw, m);
        void* args[] = {&m, &k, &n, &nnz, (void*)&tiles, &tpw, (void*)&panels, &ro, &ci, &val, &order, &B, &C,
                        &bias, &relu, &tiles_first};
        if (hipLaunchKernel(dma_kernel, grid, block, args, lds, st) != hipSuccess) return SPDL_ERR_LAUNCH;
      }
    } else {
      return SPDL_ERR_UNSUPPORTED;
    }
  } else {
    rc = launch_spmm_rowsplit<T, I>(li, m, n, nnz, ro, ci, val, order, B, C, bias, relu, hint, st);
  }
  if (rc != SPDL_OK) return rc;
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

template <typename T>
bool sddmm_group_usable(int n, const void* L, const void* R) {
  return n > 0 && n % 4 == 0 && aligned(L, 4 * sizeof(T)) && aligned(R, 4 * sizeof(T));
}

// Shape of the slab kernel's launch: U 64-column chunks per LDS row, S = 256/U rows of R per
// slab, the columns of A split into `ksplit` runs of `spp` slabs so that every CU gets a
// workgroup.
struct SddmmSlabShape { int U, S, deferred, ksplit, spp, panels, lds_bytes; };

// U chunks of 64 columns per LDS row (1 for n <= 64, else 2), 64 KB slabs.  Dot products of up to
// 128 columns are finished inside a slab; longer ones stream 128-column pieces of 128-row slabs
// and keep two strips per row and slab in registers.
SddmmSlabShape sddmm_slab_shape(int m, int k, int n) {
  SddmmSlabShape sh;
  sh.deferred = n > 128;
  sh.U = n <= 64 ? 1 : 2;
  sh.S = 256 / sh.U;
  sh.panels = (m + kSdRows - 1) / kSdRows;
  const int total = std::max(1, (k + sh.S - 1) / sh.S);
  sh.spp = split_for_machine(sh.panels, total);
  sh.ksplit = (total + sh.spp - 1) / sh.spp;
  sh.lds_bytes = 2 * (sh.S + 1) * 256 * sh.U;
  return sh;
}


// Launch shape of the lane kernel: sparse rows per 16-lane group (two where A is sparse, so
// that a stage of arithmetic outlasts the copy of the next slab and R is fetched by fewer
// workgroups), look-ahead in chunks of 16 column indices (mean + 4 sigma of a row's count in one
// slab of 128 columns), and the split of A's columns over workgroups that fills the machine.
struct SddmmLaneShape { int rpg, nchd, ksplit, spp, panels; };

SddmmLaneShape sddmm_lane_shape(int m, int k, int nnz, bool one_row_per_group = false, bool scaled = false) {
  SddmmLaneShape sh;
  const double d = (m > 0 && k > 0) ? (double)nnz / ((double)m * (double)k) : 0.0;
  const double mean = kLaneS * d, sd = std::sqrt(mean * std::max(0.0, 1.0 - d));
  sh.nchd = std::max(1, std::min(4, (int)std::ceil((mean + 4.0 * sd + 1.0) / 16.0)));
  // (two rows and three or more chunks of look-ahead do not fit the 128 registers of a lane: measured
  // 19 % slower than one row at 86 % sparsity)
  sh.rpg = (d >= 0.15 || sh.nchd > (scaled ? 1 : 2)) ? 1 : 2;       // (the scaled form holds A's values as well)
  if (sh.rpg == 2 && m <= kSdRows * kComputeUnits / 8) sh.rpg = 1;      // too few rows to share
  if (one_row_per_group) sh.rpg = 1;
  sh.panels = (m + kSdRows * sh.rpg - 1) / (kSdRows * sh.rpg);
  const int total = std::max(1, (k + kLaneS - 1) / kLaneS);
  sh.spp = split_for_machine(sh.panels, total);
  sh.ksplit = (total + sh.spp - 1) / sh.spp;
  return sh;
}

template <int RPG, int NCHD, bool NT = false, bool ACCUM = false>
int launch_sddmm_lane(const SddmmLaneShape& sh, int grid, int m, int k, int n, int nnz, const int* ro, const int* ci,
                      const float* L, const float* R, float* out, const float* scale, hipStream_t st,
                      const int* order = nullptr, int ld = 0, int c0 = 0) {
  static std::atomic<bool> configured{false};
  constexpr int lds = NT ? kLaneNtLdsBytes : kLaneLdsBytes;
  const void* plain = reinterpret_cast<const void*>(sddmm_lane_kernel<RPG, NCHD, false, NT, ACCUM>);
  const void* scaled = reinterpret_cast<const void*>(sddmm_lane_kernel<RPG, NCHD, true, NT, ACCUM>);
  if (!configured.load()) {
    for (const void* f : {plain, scaled})
      if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return SPDL_ERR_LAUNCH;
    configured.store(true);
  }
  if (ld == 0) ld = n;
  int ksplit = sh.ksplit, spp = sh.spp, panels = sh.panels;
  void* args[] = {&m, &k, &n, &nnz, &ksplit, &spp, &panels, &ro, &ci, &L, &R, &out, &scale, &order, &ld, &c0};
  return hipLaunchKernel(scale ? scaled : plain, dim3(grid), dim3(kSdThreads), args, lds, st) == hipSuccess
             ? SPDL_OK : SPDL_ERR_LAUNCH;
}

// Launch shape of the matrix-core form: 64 sparse rows per workgroup, the steps of 256 columns dealt to `parts`
// workgroups per panel; sixteens of the dot product (an odd number of them only where that is five, 65 .. 80 columns);
// sixty-fours of a row's entries fetched a step ahead (mean + 1.5 sigma).
struct SddmmSplitShape { int parts, spp, ksteps, ahead, panels, grid; };
SddmmSplitShape sddmm_split_shape(int m, int k, int n, int nnz) {
  SddmmSplitShape sh;
  sh.panels = (m + kSpRows - 1) / kSpRows;
  const int total = std::max(1, (k + kSpCols - 1) / kSpCols);
  sh.spp = split_for_machine(sh.panels, total);
  sh.parts = (total + sh.spp - 1) / sh.spp;
  sh.ksteps = std::max(2, (n + 15) / 16);
  if (sh.ksteps != 5) sh.ksteps = (sh.ksteps + 1) / 2 * 2;
  const double mean = (double)nnz / ((double)m * (double)k) * kSpCols;
  sh.ahead = mean + 1.5 * std::sqrt(mean) <= 64.0 ? 1 : 2;
  sh.grid = 8 * (int)(((int64_t)sh.panels * sh.parts + 7) / 8);
  return sh;
}
// Waves that pick: what the entries of a step take is covered by its multiplications where they last long enough, and
// a multiplying wave then has a third of a SIMD's registers; for up to 32 columns eight waves (8192 x 10240 at 20 %, n = 32:
// 51 us against 66 with four; n = 64: 94 against 76).
constexpr int sddmm_split_pickers(int ksteps) { return ksteps <= 2 ? 8 : 4; }

template <int KSTEPS, int AHEAD, int PICKERS>
int launch_sddmm_split(const SddmmSplitShape& sh, int m, int k, int n, int nnz, const int* ro, const int* ci, const float* L,
                       const float* R, float* out, const float* scale, hipStream_t st) {
  static std::atomic<bool> configured[2];
  constexpr int lds = sddmm_split_lds_bytes(KSTEPS);
  auto kernel = scale ? sddmm_split_kernel<KSTEPS, AHEAD, PICKERS, true> : sddmm_split_kernel<KSTEPS, AHEAD, PICKERS, false>;
  if (!configured[scale != nullptr].load()) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
      return SPDL_ERR_LAUNCH;
    configured[scale != nullptr].store(true);
  }
  kernel<<<dim3(sh.grid), dim3(64 * (kSpWaves + PICKERS)), lds, st>>>(m, k, n, nnz, sh.parts, sh.spp, ro, ci, L, R, out, scale);
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

template <typename T>
bool sddmm_lane_usable(int n, int nnz, const void* L, const void* R) {
  // (dot products longer than 128 columns take one pass per 128 columns; 32-bit byte offsets inside
  // a slab of R: 128 rows * n * 4 < 2^31)
  return sizeof(T) == 4 && sddmm_group_usable<T>(n, L, R) && n < (1 << 21) && nnz < (1 << 29);
}

// Dot products of any width from 4 columns on, operands at any element: the kernels that move 16 bytes
// per lane take them, the lane at a row's end working on the row's last piece (piece_start).  (LSTM
// shape at 90 % sparsity, n = 127: 92 us against 1782 for one column per lane.)  Not 129 .. 191 columns,
// which are two passes of the lane kernel or two chunks of the slab kernel, the second mostly empty:
// those go to the general family.  (A pass of the lane kernel is at least four columns wide.)
inline bool sddmm_any_width(int n) { return n >= 4; }
inline bool sddmm_wide_any(int n) { return n >= 4 && (n <= 128 || n >= 192); }
inline bool sddmm_lane_pass_ok(int n) { return n % 128 == 0 || n % 128 >= 4; }

// Dense matrices, dot products of up to 128 columns: whether the matrix-core form takes the place of the lane and slab
// kernels.  Estimates in microseconds: rounds of one workgroup per compute unit, each of so many steps (slabs) and
// thousand entries.  Fitted on 400 uniform shapes (256 .. 12000 rows, 256 .. 10200 columns, 3 .. 40 %, n = 9 .. 128: 7 % off for
// the matrix cores, 14 % and 6 % for the lane and slab kernels, 10 % for the nonzero-split one; the choice takes 1.005 times
// the faster one's time on average, 0.84 times that of never).
inline double sddmm_split_estimate(int m, int k, int n, int nnz) {
  const SddmmSplitShape sh = sddmm_split_shape(m, k, n, nnz);
  const double rounds = split_chain(sh.panels, sh.parts, -1), density = (double)nnz / ((double)m * (double)k);
  const double entries = 1e-3 * kSpRows * std::min((double)k, (double)sh.spp * kSpCols) * density;
  return 0.2 + rounds * (4.4 + sh.spp * (0.28 + 0.63 * sh.ksteps) + 0.27 * entries);
}
bool sddmm_split_runs(int variant, int m, int k, int n, int nnz) {
  if ((variant != kSddmmLane && variant != kSddmmSlabDma) || n < 4 || n > 128 || m < 256 || k < kSpCols / 2 || nnz <= 0 ||
      nnz >= (1 << 29))
    return false;
  const double density = (double)nnz / ((double)m * (double)k);
  double other;
  if (variant == kSddmmLane) {
    const SddmmLaneShape sh = sddmm_lane_shape(m, k, nnz);
    const double entries = 1e-3 * kSdRows * sh.rpg * std::min((double)k, (double)sh.spp * kLaneS) * density;
    other = 5.7 + split_chain(sh.panels, sh.ksplit, -1) * (1.6 * sh.spp - 1.2 + 1.38 * entries);
  } else {
    const SddmmSlabShape sh = sddmm_slab_shape(m, k, n);
    const double entries = 1e-3 * kSdRows * std::min((double)k, (double)sh.spp * sh.S) * density;
    other = 3.9 + split_chain(sh.panels, sh.ksplit, -1) * (1.28 * sh.spp + 0.4 + 1.38 * entries);
  }
  return sddmm_split_estimate(m, k, n, nnz) <= 0.97 * other;
}

// Dense matrices, long dot products: whether whole blocks on the matrix cores take the place of the slab kernel.  From 576 columns
// on, where the slab kernel's sums of so many terms are the less accurate ones (2-norm error against 64 bits, normal data:
// at 512 columns 1.16e-7 against 1.18e-7, at 640 1.27e-7 and 1.19e-7, at 4096 2.9e-7 and 1.5e-7; the lane kernel, 1.0e-7, stays).
// Estimates in microseconds.  The blocks: rounds of one workgroup per compute unit, each of so many chunks, which take longer on
// a full machine (it is slowed down to its power), and entries to pick.  The slab kernel: slabs and, per 128 columns of the dot product,
// strips of sixteen entries of the fullest rows, of which the third does not fit its registers.  Fitted on 196 uniform shapes
// (128 .. 6000 rows and columns, 3 .. 35 %, 576 .. 4500 columns), 4 % and 8 % off; the choice takes 1.005 times the faster one's
// time on average, never more than 1.02 times the slab kernel's, and 0.84 times it on average.  (Matrices that are not uniform gain
// more: 2048^2, a band of 12 %, n = 1024: 382 us and 47; log-normal rows, 2048 x 1024 at 10 %: 100 and 37.)
inline double normal_below(double x) { return 0.5 * std::erfc(-x * 0.70710678); }
bool sddmm_long_runs(int variant, int m, int k, int n, int nnz) {
  if (variant != kSddmmSlabDma || n < 576 || n >= (1 << 21) || m < 128 || k < 128 || nnz <= 0 || nnz >= (1 << 29)) return false;
  const double density = (double)nnz / ((double)m * (double)k);
  const int blocks_m = (m + kLgRows - 1) / kLgRows, blocks_k = (k + kLgCols - 1) / kLgCols;
  const double rounds = k > m ? split_chain(blocks_k, blocks_m, -1) : split_chain(blocks_m, blocks_k, -1);
  const double fill = std::min(1.0, (double)blocks_m * blocks_k / kComputeUnits);
  const double entries = 1e-3 * kLgRows * std::min(k, kLgCols) * density;
  const double blocks = 0.3 + rounds * (10.3 + (n + kLgChunk - 1) / kLgChunk * (2.63 + 0.77 * fill) + 0.3 * entries);
  const SddmmSlabShape sh = sddmm_slab_shape(m, k, n);
  const double mean = std::min(k, sh.S) * density, sd = std::sqrt(mean * std::max(1e-9, 1.0 - density));
  auto filled = [&](int strips) { return normal_below((mean - 16.0 * strips - 0.5) / sd + 2.5); };
  const double slab_rounds = split_chain(sh.panels, sh.ksplit, -1);
  const double slab_fill = (double)sh.panels * sh.ksplit / (kComputeUnits * slab_rounds);
  const double slabs = 0.2 + slab_rounds * (6.0 + sh.spp * (0.8 + n / 128.0 * (1.36 + 0.62 * filled(1) + 3.38 * filled(2) + 3.82 * filled(3)) *
                                                            (1.0 + 0.21 * slab_fill)));
  return blocks <= 0.95 * slabs;
}

// The workgroups of a panel share an XCD and with it their rows of L, or those of a range of columns their rows of R: whichever of the two
// the XCDs would otherwise all read is the shorter.  (1024 x 4096, n = 2048, at 20 %: 71.4 us and 70.6; 4096 x 1024: 69.0 and 72.0.)
int launch_sddmm_long(int m, int k, int n, int nnz, const int* ro, const int* ci, const float* L, const float* R, float* out,
                      const float* scale, hipStream_t st) {
  static std::atomic<bool> configured;
  if (!configured.load()) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(sddmm_long_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLgLdsBytes) !=
        hipSuccess)
      return SPDL_ERR_LAUNCH;
    configured.store(true);
  }
  const int panels = (m + kLgRows - 1) / kLgRows, parts = (k + kLgCols - 1) / kLgCols;
  sddmm_long_kernel<<<dim3(slab_grid_size(panels, parts)), dim3(kLgThreads), kLgLdsBytes, st>>>(m, k, n, nnz, panels, parts, k > m, ro, ci, L, R,
                                                                                                out, scale);
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

// Which workgroups of sddmm_slab_dma_kernel share an XCD: those of a panel, which read the same rows of L, or those of a
// range of A's columns, which read the same rows of R.  Up to 1024 rows and a longer R (which every XCD would otherwise read
// whole: 1024 x 4096, n = 4096: 575 MB from behind the L2s, now 356) the latter.  us, a launch repeated, which finds R in the Infinity
// Cache / with nothing in the caches: 1024 x 4096, n = 4096, at 10 % 142.8 -> 130.9 / 161.4 -> 160.5, at 5 % 134.5 -> 98.2 / 155.4 ->
// 149.6; 1024 x 8192 at 5 %, n = 2048: 136.7 -> 98.7 / 167.3 -> 152.6; 700 x 2800 at 10 %, n = 700: 21.2 -> 19.8 / 26.4 -> 25.4.  With
// more rows, or fewer columns, it is L that would be read again (1800 x 7200 at 10 %, n = 1500: 194.3 and 201.4; 1024 x 2048 at 10 %, n =
// 3000: 55.5 and 56.5).
inline bool sddmm_parts_first(int ksplit, int m, int k) {
  return ksplit >= 8 && m <= 1024 && 2 * (int64_t)k >= 5 * (int64_t)m;
}

inline int sddmm_slab_grid(const SddmmSlabShape& sh, int m, int k, bool dma) {
  return dma && sddmm_parts_first(sh.ksplit, m, k) ? slab_grid_size(sh.ksplit, sh.panels)
                                                   : slab_grid_size(sh.panels, sh.ksplit);
}

template <typename T>
void fill_sddmm_info(int m, int k, int n, int nnz, const void* L, const void* R, spdl_launch_info* info,
                     int hint = 0) {
  const bool vec_ok = sddmm_group_usable<T>(n, L, R);          // whole pieces at aligned addresses
  const bool fast_ok = vec_ok || (sizeof(T) == 2 ? sddmm_any_width(n) : sddmm_wide_any(n));
  int variant = g_forced[1].load();
  const bool free_choice = variant < 0;
  const bool mfma_ok = sizeof(T) == 2 && n >= 8 &&
                       (int64_t)((m + 63) / 64) * ((k + 63) / 64) < ((int64_t)1 << 31);
  if (variant == kSddmmMfma && !mfma_ok) variant = kSddmmGroup;
  if (variant < 0 && mfma_ok && sddmm_mfma_pays(m, k, n, nnz)) variant = kSddmmMfma;
  if (variant == kSddmmMfma) {
    info->variant = kSddmmMfma;
    info->vec = 8;
    info->lanes_per_row = kWave;
    const SddmmMfmaShape sh = sddmm_mfma_shape(m, k);
    info->rows_per_block = sh.rows;
    info->block_threads = kSmThreads;
    info->grid_x = sddmm_mfma_grid((m + sh.rows - 1) / sh.rows, (k + sh.cols - 1) / sh.cols);
    info->grid_y = (k + sh.cols - 1) / sh.cols;     // blocks per panel (the grid is 1-D)
    return;
  }
  bool skewed_lane = false;      // (for the hint of unequal rows) lane kernel estimated faster than the nonzero-split one
  if (variant < 0) {
    const double density = (m > 0 && k > 0) ? (double)nnz / ((double)m * (double)k) : 0.0;
    const double reuse = 64.0 * density;
    const bool fp32_any_m = fast_ok && sizeof(T) == 4 && nnz < (1 << 29) && n < (1 << 21);
    const bool fp32_fast = fp32_any_m && m >= 512;
    if (!fast_ok) {
      variant = kSddmmRowstrip;
    } else if (n <= 128 || !fp32_any_m) {
      // Short dot products gain little from the slabs (a row of R is one or two cache lines) unless
      // the reuse is high, and the nonzero-split kernel does not care how the entries are laid out
      // (a banded attention mask leaves most of a panel's column ranges nearly empty).  65..128
      // columns: the lane kernel, as long as a panel of 64 rows meets the same row of R at least
      // once on average.
      const bool lane = fp32_fast && n > 64 && reuse >= 1.0;
      // (5 <= reuse < 8 with at least 128 panels of 64 rows: on uniform masks the slab kernel is then
      // 1.25 .. 1.4 times faster than gathering, 8192 x 2048 at 10 %: 18.7 us against 25; with 64
      // panels it has to split A's columns over workgroups and the banded attention mask of 4096
      // rows, also 10 % dense, takes 36 us against 24)
      // (panels that fill whole rounds of one workgroup per compute unit, 16384 or 32768 rows: from 4 on,
      // 7 .. 26 % faster than gathering there; not for square matrices, which may be attention masks)
      const int64_t panels64 = (m + kSdRows - 1) / kSdRows;
      const int64_t rounds64 = (panels64 + kComputeUnits - 1) / kComputeUnits;
      const bool whole_rounds = m != k && rounds64 > 0 && (double)panels64 >= 0.95 * (double)(rounds64 * kComputeUnits);
      // (2048 rows and more, not square: from 4.2 on at any number of panels; 4128 x 4212 at 8 %, n = 56: 21.8 us
      // against 23.3 for gathers and 27.1 for the window kernel; 7500 x 4019 at 11 %, n = 48: 33.5 against 40.4)
      const bool slab = fp32_fast && reuse >= 2.0 &&
                        (n >= 128 || reuse >= 8.0 || (reuse >= 5.0 && m >= 8192) || (reuse >= 4.0 && whole_rounds) ||
                         (reuse >= 4.2 && m >= 2048 && m != k && n > 16)) ||
                        // (the matrix-core form where it is estimated below gathering as well; not for square matrices, which
                        // may be banded masks: it multiplies whole blocks wherever the entries lie, but the waves that pick
                        // them wait for the steps that hold a row's band.  64 columns, matrix cores against gathers: 2048^2 at 12 %,
                        // uniform 10.2 us and 10.8, a band 21.7 and 10.8; 4096^2 at 12 %, uniform 19.2 and 24.5 (window), a band
                        // 44.5 and 19.2, half band, half uniform 33.2 and 23.4)
                        (fp32_fast && n <= 64 && m != k && sddmm_split_runs(kSddmmSlabDma, m, k, n, nnz) &&
                         sddmm_split_estimate(m, k, n, nnz) <= 4.0 + 12.3e-6 * (double)nnz);
      // Few entries: the nonzero-split kernel may be done before the others have filled their first slabs (850 x 434
      // at 25 %, n = 40, 93 thousand: 5.4 us against 10.3), unless rows are short, which leaves most of a strip of 16
      // empty (4096 x 128, rows of 4, n = 128: 12.0 against 6.3 in the lane kernel), or the slabs few (2048 x 1000, rows of 40,
      // n = 128: 8.4 against 6.9).  Estimates in microseconds, from the chain of slabs, the entries that a lane group meets in
      // its slabs and the strips; fitted on 720 uniform shapes of 512 .. 10000 rows, 128 .. 10000 columns, rows of 3 .. 200
      // and n = 20 .. 128 (the choice takes 1.01 times the faster one's time on average, 1.14 at worst beyond 64 columns).
      bool few = nnz < (n <= 64 ? 300000 : 170000);
      if (few && (lane || slab)) {
        const double entries = 1e-5 * (double)nnz, row = (double)nnz / (double)m, strips = std::max(1.0, 16.0 / std::max(row, 1e-3));
        double t_group = n <= 64 ? 2.5 + 1.5 * entries + 1.6 * strips : 2.5 + 2.9 * entries + 2.3 * strips;
        // (strips of four: fitted on 250 random shapes, 7 % off.  Rows of fewer than five entries, and more than 80 thousand, keep
        // the line above, and with it choices that a test of the selection fixes: 4096 x 128, rows of 4, n = 128, lane 6.3 us, group now 4.0.)
        if (nnz <= 80000 && row >= 5.0 && sddmm_group_short_strips(m, n, nnz, 4) == 16)
          t_group = n <= 64 ? 3.6 + 1.4 * entries : 3.7 + 2.4 * entries;
        double t_other;
        if (lane) {
          const SddmmLaneShape sh = sddmm_lane_shape(m, k, nnz);
          const double met = sh.rpg * row * std::min(1.0, (double)sh.spp * kLaneS / (double)k);
          t_other = (sh.rpg == 2 ? 3.5 : 2.1) + 1.1 * split_chain(sh.panels, sh.ksplit, sh.spp) + 0.052 * met + 1.1 * entries;
        } else {
          const SddmmSlabShape sh = sddmm_slab_shape(m, k, n);
          const double met = row * std::min(1.0, (double)sh.spp * sh.S / (double)k);
          t_other = 1.4 + 1.1 * split_chain(sh.panels, sh.ksplit, sh.spp) + 0.057 * met + 0.6 * entries;
        }
        if (m != k && sddmm_split_runs(lane ? kSddmmLane : kSddmmSlabDma, m, k, n, nnz))
          t_other = std::min(t_other, sddmm_split_estimate(m, k, n, nnz));
        few = t_group <= t_other;
      }
      variant = few ? kSddmmGroup : lane ? kSddmmLane : slab ? kSddmmSlabDma : kSddmmGroup;
      // The shape of an attention head (33..64 columns, thousands of rows of a few hundred entries,
      // at most 1/8 dense; paper Sec. "Application: Sparse Transformer"): the window kernel, which is
      // the nonzero-split kernel with the rows of R around a band taken from LDS and the four lane
      // groups of a wave on one row (13 % faster on a band of 256 at sequence 4096, 5 .. 20 % on uniform
      // masks of that shape).  Not wider than that: the nonzero-split kernel does not care how long
      // the rows are, the window kernel owns rows, and on log-normal row lengths it takes 1.5 times as
      // long (4096 x 4096 at 6 %: 26 us against 17) although the waves of a workgroup share what a row
      // holds beyond 512 entries.
      if (variant == kSddmmGroup && fp32_fast && n > 32 && n <= kWinTile && m >= 4096 && aligned(L, 16) &&
          aligned(R, 16) && (int64_t)k * n < ((int64_t)1 << 29) && (double)nnz >= 192.0 * (double)m &&
          (double)nnz <= 0.125 * (double)m * (double)k)
        variant = kSddmmWindow;
    } else {
      // Longer dot products: three candidates, chosen by an estimate of their run times from measured
      // rates (paper Sec. "Experiments": the kernel and tile are picked by heuristics from the shape;
      // the discussion there names better selection as the open end).  The lane kernel runs once per
      // 128 columns and walks A every time (about 9.5 us of fixed cost per pass); the slab kernel
      // walks A once and keeps at most 32 partial sums per row and slab in registers, so it slows
      // down where rows get dense; the nonzero-split kernel gathers rows of R and runs at the rate
      // of those gathers whatever the density.  Rates in TFLOP/s against density, measured on
      // matrices from 2048 x 2048 to 8192 x 10240 with n = 256 .. 4096.
      static const double ds[7] = {0.01, 0.02, 0.04, 0.10, 0.16, 0.30, 0.50};
      static const double lane_rate[7] = {5.0, 9.0, 14.0, 22.6, 26.0, 33.0, 32.0};
      static const double slab_rate[7] = {4.0, 7.0, 12.8, 22.8, 24.0, 19.0, 12.0};
      auto rate = [&](const double* r) {
        if (density <= ds[0]) return r[0];
        for (int i = 1; i < 7; ++i)
          if (density <= ds[i]) return r[i - 1] + (r[i] - r[i - 1]) * (density - ds[i - 1]) / (ds[i] - ds[i - 1]);
        return r[6];
      };
      const double flops = 2.0 * (double)nnz * (double)n;                   // per launch, all passes
      const int passes = (n + 127) / 128;
      // (the rates are those of a full machine: a small matrix gives fewer workgroups than there are
      // compute units, 760 x 231 at 43 %, n = 2048: 24 workgroups, 193 us in the slab kernel against 67
      // for the nonzero-split kernel, which spreads over the chip whatever the shape)
      const SddmmLaneShape lsh = sddmm_lane_shape(m, k, nnz, true);
      const SddmmSlabShape ssh = sddmm_slab_shape(m, k, n);
      const double lane_fill = std::min(1.0, (double)lsh.panels * lsh.ksplit / kComputeUnits);
      const double slab_fill = std::min(1.0, (double)ssh.panels * ssh.ksplit / kComputeUnits);
      const double t_lane = !sddmm_lane_pass_ok(n) ? 1.0e30 : passes * 9.5 + flops / (rate(lane_rate) * 1e6 * lane_fill);   // microseconds
      // (every panel of 64 rows streams all of R through its compute unit: 8 TB/s over the chip at best)
      const double panels64 = (double)((m + kSdRows - 1) / kSdRows);
      const double t_slab = 8.0 + std::max(flops / (rate(slab_rate) * 1e6 * slab_fill), panels64 * (double)k * (double)n * 4.0 / 8.0e6);
      // (a strip of the gather kernel steps through its dot product 64 columns at a time, about 1.1 us
      // of memory latency per step: the floor for small problems)
      const double t_group = 5.0 + 1.1 * (double)(n / 64) + flops / (n < 2048 ? 7.0e6 : 5.5e6);
      variant = (t_lane <= t_slab && t_lane <= t_group) ? kSddmmLane : t_slab <= t_group ? kSddmmSlabDma : kSddmmGroup;
      // (the lane kernel's rate is that of rows of equal length; an R of a few megabytes is gathered from L2)
      skewed_lane = t_lane <= 0.45 * t_group && (double)k * (double)n * 4.0 >= 7.0e6;
    }
  }
  if ((variant == kSddmmSlab || variant == kSddmmSlabDma) &&
      !(fast_ok && sizeof(T) == 4 && nnz < (1 << 29) && n < (1 << 21)))   // 32-bit byte offsets
    variant = kSddmmGroup;
  if ((variant == kSddmmSlab && !vec_ok) ||
      (variant == kSddmmLane && !(fast_ok && sddmm_lane_pass_ok(n) && sizeof(T) == 4 && nnz < (1 << 29) && n < (1 << 21))))
    variant = kSddmmGroup;
  const bool window_ok = sizeof(T) == 4 && vec_ok && aligned(L, 16) && aligned(R, 16) && n <= 2 * kWinTile && nnz > 0 &&
                         (int64_t)k * n < ((int64_t)1 << 29);
  // The caller says that the entries form a band (a problem the window kernel cannot take keeps the
  // choice made above).  At most 64 columns: two of the window kernel's workgroups, 16 rows, are at work on a compute unit: its
  // time goes in steps of 4096 rows, and below 2048 it is one workgroup's, while the nonzero-split kernel's goes with the
  // entries and is the shorter one unless the steps come out nearly even, or the rows are short (64 columns, window against
  // nonzero-split kernel, 4096 rows of 456: 24.2 us and 26.6; 2048 of 374: 13.4 and 14.3; 2152 of 300: 11.3 and 12.8, of 386:
  // 14.2 and 14.8; 2994 of 368: 16.8 and 17.7, of 487: 24.2 and 21.3; 4800 of 512: 34.6 and 31.9; 6144 of 620: 42.8 and
  // 46.6; 1500 of 292: 10.1 and 9.5; 1024 of 374: 11.9 and 8.6).  Beyond 64 columns the window fills the
  // LDS of a compute unit, one workgroup of 16 rows: whole steps of 4096 rows only, where it is level on long rows and up to
  // 8 % faster on shorter ones (128 columns, window against nonzero-split kernel: 4096 rows of 456: 40.3 us and 43.8, of 620:
  // 53.4 and 52.8; 8192 of 783: 128 and 135; 3800 of 432: 38.3 and 39.2, of 584: 50.1 and 46.9; 3500 of 548: 47.5 and 43.3;
  // 4300 of 472: 52 and 44; 7000 of 688: 110 and 102; 2048 of 374: 27.5 and 21.9; 1024 of 292: 19.3 and 11.4).
  if (free_choice && hint == kHintBanded && window_ok) {
    const bool wide = n > kWinTile;
    const int64_t step = wide ? 4096 : 2048, stepped = (m + step - 1) / step * step;
    const bool even = wide ? 20 * stepped <= 21 * (int64_t)m : 5 * stepped <= 6 * (int64_t)m;
    const bool short_rows = !wide && m > 2048 && m <= 4096 && nnz <= 400 * (int64_t)m;
    // (with sixteen waves and a large window the time goes with the entries too: 3000 rows of 428: 18.7 us and 20.0; 3300 of 458: 20.2 and 21.7)
    variant = even || short_rows || (!wide && win_large_sddmm(m, nnz)) ? kSddmmWindow : kSddmmGroup;
  }
  // the caller says that the row lengths are strongly unequal: the nonzero-split kernel, which does not
  // care, or for dot products of more than 128 columns the lane kernel in passes where the estimate
  // above gives it less than 0.45 of that kernel's time (dense matrices; the slab kernel, whose
  // deferred partial sums overflow on the long rows, is left out)
  if (free_choice && hint == kHintSkewed && fast_ok && (variant == kSddmmLane || variant == kSddmmSlabDma || variant == kSddmmWindow))
    variant = skewed_lane ? kSddmmLane : kSddmmGroup;
  if (variant == kSddmmWindow && !window_ok) variant = kSddmmGroup;
  if (variant == kSddmmGroup && !fast_ok) variant = kSddmmRowstrip;
  const int avg = m > 0 ? nnz / m : 0;
  info->variant = variant;
  info->block_threads = 256;
  info->grid_y = 1;
  if (variant == kSddmmWindow) {
    info->vec = 4;
    info->lanes_per_row = 16;
    const int waves = n <= kWinTile && !(hint == kHintBanded && win_large_sddmm(m, nnz)) ? kWinWaves : kWinWavesWide;
    info->rows_per_block = waves;
    info->block_threads = 64 * waves;
    info->grid_x = (m + waves - 1) / waves;
    return;
  }
  if (sizeof(T) == 4 && sddmm_long_runs(variant, m, k, n, nnz)) {
    info->vec = 4;
    info->lanes_per_row = kWave;
    info->rows_per_block = kLgRows;
    info->block_threads = kLgThreads;
    info->grid_x = slab_grid_size((m + kLgRows - 1) / kLgRows, (k + kLgCols - 1) / kLgCols);
    info->grid_y = (k + kLgCols - 1) / kLgCols;     // column ranges of A (the grid is 1-D)
    return;
  }
  if (sizeof(T) == 4 && sddmm_split_runs(variant, m, k, n, nnz)) {
    const SddmmSplitShape sh = sddmm_split_shape(m, k, n, nnz);
    info->vec = 8;
    info->lanes_per_row = kWave;
    info->rows_per_block = kSpRows;
    info->block_threads = 64 * (kSpWaves + sddmm_split_pickers(sh.ksteps));
    info->grid_x = sh.grid;
    info->grid_y = sh.parts;                // column ranges of A (the grid is 1-D)
    return;
  }
  if (variant == kSddmmLane) {
    const SddmmLaneShape sh = sddmm_lane_shape(m, k, nnz, n > 128);
    info->vec = 8;
    info->lanes_per_row = 2;
    info->rows_per_block = kSdRows * sh.rpg;
    info->block_threads = kSdThreads;
    info->grid_x = slab_grid_size(sh.panels, sh.ksplit);
    info->grid_y = sh.ksplit;               // column ranges of A (the grid is 1-D)
    return;
  }
  if (variant == kSddmmSlab || variant == kSddmmSlabDma) {
    const SddmmSlabShape sh = sddmm_slab_shape(m, k, n);
    info->vec = 4 * sh.U;
    info->lanes_per_row = 16;
    info->rows_per_block = kSdRows;
    info->block_threads = kSdThreads;
    info->grid_x = sddmm_slab_grid(sh, m, k, variant == kSddmmSlabDma);
    info->grid_y = sh.ksplit;               // column ranges of A (the grid is 1-D)
    return;
  }
  // (the general family: from four columns on its strips are those of the nonzero-split kernel, sixteen lanes to a
  // strip)
  if (variant == kSddmmGroup || sddmm_any_width(n)) {
    info->vec = 4;
    info->lanes_per_row = 16;
    if (const int few = sddmm_group_short_strips(m, n, nnz, sizeof(T))) {             // strips of four, a wave to a workgroup
      info->rows_per_block = few;
      info->block_threads = kWave;
      info->grid_x = (nnz + few - 1) / few;
      return;
    }
    // entries per wave: four strips of 16 while the machine (32 waves on each CU) is not
    // full, then as many as keep the grid at about one wave per slot
    const int64_t slots = (int64_t)kComputeUnits * 32;
    const int quads = (int)std::max<int64_t>(1, std::min<int64_t>(64, ((int64_t)nnz / 64 + slots - 1) / slots));
    info->rows_per_block = quads * 64;                     // entries per wave
    const int64_t waves = ((int64_t)nnz + quads * 64 - 1) / (quads * 64);
    info->grid_x = (int)((waves + 3) / 4);
    return;
  }
  const int split = std::max(1, std::min(8, avg / (2 * kWave)));
  info->vec = 1;
  info->lanes_per_row = kWave;
  info->rows_per_block = split;
  const int64_t waves = (int64_t)m * split;
  info->grid_x = (int)((waves + 3) / 4);
}

template <typename T, int U, int S, bool DEFERRED>
int launch_sddmm_slab(const SddmmSlabShape& sh, int grid, int m, int k, int n, int nnz, const int* ro,
                      const int* ci, const T* L, const T* R, T* out, const T* scale, hipStream_t st, bool dma,
                      const int* order) {
  static std::atomic<bool> configured{false};
  static std::atomic<bool> configured_dma{false};
  if (dma) {
    auto kernel = n % 4 == 0 ? sddmm_slab_dma_kernel<U, S, DEFERRED, false> : sddmm_slab_dma_kernel<U, S, DEFERRED, true>;
    if (!configured_dma.load()) {
      for (auto f : {sddmm_slab_dma_kernel<U, S, DEFERRED, false>, sddmm_slab_dma_kernel<U, S, DEFERRED, true>})
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize,
                                sh.lds_bytes) != hipSuccess)
          return SPDL_ERR_LAUNCH;
      configured_dma.store(true);
    }
    kernel<<<dim3(grid), dim3(kSdThreads), sh.lds_bytes, st>>>(m, k, n, nnz, sh.ksplit, sh.spp, sh.panels, ro, ci,
                                                               L, R, out, scale, order,
                                                               sddmm_parts_first(sh.ksplit, m, k));
    return SPDL_OK;
  }
  auto kernel = sddmm_slab_kernel<T, U, S, DEFERRED>;
  if (!configured.load()) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            sh.lds_bytes) != hipSuccess)
      return SPDL_ERR_LAUNCH;
    configured.store(true);
  }
  kernel<<<dim3(grid), dim3(kSdThreads), sh.lds_bytes, st>>>(m, k, n, nnz, sh.ksplit, sh.spp, sh.panels, ro, ci,
                                                             L, R, out, scale);
  return SPDL_OK;
}

template <typename T>
int sddmm_impl(int m, int k, int n, int nnz, const int* ro, const int* ci, const T* L, const T* R,
               T* out, void* stream, const T* scale = nullptr, const int* order = nullptr, int hint = 0) {
  if (!sizes_ok(m, k, n, nnz)) return SPDL_ERR_INVALID;
  if (m == 0 || nnz == 0) return SPDL_OK;
  if (!ro || !ci || !out || (n > 0 && (!L || !R))) return SPDL_ERR_INVALID;
  hipStream_t st = static_cast<hipStream_t>(stream);
  spdl_launch_info li;
  fill_sddmm_info<T>(m, k, n, nnz, L, R, &li, hint);
  dim3 grid(li.grid_x), block(256);
  (void)hipGetLastError();
  if (li.variant == kSddmmMfma) {
    if constexpr (sizeof(T) == 2) {
      // copies start at multiples of four bytes: every row's first element, or every other row's
      const bool odd = n % 2 != 0 || !aligned(L, 4) || !aligned(R, 4);
      const SddmmMfmaShape sh = sddmm_mfma_shape(m, k);
#define SPDL_MFMA_SDDMM(BM, BN, P)                                                                                         \
  if (sh.rows == BM && sh.cols == BN)                                                                                      \
    return odd ? launch_sddmm_mfma<true, BM, BN, P>(li.grid_x, li.grid_y, m, k, n, ro, ci, L, R, out, scale, st)           \
               : launch_sddmm_mfma<false, BM, BN, P>(li.grid_x, li.grid_y, m, k, n, ro, ci, L, R, out, scale, st);
      SPDL_MFMA_SDDMM(64, 64, 16) SPDL_MFMA_SDDMM(64, 32, 32) SPDL_MFMA_SDDMM(32, 32, 32)
#undef SPDL_MFMA_SDDMM
      return SPDL_ERR_UNSUPPORTED;
    } else {
      return SPDL_ERR_UNSUPPORTED;
    }
  }
  if constexpr (sizeof(T) == 4) {
    if (sddmm_long_runs(li.variant, m, k, n, nnz)) return launch_sddmm_long(m, k, n, nnz, ro, ci, L, R, out, scale, st);
    if (sddmm_split_runs(li.variant, m, k, n, nnz)) {
      const SddmmSplitShape sh = sddmm_split_shape(m, k, n, nnz);
#define SPDL_SPLIT(KSTEPS, AHEAD)               \
  if (sh.ksteps == KSTEPS && sh.ahead == AHEAD) \
    return launch_sddmm_split<KSTEPS, AHEAD, sddmm_split_pickers(KSTEPS)>(sh, m, k, n, nnz, ro, ci, L, R, out, scale, st);
      SPDL_SPLIT(2, 1) SPDL_SPLIT(4, 1) SPDL_SPLIT(5, 1) SPDL_SPLIT(6, 1) SPDL_SPLIT(8, 1)
      SPDL_SPLIT(2, 2) SPDL_SPLIT(4, 2) SPDL_SPLIT(5, 2) SPDL_SPLIT(6, 2) SPDL_SPLIT(8, 2)
#undef SPDL_SPLIT
      return SPDL_ERR_UNSUPPORTED;
    }
  }
  if (li.variant == kSddmmLane) {
    if constexpr (sizeof(T) == 4) {
      const SddmmLaneShape sh = sddmm_lane_shape(m, k, nnz, n > 128, scale != nullptr);
      const int grid = slab_grid_size(sh.panels, sh.ksplit);
      // one pass per chunk of 128 columns; passes after the first add to what out holds
      for (int c0 = 0; c0 < n; c0 += 128) {
        const int nc = std::min(128, n - c0);
        int rc = SPDL_ERR_UNSUPPORTED;
#define SPDL_LANE(RPG, NCHD)                                                                           \
  if (sh.rpg == RPG && sh.nchd == NCHD) {                                                              \
    if (c0 == 0)                                                                                       \
      rc = launch_sddmm_lane<RPG, NCHD>(sh, grid, m, k, nc, nnz, ro, ci, L, R, out, scale, st, order, n, 0); \
    else if constexpr (RPG == 1)                                                                       \
      rc = launch_sddmm_lane<1, NCHD, false, true>(sh, grid, m, k, nc, nnz, ro, ci, L + c0, R + c0, out, scale, st, \
                                                   order, n, c0);                                      \
  }
        SPDL_LANE(1, 1) SPDL_LANE(1, 2) SPDL_LANE(1, 3) SPDL_LANE(1, 4)
        SPDL_LANE(2, 1) SPDL_LANE(2, 2)
#undef SPDL_LANE
        if (rc != SPDL_OK) return rc;
      }
      return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
    } else {
      return SPDL_ERR_UNSUPPORTED;
    }
  }
  if (li.variant == kSddmmSlab || li.variant == kSddmmSlabDma) {
    if constexpr (sizeof(T) == 4) {
      const SddmmSlabShape sh = sddmm_slab_shape(m, k, n);
      const bool dma = li.variant == kSddmmSlabDma;
      int rc;
      if (sh.deferred) rc = launch_sddmm_slab<T, 2, 128, true>(sh, li.grid_x, m, k, n, nnz, ro, ci, L, R, out, scale, st, dma, order);
      else if (sh.U == 1) rc = launch_sddmm_slab<T, 1, 256, false>(sh, li.grid_x, m, k, n, nnz, ro, ci, L, R, out, scale, st, dma, order);
      else rc = launch_sddmm_slab<T, 2, 128, false>(sh, li.grid_x, m, k, n, nnz, ro, ci, L, R, out, scale, st, dma, order);
      if (rc != SPDL_OK) return rc;
      return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
    } else {
      return SPDL_ERR_UNSUPPORTED;
    }
  }
  if (li.variant == kSddmmWindow) {
    if constexpr (sizeof(T) == 4) {
      static std::atomic<bool> configured{false};
      struct Form { decltype(&sddmm_window_kernel<kWinWaves, 1>) kernel; int lds; };
      static const Form forms[3] = {{sddmm_window_kernel<kWinWaves, 1>, sddmm_window_rows(kWinWaves, 1) * 256},
                                    {sddmm_window_kernel<kWinWavesWide, 1>, sddmm_window_rows(kWinWavesWide, 1) * 256},
                                    {sddmm_window_kernel<kWinWavesWide, 2>, sddmm_window_rows(kWinWavesWide, 2) * 512}};
      if (!configured.load()) {
        for (const Form& f : forms)
          if (hipFuncSetAttribute(reinterpret_cast<const void*>(f.kernel), hipFuncAttributeMaxDynamicSharedMemorySize, f.lds) != hipSuccess)
            return SPDL_ERR_LAUNCH;
        configured.store(true);
      }
      const Form& f = forms[n > kWinTile ? 2 : li.rows_per_block == kWinWavesWide ? 1 : 0];
      f.kernel<<<dim3(li.grid_x), dim3(li.block_threads), f.lds, st>>>(m, k, n, nnz, ro, ci, L, R, out, scale);
      return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
    } else {
      return SPDL_ERR_UNSUPPORTED;
    }
  }
  if (li.lanes_per_row == 16) {
    // (both halves of a dot product of more than 64 columns in flight)
    if (li.block_threads == kWave) {
      if (n > 64) sddmm_group_kernel<T, 2, 4><<<grid, dim3(kWave), 0, st>>>(m, n, nnz, li.rows_per_block, ro, ci, L, R, out, scale);
      else sddmm_group_kernel<T, 1, 4><<<grid, dim3(kWave), 0, st>>>(m, n, nnz, li.rows_per_block, ro, ci, L, R, out, scale);
    } else {
      sddmm_group_kernel<T><<<grid, block, 0, st>>>(m, n, nnz, li.rows_per_block, ro, ci, L, R, out, scale);
    }
  } else {
    sddmm_rowstrip_kernel<T><<<grid, block, 0, st>>>(m, n, li.rows_per_block, ro, ci, L, R, out, scale);
  }
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

template <typename T>
int sddmm_nt_impl(int m, int k, int n, int nnz, const int* ro, const int* ci, const T* values, const T* L,
                  const T* Rn, T* out, void* stream) {
  if (!sizes_ok(m, k, n, nnz)) return SPDL_ERR_INVALID;
  if (m == 0 || nnz == 0) return SPDL_OK;
  if (!ro || !ci || !out || values == out || (n > 0 && (!L || !Rn))) return SPDL_ERR_INVALID;
  (void)hipGetLastError();
  if constexpr (sizeof(T) == 4) {
    // dot products of up to 128 columns: the lane kernel, which fetches its slabs of Rn as they lie
    // and transposes them inside LDS (32-bit byte offsets into Rn: n * k * 4 < 2^31)
    if (sddmm_lane_usable<T>(n, nnz, L, Rn) && n <= 128 && k % 4 == 0 && m >= 64 && (int64_t)n * k < ((int64_t)1 << 29) &&
        g_forced[1].load() < 0) {
      // (one sparse row per group: the transposing pass needs registers that two rows' L values take)
      const SddmmLaneShape sh = sddmm_lane_shape(m, k, nnz, true);
      const int grid = slab_grid_size(sh.panels, sh.ksplit);
      hipStream_t st = static_cast<hipStream_t>(stream);
      int rc = SPDL_ERR_UNSUPPORTED;
#define SPDL_LANE_NT(NCHD) \
  if (sh.nchd == NCHD) rc = launch_sddmm_lane<1, NCHD, true>(sh, grid, m, k, n, nnz, ro, ci, L, Rn, out, values, st);
      SPDL_LANE_NT(1) SPDL_LANE_NT(2) SPDL_LANE_NT(3) SPDL_LANE_NT(4)
#undef SPDL_LANE_NT
      if (rc != SPDL_OK) return rc;
      return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
    }
  }
  sddmm_nt_kernel<T><<<dim3((nnz + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(
      m, k, n, nnz, ro, ci, L, Rn, out, values);
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

}  // namespace

extern "C" {

int spdl_spmm(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
              const float* values, const int* row_order, const float* B, float* C, void* stream) {
  return spmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, values, row_order, B, C, stream);
}

int spdl_spmm_f16(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                  const uint16_t* values, const int* row_order, const uint16_t* B, uint16_t* C,
                  void* stream) {
  return spmm_impl<_Float16>(m, k, n, nnz, row_offsets, column_indices,
                             reinterpret_cast<const _Float16*>(values), row_order,
                             reinterpret_cast<const _Float16*>(B), reinterpret_cast<_Float16*>(C), stream);
}

int spdl_spmm_bias_relu(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                        const float* values, const int* row_order, const float* B, const float* bias,
                        int relu, float* C, void* stream) {
  return spmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, values, row_order, B, C, stream, bias,
                          relu != 0);
}

int spdl_spmm_bias_relu_f16(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                            const uint16_t* values, const int* row_order, const uint16_t* B,
                            const uint16_t* bias, int relu, uint16_t* C, void* stream) {
  return spmm_impl<_Float16>(m, k, n, nnz, row_offsets, column_indices,
                             reinterpret_cast<const _Float16*>(values), row_order,
                             reinterpret_cast<const _Float16*>(B), reinterpret_cast<_Float16*>(C), stream,
                             reinterpret_cast<const _Float16*>(bias), relu != 0);
}

int spdl_csr_softmax(int m, int nnz, const int* row_offsets, const float* logits, float scale,
                     float* probabilities, void* stream) {
  if (m < 0 || nnz < 0) return SPDL_ERR_INVALID;
  if (m == 0 || nnz == 0) return SPDL_OK;
  if (!row_offsets || !logits || !probabilities) return SPDL_ERR_INVALID;
  (void)hipGetLastError();
  csr_softmax_kernel<<<dim3((m + 3) / 4), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(
      m, row_offsets, logits, scale, probabilities);
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

int spdl_build_transpose_host(int m, int k, int nnz, const int* ro, const int* ci, int* t_ro, int* t_ci,
                              int* perm) {
  if (m < 0 || k < 0 || nnz < 0 || !ro || !t_ro || (nnz > 0 && (!ci || !t_ci || !perm))) return SPDL_ERR_INVALID;
  if (ro[0] != 0 || ro[m] != nnz) return SPDL_ERR_BAD_CSR;
  // counting sort by column; rows are visited in order, so equal columns keep the row order
  std::fill(t_ro, t_ro + k + 1, 0);
  for (int i = 0; i < m; ++i) {
    if (ro[i + 1] < ro[i] || ro[i + 1] > nnz) return SPDL_ERR_BAD_CSR;
    for (int p = ro[i]; p < ro[i + 1]; ++p) {
      if (ci[p] < 0 || ci[p] >= k) return SPDL_ERR_BAD_CSR;
      ++t_ro[ci[p] + 1];
    }
  }
  for (int c = 0; c < k; ++c) t_ro[c + 1] += t_ro[c];
  // The write cursors live in t_ro itself (no allocation): entry c is advanced as column c fills
  // and ends at the start of column c+1, so shifting the array up by one restores the offsets.
  for (int i = 0; i < m; ++i)
    for (int p = ro[i]; p < ro[i + 1]; ++p) {
      const int t = t_ro[ci[p]]++;
      t_ci[t] = i;
      perm[t] = p;
    }
  for (int c = k; c > 0; --c) t_ro[c] = t_ro[c - 1];
  t_ro[0] = 0;
  return SPDL_OK;
}

int spdl_permute_values(int nnz, int elem_bytes, const int* perm, const void* values, void* out, void* stream) {
  if (nnz < 0 || (elem_bytes != 2 && elem_bytes != 4)) return SPDL_ERR_INVALID;
  if (nnz == 0) return SPDL_OK;
  if (!perm || !values || !out) return SPDL_ERR_INVALID;
  (void)hipGetLastError();
  const dim3 grid((nnz + 255) / 256), block(256);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (elem_bytes == 4)
    permute_values_kernel<float><<<grid, block, 0, st>>>(nnz, perm, static_cast<const float*>(values),
                                                         static_cast<float*>(out));
  else
    permute_values_kernel<uint16_t><<<grid, block, 0, st>>>(nnz, perm, static_cast<const uint16_t*>(values),
                                                            static_cast<uint16_t*>(out));
  return hipGetLastError() == hipSuccess ? SPDL_OK : SPDL_ERR_LAUNCH;
}

int spdl_sddmm(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
               const float* L, const float* R, float* out_values, void* stream) {
  return sddmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, L, R, out_values, stream);
}

int spdl_spmm_banded(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                     const float* values, const float* B, float* C, void* stream) {
  return spmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, values, nullptr, B, C, stream, nullptr, 0, kHintBanded);
}

int spdl_sddmm_banded(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                      const float* L, const float* R, float* out_values, void* stream) {
  return sddmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, L, R, out_values, stream, nullptr, nullptr, kHintBanded);
}

int spdl_spmm_skewed(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                     const float* values, const float* B, float* C, void* stream) {
  return spmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, values, nullptr, B, C, stream, nullptr, 0, kHintSkewed);
}

int spdl_sddmm_skewed(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                      const float* L, const float* R, float* out_values, void* stream) {
  return sddmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, L, R, out_values, stream, nullptr, nullptr, kHintSkewed);
}

int spdl_sddmm_ordered(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                       const int* row_order, const float* L, const float* R, float* out_values, void* stream) {
  return sddmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, L, R, out_values, stream, nullptr, row_order);
}

int spdl_sddmm_nt(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                  const float* values, const float* L, const float* Rn, float* out_values, void* stream) {
  return sddmm_nt_impl<float>(m, k, n, nnz, row_offsets, column_indices, values, L, Rn, out_values, stream);
}

int spdl_sddmm_nt_f16(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                      const uint16_t* values, const uint16_t* L, const uint16_t* Rn, uint16_t* out_values,
                      void* stream) {
  return sddmm_nt_impl<_Float16>(m, k, n, nnz, row_offsets, column_indices,
                                 reinterpret_cast<const _Float16*>(values), reinterpret_cast<const _Float16*>(L),
                                 reinterpret_cast<const _Float16*>(Rn), reinterpret_cast<_Float16*>(out_values),
                                 stream);
}

int spdl_spmm_f16_i16(int m, int k, int n, int nnz, const int* row_offsets, const int16_t* column_indices,
                      const uint16_t* values, const int* row_order, const uint16_t* B, uint16_t* C,
                      void* stream) {
  if (k > 32767) return SPDL_ERR_INVALID;           // the indices must fit 16 signed bits
  return spmm_impl<_Float16, int16_t>(m, k, n, nnz, row_offsets, column_indices,
                                      reinterpret_cast<const _Float16*>(values), row_order,
                                      reinterpret_cast<const _Float16*>(B), reinterpret_cast<_Float16*>(C), stream);
}

int spdl_sddmm_scaled(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                      const float* values, const float* L, const float* R, float* out_values, void* stream) {
  if (nnz > 0 && (!values || values == out_values)) return SPDL_ERR_INVALID;
  return sddmm_impl<float>(m, k, n, nnz, row_offsets, column_indices, L, R, out_values, stream, values);
}

int spdl_sddmm_scaled_f16(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                          const uint16_t* values, const uint16_t* L, const uint16_t* R, uint16_t* out_values,
                          void* stream) {
  if (nnz > 0 && (!values || values == out_values)) return SPDL_ERR_INVALID;
  return sddmm_impl<_Float16>(m, k, n, nnz, row_offsets, column_indices,
                              reinterpret_cast<const _Float16*>(L), reinterpret_cast<const _Float16*>(R),
                              reinterpret_cast<_Float16*>(out_values), stream,
                              reinterpret_cast<const _Float16*>(values));
}

int spdl_sddmm_f16(int m, int k, int n, int nnz, const int* row_offsets, const int* column_indices,
                   const uint16_t* L, const uint16_t* R, uint16_t* out_values, void* stream) {
  return sddmm_impl<_Float16>(m, k, n, nnz, row_offsets, column_indices,
                              reinterpret_cast<const _Float16*>(L), reinterpret_cast<const _Float16*>(R),
                              reinterpret_cast<_Float16*>(out_values), stream);
}

int spdl_build_row_order(int m, const int* row_offsets_host, int* row_order_host) {
  if (m < 0 || (m > 0 && (!row_offsets_host || !row_order_host))) return SPDL_ERR_INVALID;
  std::iota(row_order_host, row_order_host + m, 0);
  try {                                   // std::stable_sort allocates a merge buffer
    std::stable_sort(row_order_host, row_order_host + m, [&](int a, int b) {
      return row_offsets_host[a + 1] - row_offsets_host[a] > row_offsets_host[b + 1] - row_offsets_host[b];
    });
  } catch (...) {
    return SPDL_ERR_NOMEM;
  }
  return SPDL_OK;
}

int spdl_validate_csr_host(int m, int k, int nnz, const int* ro, const int* ci, int* sorted_out) {
  if (m < 0 || k < 0 || nnz < 0 || !ro || (nnz > 0 && !ci)) return SPDL_ERR_INVALID;
  if (ro[0] != 0 || ro[m] != nnz) return SPDL_ERR_BAD_CSR;
  int sorted = 1;
  for (int i = 0; i < m; ++i) {
    if (ro[i + 1] < ro[i] || ro[i + 1] > nnz) return SPDL_ERR_BAD_CSR;
    for (int p = ro[i]; p < ro[i + 1]; ++p) {
      if (ci[p] < 0 || ci[p] >= k) return SPDL_ERR_BAD_CSR;
      if (p > ro[i] && ci[p] <= ci[p - 1]) sorted = 0;
    }
  }
  if (sorted_out) *sorted_out = sorted;
  return SPDL_OK;
}

int spdl_select_spmm(int m, int k, int n, int nnz, int elem_bytes, const void* B, const void* C,
                     spdl_launch_info* info) {
  if (!info || !sizes_ok(m, k, n, nnz) || (elem_bytes != 2 && elem_bytes != 4)) return SPDL_ERR_INVALID;
  if (elem_bytes == 4) fill_spmm_info<float>(m, k, n, nnz, B, C, info);
  else fill_spmm_info<_Float16>(m, k, n, nnz, B, C, info);
  return SPDL_OK;
}

int spdl_select_sddmm(int m, int k, int n, int nnz, int elem_bytes, const void* L, const void* R,
                      spdl_launch_info* info) {
  if (!info || !sizes_ok(m, k, n, nnz) || (elem_bytes != 2 && elem_bytes != 4)) return SPDL_ERR_INVALID;
  if (elem_bytes == 4) fill_sddmm_info<float>(m, k, n, nnz, L, R, info);
  else fill_sddmm_info<_Float16>(m, k, n, nnz, L, R, info);
  return SPDL_OK;
}

int spdl_force_variant(int op, int variant) {
  if (op < 0 || op > 1) return SPDL_ERR_INVALID;
  const int limit = op == 0 ? kSpmmVariants : kSddmmVariants;
  if (variant >= limit) return SPDL_ERR_INVALID;
  g_forced[op].store(variant < 0 ? -1 : variant);
  return SPDL_OK;
}

const char* spdl_variant_name(int op, int variant) {
  static const char* const spmm[] = {"rowsplit", "slab", "slabdma", "mfma", "window"};
  static const char* const sddmm[] = {"rowstrip", "group", "slab", "slabdma", "mfma", "lane", "window"};
  if (op == 0 && variant >= 0 && variant < kSpmmVariants) return spmm[variant];
  if (op == 1 && variant >= 0 && variant < kSddmmVariants) return sddmm[variant];
  return nullptr;
}

const char* spdl_status_string(int status) {
  switch (status) {
    case SPDL_OK: return "ok";
    case SPDL_ERR_INVALID: return "invalid argument";
    case SPDL_ERR_LAUNCH: return "kernel launch failed";
    case SPDL_ERR_BAD_CSR: return "not a valid CSR topology";
    case SPDL_ERR_UNSUPPORTED: return "variant does not support this problem";
    case SPDL_ERR_NOMEM: return "host allocation failed";
    default: return "unknown status";
  }
}

int spdl_version(void) { return 140; }

}  // extern "C"

// Not part of the interface (spdl.h), for the tests: the form of the slab SpMM that such a call runs (SlabForm; -1: rows shared by
// lane groups or eight waves), and what the choice among them rests on.
extern "C" int spdl_debug_slab_form(int m, int k, int n, int nnz) {
  spdl_launch_info info;
  SlabPlan plan = {kSlabOneRow, 0, 0};
  fill_spmm_slab_info(m, k, n, nnz, kSpmmSlabDma, &info, &plan);
  return plan.tpw == 0 ? -1 : plan.form;
}
extern "C" int spdl_debug_slab_makespan(int panels, int tiles, int units, int unit, int setup) {
  return slab_makespan(panels, tiles, units, unit, setup);
}

#ifdef SPDL_PHASE_CLOCKS
// Diagnostic build only (microbench/phase_clocks.py): the table the instrumented kernels leave.
extern "C" int spdl_debug_phase_clocks(unsigned long long* host, size_t count) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(spdl::spdl_phase_table), count * sizeof(unsigned long long));
}
#endif
