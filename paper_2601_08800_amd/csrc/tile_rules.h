// How high the row tiles of a grouped GEMM are where that depends on the rows that each expert
// really has: the kernels that write the tile tables decide it, since the host only knows a
// bound on all rows together.  Plain arithmetic, apart from the kernels so that it can be
// checked on the CPU.
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define MOE_RULE __host__ __device__ inline
#else
#define MOE_RULE inline
#endif

namespace moe {

constexpr int kCUs = 256;             // compute units: workgroups of a whole LDS that run at a time
constexpr int kSplitMax = 4;          // parts of a tile that is cut along K, at most
constexpr int kSplitMinSteps = 24;    // ... and the 64-deep K steps of a part, at least

// Parts into which each of the `left` tiles of the last, partly filled round is cut along K
// (`cap`: as many as K allows); 1: they stay whole.  min(kCUs / left, kSplitMax), without a
// division: it stands at the head of every workgroup.
MOE_RULE int split_parts(int left, int cap) {
  if (left <= 0 || left > kCUs / 2) return 1;
  static_assert(kSplitMax == 4, "the steps below");
  const int parts = left > kCUs / 3 ? 2 : (left > kCUs / 4 ? 3 : 4);
  return cap < 1 ? 1 : (parts < cap ? parts : cap);
}

// Time of a launch of `total` tiles in twelfths of a tile's.
MOE_RULE long rounds12(long total, int cap) {
  const int left = int(total & (kCUs - 1)), parts = split_parts(left, cap);
  const int part12 = parts == 1 ? 12 : (parts == 2 ? 6 : (parts == 3 ? 4 : 3));
  return total / kCUs * 12 + (left ? part12 : 0);
}

// Workgroups of such a launch.
MOE_RULE long split_grid(long total, int cap) {
  const int left = int(total & (kCUs - 1));
  return total - left + long(left) * split_parts(left, cap);
}

// Row tiles of at most bm rows, at most.
MOE_RULE int max_row_tiles(int rows_capacity, int n_experts, int bm) {
  return rows_capacity / bm + (n_experts < rows_capacity ? n_experts : rows_capacity);
}

// Workgroups of a launch of the tall-tile kernel: room for the parts of the leftover tiles behind
// the whole ones; `twice`: and for as many tiles of half the width, where the device may choose those.
MOE_RULE int tall_grid(int row_tiles, int nt, bool twice) {
  const int times = twice ? 2 : 1;
  return (row_tiles * nt * times + 7) / 8 * 8 + times * kCUs;
}

// e4m3 weights, bf16 activations: the GEMM that may have the short tiles of e4m3_body in the
// place of the tall-tile kernel's own.
struct ShortTiles {
  int nt;              // column tiles of a short tile's width (0: no choice, the kernel's own tiles) ...
  int nt_own;          // ... and of the kernel's own tiles
  int cap;             // parts along K
  int grid;            // workgroups launched
  bool gemm1, wide;    // wide: 512 weight rows a tile, twice a short one's
};

// Height of the short tiles, or 0: the kernel's own.  t64, t96, own: row tiles that the experts'
// rows come to at 64 rows, at 96 and at the kernel's own height; over128, over192: one of the own
// tiles has more rows than that.
//  - Several experts: the short tiles read codes by whole lines and have all wavefronts work on
//    few rows, but fetch the weights once per 64 rows.  They win where they come to no more
//    rounds of the CUs.  Kernel times of 1770 batches (1 to 200 rows per expert, even to Zipf
//    1.2, hidden 2048 to 7168, I 384 to 2048, 4 to 128 experts) against the kernel's own tiles:
//    GEMM-1 with 64 rows 0.99 to 2.5 times as fast where the rule takes them (mean 1.2; up to 1.25
//    times the rounds against tiles of more than 128 rows, whose K steps are longer, 1.00 to 1.4, up to 1.375
//    times against more than 192 rows 0.99 to 1.4; with as much against lower ones 0.89 to 1.0), 0.73 to
//    1.1 at half as many again; with 96 rows 0.96 to 1.5 (mean 1.13).  GEMM-2 with 64 rows 0.94 to 1.5 (mean
//    1.15), with 96 from 0.90, hence only GEMM-1; against the wide tiles, counted double, 1.07 to 1.3
//    with fewer rounds, 0.90 to 1.13 with as many.  Launches of less than a round keep their own
//    tiles, whose K split is the better one (8 experts, I 1024: 0.87 to 0.97).
//  - A single expert (the shared one of a layer): only GEMM-1 and from 176 to 256 short
//    tiles, nearly one round, where its own tiles are a few that are cut along K.  Alone, hidden
//    7168, us (I 1024 if not said): 136 tiles 91 -> 95, 160 105 -> 98 and (I 2048) 110 -> 111, 192 110 -> 99,
//    232 127 -> 107, 256 129 -> 109; 320 and more were slower.  Beside the routed path of its layer 1300
//    tokens 346 -> 328, 1531 340 -> 319, 2040 462 -> 440 (parts of fewer tiles would keep the CUs from
//    the route: 1000 tokens 312 -> 350).
MOE_RULE int short_tile_rows(const ShortTiles& s, int n_experts, int t64, int t96, int own, bool over128,
                             bool over192) {
  const long w64 = long(t64) * s.nt, w96 = long(t96) * s.nt;
  if (n_experts == 1) return s.gemm1 && w64 >= 176 && w64 <= kCUs && w64 <= s.grid ? 64 : 0;
  const long r = rounds12(long(own) * s.nt_own, s.cap);
  if (r < 12) return 0;
  long most = s.wide ? 2 * r - 1 : r;
  const long most96 = s.gemm1 ? most : 0;
  if (s.gemm1) most += over192 ? r * 3 / 8 : (over128 ? r / 4 : 0);
  if (rounds12(w64, s.cap) <= most && split_grid(w64, s.cap) <= s.grid) return 64;
  return rounds12(w96, s.cap) <= most96 && split_grid(w96, s.cap) <= s.grid ? 96 : 0;
}

}  // namespace moe

#undef MOE_RULE
