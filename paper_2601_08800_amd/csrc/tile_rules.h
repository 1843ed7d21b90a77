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

// Row tiles that the experts' rows come to at the kernel's own height and at 64, 96 and 128 rows,
// and the rows of the tallest own one.
struct RowTiles {
  int own, t64, t96, t128, tallest;
};

// Height of the short tiles, or 0: the kernel's own.
//  - Several experts: the height whose rounds of the CUs come to the least, each at the time of its
//    tiles' K step.  The steps (of a short tile by 64 / 96 / 128 rows; of an own one by the tallest,
//    up to 96, 128, 160, 192, 224 and 256 rows; a 64-row short tile is 20) were fitted to the
//    times of 308 batches (4 to 170 rows per expert, even to Zipf 1.2, hidden 2048 to 7168, I 384 to 2048,
//    16 to 128 experts) at all four heights: GEMM-1 7 us per 1024 of K at 20.  More rounds take an
//    own tile's step for at most 28, as the shorter tiles beside it fill the CUs.  96 and 128 rows only where
//    tiles of 64 would be at most 1.5 and 1.4 times as many (few long experts among short ones):
//    full ones are slower than the fit (experts of 89 rows, 128-row tiles 253 -> 283).  Of the batches' FFN
//    the rule takes 4.5 % off in GEMM-1 and 1.3 % in GEMM-2; the best choice each time, 6.2 and 2.0;
//    128-row tiles wherever the capacity gives 16 to 64 rows, 1.7 and 0.5.
//    Against the wide tiles only 64 rows, with fewer rounds counted double (1.07 to 1.3 times as fast, 0.90 to
//    1.13 with as many).  Launches of less than a round keep their own tiles, whose K split is
//    the better one (8 experts, I 1024: 0.87 to 0.97).
//  - A single expert (the shared one of a layer, whose route and dispatch run beside it): only GEMM-1,
//    and 128 rows where that gives 96 to 160 tiles, which stay whole: they leave a good part of the CUs
//    to the route, where its own tiles, cut along K, fill them.  Layers of 700 to 4449 tokens (hidden 7168, I 512 to
//    2048) on such tiles against its own, us: 1531 359 -> 338, 1800 468 -> 449, 1902 417 -> 374, 2040 456 -> 399, 2336 425 ->
//    412, 2500 501 -> 490, 4090 436 -> 426, but 1621 386 -> 392, 3128 360 -> 370, 700 (I 2048) 452 -> 467; in the mean 2 %
//    faster.  From 48 to 95 tiles 2 % slower, past 160 as much either way.  Alone they are slower: 1531 rows 107 ->
//    130, 2040 131 -> 139, 2500 150 -> 171.
//    (Tiles of 64 rows, 176 to 256 of them, are the fastest alone, 97 and 110, but 355 and 435 a layer.)
MOE_RULE int own_step(const ShortTiles& s, int tallest, bool rounds) {
  const int nb = (tallest + 31) / 32;
  const int step = s.gemm1 ? (nb <= 3 ? 26 : (nb == 4 ? 27 : (nb == 5 ? 29 : (nb == 6 ? 32 : (nb == 7 ? 35 : 38)))))
                           : (nb <= 3 ? 23 : (nb == 4 ? 24 : (nb == 5 ? 26 : (nb == 6 ? 28 : (nb == 7 ? 30 : 32)))));
  return s.gemm1 && rounds && step > 28 ? 28 : step;
}

MOE_RULE int short_tile_rows(const ShortTiles& s, int n_experts, const RowTiles& t) {
  const long w64 = long(t.t64) * s.nt, w96 = long(t.t96) * s.nt, w128 = long(t.t128) * s.nt;
  if (n_experts == 1) return s.gemm1 && w128 >= 96 && w128 <= 160 && (w128 + 7) / 8 * 8 <= s.grid ? 128 : 0;
  const long r = rounds12(long(t.own) * s.nt_own, s.cap), r64 = rounds12(w64, s.cap);
  if (r < 12) return 0;
  const bool fits64 = split_grid(w64, s.cap) <= s.grid;
  if (s.wide) return fits64 && r64 <= 2 * r - 1 ? 64 : 0;
  long best = r * own_step(s, t.tallest, r > 18) + 1;
  int rows = 0;
  if (fits64 && r64 * 20 < best) { best = r64 * 20; rows = 64; }
  const long c96 = rounds12(w96, s.cap) * (s.gemm1 ? 24 : 23), c128 = rounds12(w128, s.cap) * (s.gemm1 ? 27 : 26);
  if (2 * t.t64 <= 3 * t.t96 && c96 < best && split_grid(w96, s.cap) <= s.grid) { best = c96; rows = 96; }
  if (5 * t.t64 <= 7 * t.t128 && c128 < best && split_grid(w128, s.cap) <= s.grid) rows = 128;
  return rows;
}

}  // namespace moe

#undef MOE_RULE
