// The choice of row tiles by the rows that the experts have (tile_rules.h), over row counts from
// even to one expert with everything, capacities from tight to sixteen times the rows:
//  - the chosen tiles' rounds of the CUs, at their K step's time, come to no more than those of the
//    kernel's own (recomputed here by another route), and the launch that was sized for the kernel's own tiles holds them: where it does not,
//    they are not taken;
//  - a single expert has short tiles only where they take 96 to 160 of the 256 CUs, and long groups
//    never have them, however loose the capacity is.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "tile_rules.h"

using namespace moe;

static unsigned seed = 1;
static unsigned rnd() { return seed = seed * 1664525u + 1013904223u, seed >> 8; }

static int tiles(const std::vector<int>& rows, int h) {
  long n = 0;
  for (int m : rows) n += (m + h - 1) / h;
  return int(n);
}

static RowTiles count(const std::vector<int>& rows, int bm) {
  RowTiles t{tiles(rows, bm), tiles(rows, 64), tiles(rows, 96), tiles(rows, 128), 96};
  for (int m : rows)
    if (m > 0) {
      const int n = (m + bm - 1) / bm, high = ((m + n - 1) / n + 31) / 32 * 32;
      t.tallest = high > t.tallest ? high : t.tallest;
    }
  return t;
}

static void fail(const char* what, const ShortTiles& s, int n, int own_rows, int got) {
  std::fprintf(stderr, "%s: nt %d nt_own %d cap %d grid %d experts %d own tiles %d chosen %d\n", what, s.nt, s.nt_own,
               s.cap, s.grid, n, own_rows, got);
  std::exit(3);
}

int main() {
  long taken = 0, seen = 0, refused = 0;
  const int hs[][2] = {{7168, 1024}, {7168, 2048}, {7168, 512}, {2048, 768}, {4096, 1536}, {4096, 128}, {128, 128}, {256, 4096}};
  const int experts[] = {1, 2, 3, 8, 16, 32, 48, 128, 512};
  const int averages[] = {1, 3, 13, 20, 47, 64, 65, 97, 130, 200, 520, 3000};
  for (const auto& z : hs)
    for (int n : experts)
      for (int avg : averages)
        for (int skew = 0; skew < 6; ++skew)
          for (int loose = 1; loose <= 16; loose *= 4) {
            std::vector<int> rows(n);
            const long all = long(n) * avg;
            long left = all;
            for (int e = 0; e < n; ++e) {
              const double even = double(all) / n;
              const double want = skew == 0 ? even : skew == 5 ? (e == n / 2 ? double(all) : 0.0)
                                                               : even * std::pow(rnd() % 1000 / 500.0 + 1e-3, skew);
              rows[e] = int(want < double(left) ? want : double(left));
              left -= rows[e];
            }
            long have = 0;
            for (int m : rows) have += m;
            const int capacity = int(all * loose);
            for (int g = 0; g < 3; ++g) {                 // GEMM-1, GEMM-2 on tall tiles, on wide ones
              const bool gemm1 = g == 0, wide = g == 2;
              const int N = gemm1 ? z[1] : z[0], K = gemm1 ? z[0] : z[1], bn = gemm1 ? 128 : 256, own_bn = wide ? 512 : bn;
              for (int bm : {128, 160, 256}) {
                if (wide && bm != 128) continue;
                const int nt_own = (N + own_bn - 1) / own_bn, own = tiles(rows, bm);
                ShortTiles s{(N + bn - 1) / bn, nt_own, K / 64 / kSplitMinSteps,
                             tall_grid(max_row_tiles(capacity, n, bm), nt_own, wide), gemm1, wide};
                const RowTiles t = count(rows, bm);
                const int h = short_tile_rows(s, n, t);
                ++seen;
                ShortTiles free_grid = s;
                free_grid.grid = 0x7fffffff;
                refused += short_tile_rows(free_grid, n, t) != h;
                if (h == 0) continue;
                ++taken;
                if (h != 64 && (wide || (h != 96 && h != 128))) fail("height", s, n, own, h);
                const long total = long(tiles(rows, h)) * s.nt;
                if ((n == 1 ? (total + 7) / 8 * 8 : split_grid(total, s.cap)) > s.grid) fail("grid", s, n, own, h);
                if (n == 1) {
                  if (!gemm1 || h != 128 || total < 96 || total > 160) fail("single expert", s, n, own, h);
                  continue;
                }
                const long mine = rounds12(total, s.cap), theirs = rounds12(long(own) * nt_own, s.cap) * (wide ? 2 : 1);
                const double step = h == 64 ? 20 : h == 96 ? (gemm1 ? 24 : 23) : (gemm1 ? 27 : 26);
                const double own_steps[2][6] = {{23, 24, 26, 28, 30, 32}, {26, 27, 29, 32, 35, 38}};
                double theirs_step = own_steps[gemm1][t.tallest / 32 - 3];
                if (gemm1 && theirs > 18 && theirs_step > 28) theirs_step = 28;
                if (wide ? mine >= theirs : mine * step > theirs * theirs_step) fail("rounds", s, n, own, h);
                if (h == 128 && t.t64 > 1.4 * t.t128) fail("full tiles", s, n, own, h);
                if (theirs < 12) fail("less than a round", s, n, own, h);
              }
            }
          }
  // rows per expert that fill the tall tiles, whatever the capacity (7168 -> 1024, 32 experts), and
  // a shared expert of thousands of rows, however many experts its layer has
  for (int m : {200, 512, 1024}) {
    std::vector<int> rows(32, m);
    ShortTiles s{8, 8, 4, tall_grid(max_row_tiles(32 * m, 32, 160), 8, false), true, false};
    if (short_tile_rows(s, 32, count(rows, 160))) fail("long groups", s, 32, m, -1);
  }
  for (int m : {64, 400, 640, 1000, 2600, 4096, 8192, 16384}) {
    std::vector<int> rows(1, m);
    ShortTiles s{8, 8, 4, tall_grid(max_row_tiles(m, 1, 256), 8, false), true, false};
    if (short_tile_rows(s, 1, count(rows, 256))) fail("shared expert", s, 1, m, -1);
  }
  // and batches that do take them: 32 experts of 40 rows; the same with one of 90; 1531 tokens of the shared expert
  {
    std::vector<int> rows(32, 40);
    ShortTiles s{8, 8, 4, tall_grid(max_row_tiles(32 * 40 * 8, 32, 256), 8, false), true, false};
    if (short_tile_rows(s, 32, count(rows, 256)) != 64) fail("even batch", s, 32, 40, 0);
    std::vector<int> mixed = rows;
    mixed[3] = 97;
    for (int e = 4; e < 15; ++e) mixed[e] = 70;
    if (short_tile_rows(s, 32, count(mixed, 256)) != 128) fail("one of four row blocks", s, 32, 40, 0);
    rows[3] = 90;
    if (short_tile_rows(s, 32, count(rows, 256)) != 96) fail("a longer group", s, 32, 40, 0);
    std::vector<int> one(1, 1531);
    ShortTiles u{8, 8, 4, tall_grid(max_row_tiles(1531, 1, 256), 8, false), true, false};
    if (short_tile_rows(u, 1, count(one, 256)) != 128) fail("a share of the CUs", u, 1, 1531, 0);
  }
  if (taken < 100 || refused * 100 > taken) {
    std::fprintf(stderr, "%ld of %ld taken, %ld refused for the launch's size\n", taken, seen, refused);
    return 4;
  }
  std::printf("tile rules: ok, short tiles in %ld of %ld, %ld refused for the launch's size\n", taken, seen, refused);
  return 0;
}
