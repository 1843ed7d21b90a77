// Walks every load that the short-K GEMM-2 kernel makes of an expert's weights and checks
// that what the hardware reads lies inside that expert's matrix.  The range check is
// taken at its narrowest: it sees the lane's own offset only.
#include <cstdio>
#include <cstdlib>

#include "shortk_layout.h"

template <int NKS> static void walk(int N, int K) {
  using namespace moe;
  const long matrix = long(N) * K * 2;
  const int blocks = (N + 127) / 128;
  long read = 0;
  for (int nb = 0; nb < blocks; ++nb) {
    const ShortKWindow w = shortk_window(nb, N, K);
    for (int slot = 0; slot < ShortK<NKS>::kLoads * 64; ++slot) {
      const int off = shortk_slot_offset<NKS>(slot, K);
      if (off < 0 || long(off) + 16 > w.bytes) continue;      // out of the window: zeros
      const long at = long(w.first) + off;
      if (at < 0 || at + 16 > matrix) {
        std::fprintf(stderr, "N %d K %d block %d slot %d reads %ld of %ld\n", N, K, nb, slot, at, matrix);
        std::exit(3);
      }
      read += 16;
    }
  }
  if (read != matrix) {                                        // each weight exactly once
    std::fprintf(stderr, "N %d K %d: %ld of %ld bytes read\n", N, K, read, matrix);
    std::exit(4);
  }
}

int main() {
  const int Ns[] = {8, 120, 128, 136, 248, 256, 264, 1000, 2048, 2056, 7168, 7288};
  for (int N : Ns)
    for (int K = 8; K <= moe::kShortKMax; K += 8) {
      const int ks = (K + 15) / 16;
      if (ks <= 2) walk<2>(N, K);
      else if (ks <= 4) walk<4>(N, K);
      else if (ks <= 6) walk<6>(N, K);
      else walk<8>(N, K);
    }
  std::puts("short-K loads: ok");
  return 0;
}
