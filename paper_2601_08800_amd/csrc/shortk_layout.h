// Where the short-K GEMM-2 kernel reads the weights: plain index arithmetic, apart from
// the kernel so that it can be checked on the CPU.
#pragma once

#include <stddef.h>

namespace moe {

constexpr int kShortKMax = 128;             // longest K of the kernel
constexpr int kShortKOut = 0x7fffffff;      // a lane offset that is out of every window: reads zeros

// NKS: K sub-steps of 16.  Counts of 16-byte slots.
template <int NKS> struct ShortK {
  static constexpr int kPieces = NKS * 2 + 1;                      // of an LDS row: odd
  static constexpr int kLoads = 2 * kPieces;                       // instructions of 64 slots per stage
  static constexpr int kTurn = 32 * 9;                             // one wavefront's 32 x 64 outputs
  static constexpr int kLoaded = 128 * kPieces;                    // 128 weight rows
  static constexpr int kStage = kLoaded > 4 * kTurn ? kLoaded : 4 * kTurn;
};

// Byte offset, inside the block's window, of what goes to slot `slot` of a stage.
template <int NKS> constexpr int shortk_slot_offset(int slot, int K) {
  const int row = slot / ShortK<NKS>::kPieces, piece = slot - row * ShortK<NKS>::kPieces;
  return piece * 8 < K ? (row * K + piece * 8) * 2 : kShortKOut;
}

// The rows of one expert's w_down [N, K] that block nb of 128 output columns has.
struct ShortKWindow {
  size_t first;   // byte offset of the first
  int bytes;      // length
};
constexpr ShortKWindow shortk_window(int nb, int N, int K) {
  const int rows = N - nb * 128 < 128 ? N - nb * 128 : 128;
  return {size_t(nb) * 128 * K * 2, rows * K * 2};
}

}  // namespace moe
