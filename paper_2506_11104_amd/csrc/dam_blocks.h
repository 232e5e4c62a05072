// The number of 32-key blocks that a run of listed tiles stands for (bits 1 .. 4 of a tile's kind: its occupied key quarters).
// Plain C++ that reads the run's n bytes and no others, wherever it starts: whole aligned words where there are any, so that
// a long run takes few loads, single bytes in front of and behind them. (constexpr: callable on the device and on the host.)
#pragma once
#include <stdint.h>

namespace dam {

constexpr int blocks_of_tiles(const uint8_t *kind, int n) {
  int blocks = 0, x = 0;
  for (; x < n && (reinterpret_cast<uintptr_t>(kind + x) & 3); ++x) blocks += __builtin_popcount(kind[x] & 0x1Eu);
  for (; x + 4 <= n; x += 4) {
    uint32_t four = 0;
    __builtin_memcpy(&four, __builtin_assume_aligned(kind + x, 4), 4);
    blocks += __builtin_popcount(four & 0x1E1E1E1Eu);
  }
  for (; x < n; ++x) blocks += __builtin_popcount(kind[x] & 0x1Eu);
  return blocks;
}

}  // namespace dam
