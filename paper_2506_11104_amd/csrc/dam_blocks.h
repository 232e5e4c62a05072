// The number of 32-key blocks that a run of listed tiles stands for (bits 1 .. 4 of a tile's kind: its occupied key quarters).
// Plain C++ that reads the run's n bytes and no others, wherever it starts: aligned words, four of them in flight, and single
// bytes in front of and behind them. (Places past an end are read as the last one inside and not counted, so that no load waits
// for a test. constexpr: callable on the device and on the host.)
#pragma once
#include <stdint.h>

namespace dam {

constexpr int blocks_of_tiles(const uint8_t *kind, int n) {
  if (n < 1) return 0;
  const int to_word = (int)(-reinterpret_cast<uintptr_t>(kind) & 3), lead = to_word < n ? to_word : n;
  const int words = (n - lead) / 4, tail = n - lead - 4 * words;
  uint32_t ends[6] = {};
  for (int x = 0; x < 3; ++x) {
    const int at = x < n ? x : n - 1;
    ends[x] = kind[at];
    ends[3 + x] = kind[n - 1 - at];
  }
  int blocks = 0;
  for (int w = 0; w < words; w += 4) {
    uint32_t four[4] = {};
    for (int y = 0; y < 4; ++y)
      __builtin_memcpy(&four[y], __builtin_assume_aligned(kind + lead + 4 * (w + y < words ? w + y : words - 1), 4), 4);
    for (int y = 0; y < 4; ++y) blocks += w + y < words ? __builtin_popcount(four[y] & 0x1E1E1E1Eu) : 0;
  }
  for (int x = 0; x < 3; ++x)
    blocks += (x < lead ? __builtin_popcount(ends[x] & 0x1Eu) : 0) + (x < tail ? __builtin_popcount(ends[3 + x] & 0x1Eu) : 0);
  return blocks;
}

}  // namespace dam
