// Which query tiles of which head a workgroup of the two passes of the block index takes, and the grid they are launched in.
// Plain C++ (constexpr: callable on the device and on the host).
#pragma once
#include <stdint.h>

namespace dam {

// Workgroups are numbered through the grid row by row. A row of all of them would hold more than the 2^32 work-items that a launch
// takes in one direction from 2^24 workgroups on (many maps of long sequences).
constexpr unsigned kGridRow = 16384;
struct TurnGrid {
  unsigned x, y;
};
constexpr TurnGrid turn_grid(int64_t n_turns) {
  const unsigned x = n_turns < (int64_t)kGridRow ? (unsigned)n_turns : kGridRow;
  return TurnGrid{x, (unsigned)((n_turns + x - 1) / x)};
}

struct QueryTiles {
  int h, at;  // head, and which group of `each` query tiles of it; at < 0: the grid's last row is longer than needed
};

// Workgroup b of H heads with n groups of query tiles each (fewer than 2^31 in all), the first `inside` of which start in the true-mask block. The query
// tiles of the true-mask block come first, for all heads: their tiles are loaded and evaluated word by word, one after the
// other, and where each head's turn came by itself the last heads' were still at it when the chip had nothing else left to do.
// Then the others, the longest rows first. (64 heads x 128k tokens, captured at 4096: scan 191 -> 141 us, fill 422 -> 270; 32
// heads x 4096, captured at 1024: scan 11.2 -> 10.0, fill the same.) Patterns without a true-mask block go head by head: 32
// heads x 32k the fill 43 us so, 46 in the other order.
constexpr QueryTiles query_tiles_of(unsigned H, unsigned n, unsigned inside, unsigned b) {
  if (b >= H * n) return QueryTiles{0, -1};
  if (inside == 0) return QueryTiles{(int)(b / n), (int)(b % n)};
  const unsigned turn = b / H;
  return QueryTiles{(int)(b % H), (int)(turn < inside ? inside - 1 - turn : n - 1 - (turn - inside))};
}

}  // namespace dam
