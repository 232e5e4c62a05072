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
  int h, at;  // head, and which group of query tiles of it; behind the last one where the grid's last row is longer than needed
};

// Workgroup b of H heads with n groups of query tiles each (fewer than 2^31 in all), the first `inside` of which start in the
// true-mask block. The query tiles of the true-mask block come first, for all heads: their tiles are loaded and evaluated word by
// word, one after the other, and where each head's turn came by itself the last heads' were still at it when the chip had nothing
// else left to do. (64 heads x 128k tokens, captured at 4096: scan 191 -> 141 us, fill 422 -> 270.) Patterns without a true-mask
// block go head by head (32 heads x 32k the fill 43 us, by turns 46).
// The pattern rows behind a true-mask block, by_heads (the fill): the last group of every head, which a ragged length leaves to
// be evaluated entry by entry, then head by head, which keeps what a head's rows write and read together. Else (the scan, where
// what counts is that the long rows are spread): the heads in turn, the longest rows first. By turns / by heads, us: 32 heads x
// 32768 captured at 1024 fill 29.6 / 25.7, scan 18.5 / 16.2; 32 x 40000 at 1024 fill 37.7 / 29.6, scan 20.4 / 18.9; 16 x 128k at
// 4096 fill 97 / 70, scan 60 / 55; 16 x 128k at 256 fill 41.6 / 40.0, scan 24.0 / 29.3; 64 x 17000 at 4096 fill 105.9 / 104.7,
// scan 65.8 / 70.4; 32 x 100003 at 4096 fill 110 / 107, scan 64.8 / 67.7. A build that starts with four workgroups a CU or fewer
// (kStartsAtOnce) has nothing to keep together: whole builds of 32 heads x 8192 at 256 (512 workgroups) 29.8 / 30.5, x 4096 at 1024
// (1024) 61.9 / 62.5; 64 x 12000 at 512 (1536) 66.5 / 62.9, 64 x 14300 at 512 (1792) 67.3 / 65.0.
constexpr unsigned kStartsAtOnce = 1024;
constexpr QueryTiles query_tiles_of(unsigned H, unsigned n, unsigned inside, unsigned b, bool by_heads) {
  if (b >= H * n) return QueryTiles{0, (int)n};
  if (inside == 0) return QueryTiles{(int)(b / n), (int)(b % n)};
  const unsigned turn = b / H;
  if (turn < inside) return QueryTiles{(int)(b % H), (int)(inside - 1 - turn)};
  if (turn == inside || !by_heads || H * n <= kStartsAtOnce) return QueryTiles{(int)(b % H), (int)(n - 1 - (turn - inside))};
  const unsigned c = b - H * (inside + 1), each = n - inside - 1;
  return QueryTiles{(int)(c / each), (int)(inside + c % each)};
}

}  // namespace dam
