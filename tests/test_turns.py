"""The turns of the block index's two passes (dam_turns.h, plain C++): the grid numbers every group of query tiles of every head
exactly once, and none of its directions exceeds what a launch of 256 work-items per workgroup takes. On the CPU."""
import subprocess

from paper_2506_11104_amd import build as hip_build

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "dam_turns.h"
using namespace dam;
#define CHECK(x) if (!(x)) return std::printf("%s: H %lld n %d inside %d\n", #x, (long long)H, n, inside), 1
int main() {
  const int sizes[][2] = {{1, 1}, {1, 7}, {3, 1}, {64, 16}, {64, 17}, {64, 256}, {64, 257}, {16384, 1}, {16385, 1}, {4097, 4}, {40, 1000}};
  for (auto &s : sizes)
    for (int inside : {0, 1, s[1] / 2, s[1]})
      for (bool by_heads : {false, true}) {
        const int64_t H = s[0];
        const int n = s[1];
        const TurnGrid g = turn_grid(H * n);
        std::vector<char> seen(H * n, 0);
        QueryTiles before{0, -1};
        for (unsigned y = 0; y < g.y; ++y)
          for (unsigned x = 0; x < g.x; ++x) {
            const int64_t b = (int64_t)y * g.x + x;
            const QueryTiles t = query_tiles_of((unsigned)H, n, inside, (unsigned)b, by_heads);
            CHECK((t.at == n) == (b >= H * n));
            if (t.at == n) continue;
            CHECK(t.h >= 0 && t.h < H && t.at >= 0 && t.at < n && !seen[t.h * n + t.at]);
            seen[t.h * n + t.at] = 1;
            // the true-mask block first, then every head's last group; whose turn it is next, by heads and by turns
            CHECK(inside == 0 || (b < H * inside) == (t.at < inside));
            CHECK(inside == 0 || b < H * inside || (b < H * (inside + 1)) == (t.at == n - 1));
            const bool heads = inside == 0 || (by_heads && H * n > 1024 && b > H * (inside + 1));
            if (b > 0 && b != H * (inside + 1)) CHECK(heads ? t.h - before.h == (t.at == inside) : t.h == (before.h + 1) % H);
            before = t;
          }
        for (char c : seen) CHECK(c);
      }
  // many maps of long sequences: 65535 x 65600 tokens, 5120 x 1M, tiles of 64
  const int64_t many[][2] = {{65535, 257}, {5120, 4096}, {1, 1 << 20}, {300000, 1000}};
  for (auto &s : many) {
    const int64_t H = s[0];
    const int n = (int)s[1], inside = 0;
    const TurnGrid g = turn_grid(H * n);
    CHECK((int64_t)g.x * 256 < (1LL << 32) && g.y <= 65535 && (int64_t)g.x * g.y >= H * n && (int64_t)g.x * (g.y - 1) < H * n);
  }
  return std::puts("all"), 0;
}
"""


def test_every_query_tile_has_one_turn(tmp_path):
    src, exe = tmp_path / "turns.cpp", tmp_path / "turns"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I" + hip_build.CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "all", r.stdout + r.stderr
