"""The block counts that put the prefill's work items into order (dam_blocks.h) are those of the items' own tile kinds, and no
byte behind the caller's array is read, whatever its alignment and length: the header, plain C++, runs here on the CPU under
AddressSanitizer over arrays of exactly the size read."""
import os
import subprocess

from paper_2506_11104_amd import build as hip_build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "dam_blocks.h"
int main() {
  for (int lead = 0; lead < 4; ++lead)
    for (int n = 0; n <= 70; ++n) {
      // an array that starts anywhere and ends where its allocation does; what stands in front would change the count
      uint8_t *const all = static_cast<uint8_t *>(malloc(lead + n));
      uint8_t *const kind = all + lead;
      int want = 0;
      for (int x = 0; x < lead; ++x) all[x] = 0xFF;
      for (int x = 0; x < n; ++x) {
        kind[x] = static_cast<uint8_t>(rand());
        want += __builtin_popcount(kind[x] >> 1 & 15);
      }
      const int got = dam::blocks_of_tiles(kind, n);
      if (got != want) return std::printf("lead %d, %d tiles: %d, not %d\n", lead, n, got, want), 1;
      free(all);
    }
  return std::puts("all"), 0;
}
"""


def test_only_the_tiles_own_kinds_are_read(tmp_path):
    src, exe = tmp_path / "blocks.cpp", tmp_path / "blocks"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I" + hip_build.CSRC, str(src),
                    "-o", str(exe)], check=True, timeout=120)
    env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0:detect_leaks=0")
    r = subprocess.run([str(exe)], env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "all", r.stdout + r.stderr[-2000:]
