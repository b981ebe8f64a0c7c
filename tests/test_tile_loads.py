"""Every address of the LM-head tile kernel's loads into LDS, walked on the CPU: no lane leaves the
operand, whether the buffer bounds check counts the scalar offset or not, and every row inside the
operand is loaded at its place."""
import subprocess

from paper_2609_16450_amd import build as eb_build

WALK = r"""
#include <cstdio>
#include <vector>
#include "tile_loads.hpp"
using namespace eb;
int main() {
  const uint32_t hiddens[] = {64, 128, 320, 4096};
  for (uint32_t hidden : hiddens) {
    const uint32_t rb = 2 * hidden;
    for (int height = 96; height <= 256; height += 32)      // of a tile: 32 TN positions, or W's 256
      for (int rows = 1; rows <= height; ++rows) {          // of it inside the operand
        std::vector<int> seen(rows, 0);
        for (int q = 0; q < height / 8; ++q) {              // one load instruction: 8 rows
          const int row0 = tile_load_row0(q, rows);
          const uint32_t range = tile_load_range(row0, rows, rb);
          for (uint32_t stage = 0; stage < hidden / 64; stage += hidden / 64 > 1 ? hidden / 64 - 1 : 1)
            for (int lane = 0; lane < 64; ++lane) {
              const uint32_t voff = tile_load_voff(q & 1, lane, rb), soff = stage * 128;
              // the two readings of the check; unsigned, as a wrap would let everything pass
              const bool without = voff + 16 <= range, with = voff + 16 <= range - soff;
              const int row = 8 * q + lane / 8;
              const uint64_t at = uint64_t(row0) * rb + voff + soff;
              if (soff >= range || (without || with) != (without && with)) return 1;
              if (without && at + 16 > uint64_t(rows) * rb) return 2;
              if (row < rows) {
                const int chunk = (lane & 7) ^ tile_swizzle(row);
                if (!without || at != uint64_t(row) * rb + 128 * stage + 16 * chunk) return 3;
                seen[row] += stage == 0 ? 1 : 0;
              }
            }
        }
        for (int n : seen)
          if (n != 8) return 4;                             // eight chunks of 16 bytes
      }
  }
  return 0;
}
"""


def test_loads_stay_in_the_operand(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", eb_build.CSRC, str(src), "-o", str(exe)],
                   check=True)
    assert subprocess.run([str(exe)], timeout=100).returncode == 0
