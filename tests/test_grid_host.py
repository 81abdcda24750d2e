"""The workgroup schedule (csrc/grid.hpp) on the CPU: every (head, tile) exactly
once for each issue order, the most work first within a group of the causal
order, and a head of a full group on one XCD."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_33916_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <set>
#include <utility>
#include <vector>
#include "grid.hpp"
struct Args { int n, ntiles, nblocks, hgroup; };
int main() {
  const int all_heads[] = {1, 2, 7, 8, 9, 12, 16, 24, 64, 65, 100};
  const int all_n[] = {1, 127, 128, 129, 1000, 4096, 16384};
  for (int heads : all_heads) for (int n : all_n) for (int rows : {32, 128, 192, 256}) for (int per_cu : {1, 2, 4})
    for (int causal = 0; causal < 2; ++causal) for (int reverse = 0; reverse < 2; ++reverse) {
      Args a{}; a.n = n;
      attn::set_grid(a, heads, rows, per_cu);
      const int hg = causal ? a.hgroup : 0, rem = causal ? heads % a.hgroup : 0;
      if (a.hgroup < 1 || a.hgroup > heads || (a.hgroup < heads && a.hgroup % 8)) { std::printf("hgroup\n"); return 1; }
      std::set<std::pair<int, int>> seen;
      std::vector<int> last(heads, -1), xcd(heads, -1);
      for (int b = 0; b < a.nblocks; ++b) {
        int h = -1, t = -1;
        attn::block_map(b, a.nblocks, a.ntiles, hg, reverse, h, t);
        if (h < 0 || h >= heads || t < 0 || t >= a.ntiles || !seen.insert({h, t}).second) { std::printf("map\n"); return 1; }
        if (!causal) continue;
        const int rank = reverse ? a.ntiles - 1 - t : t;
        if (rank != last[h] + 1) { std::printf("order\n"); return 1; }
        last[h] = rank;
        if (h >= rem && a.hgroup % 8 == 0) {
          const int x = b % 8;
          if (xcd[h] >= 0 && xcd[h] != x) { std::printf("xcd\n"); return 1; }
          xcd[h] = x;
        }
      }
    }
  std::printf("ok\n");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_block_map_covers_every_tile_once(tmp_path):
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
