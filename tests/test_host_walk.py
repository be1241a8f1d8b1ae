"""How the units of a launch are dealt to workgroups (csrc/walk.hip.h), without a GPU: its host code in a small program."""
import os
import shutil
import subprocess

import pytest

import paper_2603_06619_amd as nat

CSRC = os.path.join(os.path.dirname(os.path.abspath(nat.__file__)), "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "walk.hip.h"
int main() {
  using namespace nat;
  const int units_of[] = {1, 2, 255, 256, 257, 511, 512, 513, 594, 1024, 1188, 1189, 2047, 2970, 9504, 19008, 58212};
  const int slices[] = {2, 8, 10, 32, 38, 80, 112, 128, 160, 256, 480, 512, 513, 8192};
  for (int units : units_of)
    for (int kt : slices) {
      const int walk = walk_length(units, kt), grid = walk_grid(units, walk), rounds = units / kNumCU;
      // no workgroup is dealt more than a third of the launch (two units of a short one), nor more slices than the budget
      if (walk < 1 || (walk > 2 && walk * 3 > rounds) || (walk > 1 && walk * kt > kWalkBudget)) return std::printf("length %d of %d x %d\n", walk, units, kt), 1;
      std::vector<int> taken(units, 0);
      for (int b = 0; b < grid; ++b) {
        const Walk w = walk_of(b, walk, units);
        int n = 0;
        for (int id = w.first; id < w.end; id += kNumCU, ++n) {
          if (id < 0 || id >= units || taken[id]++) return std::printf("unit %d of %d\n", id, units), 1;
          if (id % kNumCU != b % kNumCU || id / (walk * kNumCU) != b / kNumCU) return std::printf("order: unit %d, workgroup %d\n", id, b), 1;
        }
        if (n < 1 || n > walk) return std::printf("workgroup %d takes %d of %d\n", b, n, units), 1;
      }
      for (int id = 0; id < units; ++id)
        if (!taken[id]) return std::printf("unit %d of %d left out\n", id, units), 1;
    }
  // long contractions: one unit per workgroup (a hidden size of 5120 is 160 slices; 8192 tokens of dW are 256)
  if (logits_walk(44550, 128, 8, 75) < 2 || logits_walk(44550, 130, 8, 75) != 1 || logits_walk(19008, 160, 8, 32) != 1) return std::printf("logits\n"), 1;
  if (dw_walk(9504, 256) < 2 || dw_walk(9504, 258) != 1) return std::printf("dW\n"), 1;
  // one token more than 64 full tile columns does not take the walk from them; 45 more than one does, whose short tile saves more
  if (last_blocks(16385, 65) != 2 || logits_walk(594 * 65, 32, 2, 65) < 2) return std::printf("16385 tokens\n"), 1;
  if (last_blocks(301, 2) != 2 || logits_walk(594 * 2, 32, 2, 2) != 1) return std::printf("301 tokens\n"), 1;
  for (int kt = 2; kt <= 128; kt += 2)
    for (int last = 2; last < 8; last += 2)
      if (logits_walk(594 * 2, kt, last, 2) != 1 || logits_walk(594 * 9, kt, last, 9) < 2) return std::printf("short tile, %d slices\n", kt), 1;
  // equal token columns: as many blocks as the tokens need, never more than the columns of 256 hold, and none for ordinary widths
  for (int n = 1; n <= 7168; ++n) {
    const int tiles = (n + kBN - 1) / kBN, blocks = column_blocks(n, tiles);
    const bool narrow = n <= 192 || (n > 256 && n <= 448) || (n > 512 && n <= 640) || (n > 768 && n <= 896) || (n > 1024 && n <= 1088) || (n > 1280 && n <= 1344);
    if (blocks > 8 || blocks * 32 * tiles < (n + 63) / 64 * 64 || (blocks < 8) != narrow) return std::printf("%d tokens: %d blocks\n", n, blocks), 1;
    if (blocks == 8 && (logits_columns_pay(8, tiles, 36, 32) || dh_columns_pay(8, tiles, 4, 288))) return std::printf("%d tokens, width of 256\n", n), 1;
  }
  // where both sides were timed: {tokens, H, V, equal columns of the logits, of dH}
  const struct { int n, H, V; bool logits, dh; } timed[] = {
      {100, 2048, 1000, false, true}, {128, 1024, 3000, false, true}, {1, 1024, 700, false, true}, {65, 1024, 32000, true, true}, {40, 64, 151936, true, true},
      {150, 192, 1000, true, true}, {150, 4096, 151936, true, true}, {300, 5120, 151936, true, true}, {301, 1024, 151936, true, true}, {330, 2048, 151936, true, true},
      {330, 4096, 151936, false, true}, {330, 5120, 32000, false, true}, {330, 5120, 20000, true, true}, {330, 4096, 64000, true, true}, {448, 5120, 151936, true, true}, {513, 4096, 151936, true, true}, {640, 1024, 32000, true, true},
      {513, 5120, 151936, false, false}, {600, 5120, 9000, true, true}, {769, 1024, 151936, false, true}, {832, 2048, 151936, false, true}, {832, 5120, 151936, false, false},
      {800, 64, 151936, true, true}, {800, 1024, 20000, false, true}, {800, 320, 20000, false, true}, {800, 1024, 32000, true, true}, {800, 4096, 100000, false, true},
      {1025, 2048, 32000, false, true}, {1025, 1024, 16000, false, true}, {1088, 5120, 151936, false, false}, {1088, 1024, 151936, true, true}, {1025, 4096, 9000, true, true},
      {1300, 4096, 151936, true, true}, {1300, 5120, 151936, false, false}};
  for (auto t : timed) {
    const int tiles = (t.n + kBN - 1) / kBN, blocks = column_blocks(t.n, tiles), rows = (t.V + 255) / 256;
    if (logits_columns_pay(blocks, tiles, rows, t.H / 32) != t.logits || dh_columns_pay(blocks, tiles, (t.H + 255) / 256, rows * 8) != t.dh)
      return std::printf("columns of %d tokens, H = %d, V = %d\n", t.n, t.H, t.V), 1;
  }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_units_are_dealt_once_in_order_and_in_short_walks(tmp_path):
    src, exe = tmp_path / "walk.hip", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout
