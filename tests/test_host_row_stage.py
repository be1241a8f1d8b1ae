"""The LDS staging of fp32 results (csrc/row_stage.hip.h), without a GPU: its host code in a small program."""
import os
import shutil
import subprocess

import pytest

import paper_2603_06619_amd as nat

CSRC = os.path.join(os.path.dirname(os.path.abspath(nat.__file__)), "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <set>
#include "row_stage.hip.h"
using namespace nat;
// the LDS serves 16 lanes at a time over its 64 banks: lanes 0-3, 12-15, 20-27 together, then 4-11, 16-19, 28-31, and the same of the upper half
template <class F> bool conflict_free(F&& at) {
  for (int upper = 0; upper < 64; upper += 32)
    for (int set = 0; set < 2; ++set) {
      std::set<int> chunks;
      for (int l = 0; l < 32; ++l) {
        const bool first = l < 4 || (l >= 12 && l < 16) || (l >= 20 && l < 28);
        if (first == (set == 0)) chunks.insert(at(upper + l) % 64 / 4);
      }
      if (chunks.size() != 16) return false;
    }
  return true;
}
int main() {
  int element[kStageFloats];
  for (int& e : element) e = -1;
  for (int i = 0; i < 4; ++i) {
    for (int l = 0; l < 64; ++l)
      for (int r = 0; r < 4; ++r) {
        const int at = stage_write_at(l, i) + r;
        if (at < 0 || at >= kStageFloats || element[at] != -1) return std::printf("write %d %d\n", l, i), 1;
        element[at] = (l % 16) * 64 + 16 * i + 4 * (l / 16) + r;
      }
    if (!conflict_free([&](int l) { return stage_write_at(l, i); })) return std::printf("banks of write %d\n", i), 1;
  }
  std::set<int> seen;
  for (int j = 0; j < 4; ++j) {
    for (int l = 0; l < 64; ++l)
      for (int r = 0; r < 4; ++r) {
        const int row = stage_read_row(l, j), col = stage_read_column(l) + r;
        if (element[stage_read_at(l, j) + r] != row * 64 + col) return std::printf("read %d %d\n", l, j), 1;
        // what an instruction stores: 256 bytes in a row by 16 lanes, four rows
        if (row != 4 * j + l / 16 || row != stage_read_row(0, j) + stage_read_row(l, 0) || col != 4 * (l % 16) + r) return std::printf("row %d %d\n", l, j), 1;
        seen.insert(row * 64 + col);
      }
    if (!conflict_free([&](int l) { return stage_read_at(l, j); })) return std::printf("banks of read %d\n", j), 1;
  }
  return seen.size() == kStageFloats ? 0 : 1;
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_staged_results_come_back_as_whole_rows(tmp_path):
    src, exe = tmp_path / "stage.hip", tmp_path / "stage"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout
