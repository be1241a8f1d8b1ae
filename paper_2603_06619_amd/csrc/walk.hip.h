// How the units (tiles, or ranges of the contraction axis of a tile) of a launch are dealt to workgroups that take several.
#pragma once
#include <hip/hip_runtime.h>

namespace nat {

constexpr int kNumCU = 256;        // compute units (one workgroup of the matrix kernels each)
constexpr int kBN = 256;           // columns of a tile

// 16-column blocks per wavefront (two wavefronts side by side) that the last of tiles_n tiles needs for n_valid columns
__host__ __device__ inline int last_blocks(int n_valid, int tiles_n) {
  const int n = n_valid - (tiles_n - 1) * kBN;
  return n <= 64 ? 2 : n <= 128 ? 4 : 8;
}

// Groups of kNumCU workgroups take walk * kNumCU consecutive units each, workgroup b of a group its units b, b + kNumCU, ...: the units
// start in the order in which one workgroup per unit would start them, and on the same XCD.
struct Walk { int first, end; };   // units first, first + kNumCU, ... below end
__host__ __device__ inline Walk walk_of(int block, int walk, int units) {
  const int start = block / kNumCU * walk * kNumCU;
  return Walk{start + block % kNumCU, units - start < walk * kNumCU ? units : start + walk * kNumCU};
}

// workgroups of such a launch
inline int walk_grid(int units, int walk) {
  const int per_group = walk * kNumCU, rest = units % per_group;
  return units / per_group * kNumCU + (rest < kNumCU ? rest : kNumCU);
}

// Units per workgroup of a launch of units of kt k-slices each.  A compute unit that another stream's kernel holds takes nothing until that
// ends, and what its workgroup was dealt waits: so a walk is at most a third of the launch's rounds of one unit per compute unit (but
// two units), and at most kWalkBudget slices, by which the ring's first fill is a few per cent.  Log-probs beside a kernel on
// another stream that holds 16 / 32 compute units, time against the same call alone; one unit each, every unit dealt in advance, as
// here: 8192 tokens at H = 1024 1.19 / 1.23, 1.86 / 1.98, 1.24 / 1.26; 2048 at H = 4096 1.11 / 1.15, 1.81 / 1.83, 1.13 / 1.20; 512 at H = 1024
// 1.18 / 1.20, 1.44 / 1.49, 1.13 / 1.26.  What it costs alone, us, in the same order: 1963, 1852, 1861; 512 tokens 153, 142, 146; dW of 300 tokens at
// H = 4096 694, 605, 612.  A budget of 1024 slices is no faster and 1.29 / 1.35 beside the other kernel.
constexpr int kWalkBudget = 512;
inline int walk_length(int units, int kt) {
  const int rounds = units / kNumCU, most = kWalkBudget / kt;
  const int walk = rounds / 3 > 2 ? rounds / 3 : 2;
  return walk < most ? walk : most > 1 ? most : 1;
}

// Contractions of up to so many k-slices are walked: over one unit per workgroup that saves the ring's first fill and the clearing of the
// accumulators (7 k cycles of a tile that has 1090 per slice and 11 k of epilogue).  One unit each / walking, us, in turn on one box:
// logits at H = 1024 with 512 tokens 153 / 146, 1237 339 / 324, 8192 1963 / 1861; 8192 tokens at 3584 6220 / 6177, at 4096 6977 / 6976, but at 5120
// 8904 / 8961 and 25000 tokens there 27000 / 28162 (equal on another box): the longer the tiles, the further the workgroups of an XCD drift apart.
// dW at H = 4096 with 300 tokens 694 / 612, 1237 (accumulating) 1731 / 1628, 8192 7058 / 7021, but 16384 (accumulating) 14182 / 14182.  dH has two rounds
// of thousands of slices: one unit each.
constexpr int kLogitsWalkSlices = 128, kDWeightWalkSlices = 256;
// A short last tile (last < 8 blocks; of columns of 256, which calls of few tokens that read W as it is do not have) is computed by workgroups of one
// unit, so the whole launch is: what the short tile saves falls with
// the number of tile columns, what walking saves does not.  Short last tile / walked whole, log-probs of 256 (columns - 1) + 45 tokens at
// V = 151936, us: H = 64 2 columns 45.7 / 48.9, 3 63.3 / 63.0, 5 100 / 96; 256 5 133 / 137, 6 157 / 156, 8 208 / 201; 512 7 256 / 269, 8 295 / 297,
// 9 330 / 327; 1024 7 419 / 434, 8 496 / 499, 9 540 / 542, 17 1031 / 1008, 33 1986 / 1904; 2048 8 903 / 915, 9 1019 / 1014; 4096 8 1717 / 1749,
// 9 1905 / 1908, 17 3630 / 3608, 49 10795 / 10422; with 100 tokens in the last tile H = 1024 8 507 / 504, 4096 8 1747 / 1763, 9 1933 / 1916.
inline int short_tile_columns(int kt) { return kt < 12 ? 2 + kt / 2 : 8; }
inline int logits_walk(int units, int kt, int last, int tiles_n) {
  if (kt > kLogitsWalkSlices || (last < 8 && tiles_n <= short_tile_columns(kt))) return 1;
  return walk_length(units, kt);
}
inline int dw_walk(int units, int kt) { return kt <= kDWeightWalkSlices ? walk_length(units, kt) : 1; }

}  // namespace nat
