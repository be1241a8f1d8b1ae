// How the units (tiles, or ranges of the contraction axis of a tile) of a launch are dealt to workgroups that take several.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

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
// A short last tile (last < 8 blocks; of columns of 256, where logits_columns_pay says that equal ones do not pay) is computed by workgroups of one
// unit, so the whole launch is: what the short tile saves falls with
// the number of tile columns, what walking saves does not.  Short last tile / walked whole, log-probs at V = 151936, us: four columns, 32 tokens in the last,
// H = 64 74 / 73, 256 103 / 109, 448 135 / 144, 1024 238 / 262, 2048 433 / 478, 4096 827 / 893; five, 100 in the last, 64 96 / 85, 256 135 / 130, 448 178 / 175, 1024
// 317 / 318, 2048 566 / 573, 4096 1073 / 1098; six, 100 in the last, 448 213 / 203, 1024 371 / 373, 2048 677 / 673; seven, 37 or 45 in the last, 256 179 / 175, 512 256 / 269, 1024
// 419 / 434, 4096 1495 / 1511; seven, 100, 448 251 / 240, 1024 437 / 435; eight, 45, 256 208 / 201, 512 295 / 297, 1024 496 / 499, 2048 903 / 915, 4096 1717 / 1749; nine, 45, 512 330 /
// 327, 1024 540 / 542, 2048 1019 / 1014, 4096 1905 / 1908; 17 1024 1031 / 1008, 4096 3630 / 3608; 33 1024 1986 / 1904; 49 4096 10795 / 10422; 100 in the last, eight, 1024 507 / 504,
// 4096 1747 / 1763; nine 4096 1933 / 1916.
inline int short_tile_columns(int kt) { return kt < 12 ? 2 + kt / 2 : 8; }
inline int logits_walk(int units, int kt, int last, int tiles_n) {
  if (kt > kLogitsWalkSlices || (last < 8 && tiles_n <= short_tile_columns(kt))) return 1;
  return walk_length(units, kt);
}
inline int dw_walk(int units, int kt) { return kt <= kDWeightWalkSlices ? walk_length(units, kt) : 1; }

// Width, in blocks of 32 tokens, that each of tiles_n token columns needs if they are equal.  In whole pairs of 32-token
// slices, which dW reads; the logits of a call without one and dH are no wider and no narrower than its logits.
inline int column_blocks(int n_valid, int tiles_n) {
  const int per_block = 32 * tiles_n;
  return ((n_valid + 63) / 64 * 64 + per_block - 1) / per_block;
}

// A call that reads W as it is may have equal columns of 64 to 224 tokens instead of columns of 256 with a short last one: up to 192 tokens, and 257 to
// 448, 513 to 640, 769 to 896, 1025 to 1088 and 1281 to 1344.  They are walked, none is a nearly empty one, and up to 160 wide there is room for a ring
// of six slices: such a launch waits for W, and what is in flight of it decides, the less so as the columns that share its rows ask for the same.  Where that
// pays, whole log-prob call, us, columns of 256 / equal ones (tiles_m rows of tiles, kt slices):
//   one column up to 128 wide: H = 1024, V = 16000 65 tokens 27.8 / 26.7; H = 2048, V = 32000 38.2 / 35.2; H = 5120, V = 9000 80 / 68.  But a W that stays in the
//     L2s waits for nothing, and the deeper ring costs its first fill: H = 1024, V = 3000 128 tokens +4.9 %; 1536, 5000 +6.8; 2048, 1000 +5.3; 3584, 700 +7.3
//     (W of 6 to 16 MB; from 21 MB on equal ones are faster).
//   192 wide 150 tokens H = 1024 97 / 84, 4096 319 / 288.
//   one round of tiles, any number of columns: -2 to -24 % (two columns V = 5000 H = 1024 -17, three -15, four -8, five -7, six -7).
//   more rounds, up to 128 slices, V = 151936, H = 64 / 1024 / 2048 / 4096, per cent: two columns of 160 tokens -24 / -11 / -7 / -4, of 192 -24 / -7 / -3 / +2, of 224
//     -15 / -8 / -6 / -6; three of 192 -25 / -12 / -8 / -5, of 224 -20 / -6 / -3 / -2; six of 224 -15 / -7 / -5 / -4.
//     Four and five of 224 compute up to 8 % more than four and five of 256 with a last one of 64, and lose where the last round is short of tiles: four, H = 1024 /
//     2048 / 4096, 1.2 rounds (V = 20000) +7 / +8 / +10, 1.95 (32000) -8 / -5 / +1, 3.1 (50000) -2 / 0 / +6, 3.9 (64000) -14 / -7 / -4, 6.1 (100000) +1 / +6 / +5, 7.8
//     (128256) -5 / 0 / 0, 9.3 (151936) +2 / +5 / +3; five, 1.2 (16000) +9 / +9 / +8, 2.4 (32000) 0 / +3 / +1, 3.8 (50000) -10 / -8 / -6, 4.9 (64000) -10 / -6 / -1,
//     11.6 (151936) -5 / -4 / 0.  With up to 24 slices they win from two rounds on (four, H = 576 3.1 +1, 6.1 -2, 9.3 -4; H = 320 -7, -6, -9).
//   beyond 128 slices more than two columns lose up to 8 % (H = 5120, V = 151936: three +2.5, four +7, five +2, six +1); from 128 on two of 192 lose 0 to 3 % where
//     the last round is short (H = 4096, V = 100000 +1, 151936 +2) and, beyond 128, in a single one from three quarters of it on (H = 5120, V = 24000, 28000 and 32000 +2; 20000 -8).
// So chosen, against columns of 256 everywhere: 1472 log-prob calls (1 to 1344 tokens, H = 64 to 5120, V = 700 to 151936) -26 to +1.9 %, 260 loss calls -29 to +1.3 %.
constexpr int64_t kSmallHeadBytes = 20 << 20;
inline bool logits_columns_pay(int blocks, int tiles_n, int tiles_m, int kt) {
  if (blocks >= 8) return false;
  const int units = tiles_m * tiles_n, rounds = (units + kNumCU - 1) / kNumCU;
  const bool full = units * 20 >= rounds * kNumCU * 19;      // last round
  if (tiles_n == 2 && blocks == 6 && (rounds > 1 ? kt >= 128 && !full : kt > 128 && units > 176)) return false;
  if (rounds == 1) return tiles_n > 1 || blocks > 4 || (int64_t)units * kBN * kt * 64 >= kSmallHeadBytes;
  if (tiles_n <= 2) return true;
  if (kt > kLogitsWalkSlices) return false;
  if (tiles_n == 4 || tiles_n == 5) return kt <= 24 ? rounds > 2 : full && (tiles_n == 5 || rounds <= 4);
  return true;
}

// The same for dH: tiles_m tiles of hidden units, kt slices of the vocabulary, all of them in one round of ranges.  us, a short last column / equal ones: H = 1024
// 150 tokens 109 / 100, 300 188 / 155, 600 240 / 221; H = 4096 300 459 / 456, 1070 1070 / 1057.  Whole loss call with equal columns of dH against without,
// three to six of them, per cent: V = 9000, H = 1024 -2 to -7, 4096 -1 to -3, 5120 -1 to -4; V = 151936, H = 1024 -1 to +3, 4096 -2 to +1, but H = 5120 +1.5 to
// +3.4 (and at V = 32000 +1 to +4).
inline bool dh_columns_pay(int blocks, int tiles_n, int tiles_m, int kt) { return blocks < 8 && (tiles_n <= 2 || tiles_m <= 16 || kt <= 512); }

}  // namespace nat
