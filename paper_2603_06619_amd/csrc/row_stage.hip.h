// Where a wavefront's 16 x 64 block of fp32 results sits in LDS between the matrix core's lane order and whole rows.
#pragma once
#include <hip/hip_runtime.h>

namespace nat {

// A result of the core holds, in lane l of accumulator i, elements 16 i + 4 (l / 16) .. + 3 of row l % 16: an instruction that stores it writes half a
// 128-byte line of 16 rows.  Through LDS, 16 rows x 64 elements at a time, an instruction stores 256 bytes of four rows: lane l of read j holds elements
// 4 (l % 16) .. + 3 of row 4 j + l / 16.  Chunks of 16 bytes are permuted within a row (chunk c of row r at c ^ r), so that neither side has bank conflicts.
constexpr int kStageFloats = 16 * 64;     // per wavefront
__host__ __device__ inline int stage_write_at(int lane, int i) {     // floats; i = 0..3
  const int row = lane & 15;
  return row * 64 + (((4 * i + (lane >> 4)) ^ row) << 2);
}
__host__ __device__ inline int stage_read_row(int lane, int j) { return 4 * j + (lane >> 4); }     // j = 0..3
__host__ __device__ inline int stage_read_column(int lane) { return 4 * (lane & 15); }
__host__ __device__ inline int stage_read_at(int lane, int j) {
  const int row = stage_read_row(lane, j);
  return row * 64 + (((lane & 15) ^ row) << 2);
}

}  // namespace nat
