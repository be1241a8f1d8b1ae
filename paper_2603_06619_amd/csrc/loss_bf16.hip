// bf16 path of nat_loss_fwd_bwd / nat_loss_fwd_bwd_kl / nat_logp_fwd for gfx950: LM-head
// projection, full-vocabulary log-softmax, clipped GRPO surrogate with Horvitz-Thompson
// weights (Eq. 1, 3, 5, 6/9), optional KL term (Eq. 4) and entropy, and the gradients dH, dW
// (App. A) on the kept tokens.  The forward pass alone runs the first two steps below and
// keeps only the sums.
//
// Tokens are processed in chunks of at most `cap` rows (16384 or 32768 with the recommended workspace); the
// forward sweep and the dH contraction of a chunk run in sub-chunks of 8192 rows.  Per chunk:
//   reference     ref_k = h_k . W[ids_k]: the target logit, used only as the exponent shift;
//   logits GEMM   Z^T tile = W_tile . H^T on bf16 MFMA with fp32 accumulators; the epilogue never
//                 stores Z: it stores E = exp(z - ref_k) as bf16, ONCE, rows = token (soft-max
//                 numerators: bf16 keeps their relative precision), per (token, 128-row vocabulary
//                 granule) partial sums of E, and the exact target logit;
//   token stats   S_k = sum of the partials (fixed order), lse = ref + log S, log-prob, ratio,
//                 clipped surrogate, c_k = dLoss/dlogp_k, beta_k = -c_k / S_k;
//                 dz_kv = beta_k E_kv, except the target entry c_k (1 - p_target), which is
//                 patched into E as -S_k (1 - p_target), computed in fp32 before rounding;
//   dH GEMM       dH = diag(beta) (E . W)            (contraction over the vocabulary);
//   dW GEMM       dW (+)= E^T . (diag(beta) H_chunk) (contraction over the chunk's tokens, fp32,
//                 one owner per output tile, chunks in order: deterministic).  Its A operand is
//                 the same copy of E, which is stored along this contraction's k axis: the tile
//                 is gathered in 2 KiB pieces and fragments are formed by the transposing LDS
//                 read (ds_read_b64_tr_b16).
// The shift by the target logit needs log(p_max / p_target) < 70 for every kept token (E is
// clamped there; the token statistics count the tokens this may have touched); a token the current
// policy gives less than e^-70 of its mode's probability does not occur for rollouts drawn from a
// behaviour policy inside the clip range.
// All three contractions run through one "NT" kernel (both operands contiguous along the
// contraction axis; the k-major A operand of dW is the one exception described above).  Every
// operand is kept in a blocked layout in the workspace: blocks of 256 rows x 32 k-elements (16 KiB,
// contiguous), ordered k-fastest inside a 256-row tile, so a workgroup streams one contiguous
// region per operand instead of 256 strided rows.  W and H_chunk are repacked (plain and
// transposed); the soft-max numerators are produced directly in that layout.  Short batches do not
// repack W (direct_tokens): the logits contraction reads its rows, the dH contraction, turned round to
// dH^T = W^T E^T, reads them as a k-major operand.
#include "nat_internal.h"
#include "grpo_scalar.hip.h"

#include <type_traits>

namespace nat {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
// The soft-max numerators are written once and read back only by the two backward contractions,
// long after they have left the L2: non-temporal stores (1 % on the logits kernel).
#define NAT_E_STORE(ptr, val) __builtin_nontemporal_store((val), (ptr))

constexpr int kBM = 256, kBN = 256, kBK = 32;     // block tile: 4 wavefronts of 128 x 128 or 8 of 128 x 64
constexpr int kStages = 4;                        // LDS ring of k-slices (4 x 32 KiB)
constexpr int kGranule = 128;                     // vocabulary rows per soft-max partial
constexpr int kTileBytes = kBM * kBK * 2;         // 16 KiB per operand per stage
// Wavefronts per workgroup of each contraction (4: one per SIMD, 128 x 128 each, 256 accumulator
// registers; 8: two per SIMD, 128 x 64 each: row-major operands only).  Measured on the Qwen3-8B
// head with the row-major kernel: dH 2 % slower with 8, the logits contraction unchanged; the k-major
// dW loop is written for 4.
// Tile rows per group of the block -> tile map, per contraction (measured: 4 is 1-2 % faster than 8
// for the two backward contractions, 2 and 6 are slower, 16 is 8 % slower).
#ifndef NAT_GROUP_LOGITS
#define NAT_GROUP_LOGITS 8
#endif
#ifndef NAT_GROUP_DHIDDEN
#define NAT_GROUP_DHIDDEN 4
#endif
#ifndef NAT_GROUP_DWEIGHT
#define NAT_GROUP_DWEIGHT 4
#endif
#ifndef NAT_WAVES_LOGITS
#define NAT_WAVES_LOGITS 4
#endif
#ifndef NAT_WAVES_DHIDDEN
#define NAT_WAVES_DHIDDEN 4
#endif
#ifndef NAT_WAVES_DWEIGHT
#define NAT_WAVES_DWEIGHT 4
#endif
constexpr int kMaxChunk = 32768;                  // most token rows per chunk (see recommended_cap)
constexpr int kNumCU = 256;                       // compute units (one workgroup of these kernels each)
constexpr int kMinSlicesPerRange = 32;            // least k-slices per range of a cut contraction axis, on average
#ifndef NAT_SUBCHUNK
#define NAT_SUBCHUNK 8192
#endif
constexpr int kSubChunk = NAT_SUBCHUNK;           // smallest token count per launch of the logits and dH contractions

// two floats -> two bf16 in one 32-bit word (lo in bits 0..15): one packed conversion instruction
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float x) {
  const __bf16 b = (__bf16)x;
  return __builtin_bit_cast(uint16_t, b);
}

// ------------------------------------------------------------ blocked layout ----
constexpr int kBlkElems = 256 * 32;               // one block: 256 rows x 32 k-elements

// element (row, k) of an operand with kb = K/32 k-slices.  Inside a row of a block the four
// 16-byte chunks are stored permuted (chunk index XOR bits 2..3 of the row): a block is then a
// byte-for-byte image of the bank-conflict-free LDS tile, and the direct-to-LDS copy reads it
// linearly, 16 bytes per lane.
__host__ __device__ __forceinline__ int64_t blk_off(int row, int k, int kb) {
  return ((int64_t)(row >> 8) * kb + (k >> 5)) * kBlkElems + ((row & 255) << 5) +
         (((((k & 31) >> 3) ^ ((row >> 2) & 3))) << 3) + (k & 7);
}

// Repack a row-major matrix in [R, C] (leading dimension ld_in) into the blocked layout,
// in one or both orientations, zero-filling the padding:
//   out_rk: rows = r (padded to Rp, multiple of 256), k = c (C must be a multiple of 32);
//   out_cr: rows = c (padded to Cp, multiple of 256), k = r (padded to Rp).
//   row_scale: optional [R] factor applied to row r of the input in out_cr (fp32 product, rounded once).
//   kb_cr: k-slices of the operand out_cr belongs to (Rp / 32 when the input is the whole operand;
//          more when the rows are a range of a longer contraction axis: out_cr then points at the
//          range's first k-slice).
// One workgroup repacks a 64 x 64 tile, 16 bytes (8 elements) per access on the global side: rows of
// the input and 16-byte chunks of the blocked layout are both 16-byte aligned (C and ld_in multiples
// of 8, pointers 16-byte aligned: checked at the entry points).
__global__ void __launch_bounds__(256)
pack_blocked_kernel(const uint16_t* __restrict__ in, int64_t ld_in, int R, int C, int Rp, int Cp,
                    uint16_t* __restrict__ out_rk, uint16_t* __restrict__ out_cr, int kb_cr,
                    const float* __restrict__ row_scale) {
  union Chunk { uint4 q; uint16_t e[8]; };
  __shared__ __attribute__((aligned(16))) uint16_t tile[64][72];     // 144-byte rows: 16-byte aligned chunks
  const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
  const int cc = threadIdx.x & 7, jr = threadIdx.x >> 3;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int j = jr + 32 * i;
    const int r = r0 + j, c = c0 + 8 * cc;
    Chunk x;
    x.q = make_uint4(0u, 0u, 0u, 0u);
    if (r < R && c < C) x.q = *reinterpret_cast<const uint4*>(in + (int64_t)r * ld_in + c);
    if (out_rk && c < C) *reinterpret_cast<uint4*>(out_rk + blk_off(r, c, C >> 5)) = x.q;
    if (row_scale && r < R) {
      const float f = row_scale[r];
#pragma unroll
      for (int e = 0; e < 8; ++e) x.e[e] = f32_to_bf16_bits(__builtin_bit_cast(float, (uint32_t)x.e[e] << 16) * f);
    }
    *reinterpret_cast<uint4*>(&tile[j][8 * cc]) = x.q;
  }
  if (!out_cr) return;
  __syncthreads();
  // transposed: row c of the output holds k = r; the tile's 64 r are two k-slices, each a contiguous
  // 4 KiB (64 rows x 64 bytes) of the blocked operand; four neighbouring threads write one 64-byte row
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = threadIdx.x + 256 * i;
    const int cj = (q >> 2) & 63, rbase = (q >> 8) * 32 + (q & 3) * 8;
    Chunk y;
#pragma unroll
    for (int e = 0; e < 8; ++e) y.e[e] = tile[rbase + e][cj];
    *reinterpret_cast<uint4*>(out_cr + blk_off(c0 + cj, r0 + rbase, kb_cr)) = y.q;
  }
}

// ------------------------------------------------------------------- GEMM ----
struct GemmArgs {
  const uint16_t* A;          // [tiles_m * 256, K] in the blocked layout
  const uint16_t* B;          // [tiles_n * 256, K] in the blocked layout
  int K;                      // multiple of kBK
  int tiles_m, tiles_n;
  int group_m;                // tile rows walked together (see tile_of_block)
  int kb_a_src;               // k-major A only (see TileLoaderKMajor): k-slices of the source operand
  int kb_b;                   // k-slices of the B operand as it is stored (>= K / kBK)
  // k_splits > 1: the contraction axis of the last tail_tiles tiles in launch order (all of them when there are fewer
  // than compute units) is cut into k_splits ranges of kt_per_split k-slices, one workgroup per (tile, range); the
  // epilogue is told which slab its raw sums go to (position among the cut tiles * k_splits + range)
  int k_splits, kt_per_split, tail_tiles;
  int src_rows, src_cols;     // A read from a row-major matrix (TileLoaderRows, TileLoaderKMajorRows): its extent
};

// Block id -> output tile.  Blocks are dealt round-robin to the 8 XCDs, so ids
// congruent mod 8 share an L2: give each XCD a contiguous range of tiles, walked
// in groups of `group_m` tile-rows so that concurrently resident blocks reuse A and B tiles.
__device__ __forceinline__ void tile_of_block(const GemmArgs& g, int pid, int& tm, int& tn) {
  const int total = g.tiles_m * g.tiles_n;
  int logical = pid;
  const int per_xcd = total / 8;
  if (pid < per_xcd * 8) logical = (pid & 7) * per_xcd + (pid >> 3);
  const int kGroupM = g.group_m;
  const int group_sz = kGroupM * g.tiles_n;
  const int group = logical / group_sz;
  const int first_m = group * kGroupM;
  const int rows = g.tiles_m - first_m < kGroupM ? g.tiles_m - first_m : kGroupM;
  const int in_group = logical - group * group_sz;
  tm = first_m + in_group % rows;
  tn = in_group / rows;
}

// Byte offset of 16-byte chunk c (0..3) of row r in a [256][32] bf16 LDS tile (64-byte rows).
// A ds_read_b128 is served 16 lanes at a time over 64 banks; 16 consecutive rows at one
// chunk index would fall on 4 bank groups, so the chunk is XOR-ed with bits 2..3 of the row.
__device__ __forceinline__ int lds_chunk_off(int r, int c) { return r * (kBK * 2) + ((c ^ ((r >> 2) & 3)) << 4); }

// Global -> LDS copy of one [256][32] bf16 operand block (16 KiB, contiguous in memory)
// without staging registers: the NW wavefronts issue 16 direct-to-LDS loads of 16 bytes per
// lane between them.  One instruction copies 1 KiB (16 tile rows) linearly: the hardware
// places lane l at byte 16*l of that KiB, and the block in memory already has the LDS tile's
// chunk order.
template <int NW>
struct TileLoader {
  static constexpr int kLoads = kTileBytes / 1024 / NW;     // per wavefront
  const uint16_t* src;           // this lane's chunk in k-slice 0 of load 0

  // A wavefront copies kLoads consecutive KiB of the block (16 * kLoads rows): the loads of one
  // slice differ only in the instruction's immediate offset, which the hardware adds to both the
  // global and the LDS address, so one address and one LDS base serve all of them.
  __device__ __forceinline__ void init(const uint16_t* base, int tile, int kb, int wave, int lane) {
    src = base + (int64_t)tile * kb * kBlkElems + wave * (kLoads * 16 * kBK) + lane * 8;
  }
  __device__ __forceinline__ void start_at(int kt0) { src += (int64_t)kt0 * kBlkElems; }   // slice 0 := slice kt0
  // load kIdx = 0 .. kLoads - 1 of this wavefront's share
  template <int kIdx>
  __device__ __forceinline__ void issue_one(char* lds_tile, int kt, int wave) const {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (int64_t)kt * kBlkElems),
                                     (__attribute__((address_space(3))) void*)(lds_tile + wave * (kLoads * 1024)), 16,
                                     kIdx * 1024, 0);
  }
  __device__ __forceinline__ void issue(char* lds_tile, int kt, int wave) const {
    const uint16_t* p = src + (int64_t)kt * kBlkElems;
    char* dst = lds_tile + wave * (kLoads * 1024);
    static_assert(kLoads == 4 || kLoads == 2, "immediate offsets below are written out");
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                     (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                     (__attribute__((address_space(3))) void*)dst, 16, 1024, 0);
    if (kLoads == 4) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                       (__attribute__((address_space(3))) void*)dst, 16, 2048, 0);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                       (__attribute__((address_space(3))) void*)dst, 16, 3072, 0);
    }
  }
};

// The first 128 rows of a [256][32] operand block: 8 KiB of each slice, two loads for each of 4 wavefronts.
struct HalfTileLoader {
  static constexpr int kLoads = 2;
  const uint16_t* src;
  __device__ __forceinline__ void init(const uint16_t* base, int tile, int kb, int wave, int lane) {
    src = base + (int64_t)tile * kb * kBlkElems + wave * 1024 + lane * 8;
  }
  __device__ __forceinline__ void start_at(int kt0) { src += (int64_t)kt0 * kBlkElems; }
  template <int kIdx>
  __device__ __forceinline__ void issue_one(char* lds_tile, int kt, int wave) const {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (int64_t)kt * kBlkElems),
                                     (__attribute__((address_space(3))) void*)(lds_tile + wave * 2048), 16, kIdx * 1024, 0);
  }
  __device__ __forceinline__ void issue(char* lds_tile, int kt, int wave) const {
    issue_one<0>(lds_tile, kt, wave);
    issue_one<1>(lds_tile, kt, wave);
  }
};

// The same copy for an A operand that is only stored with its rows along THIS contraction's k axis
// (the soft-max numerators: rows = token, k = vocabulary, read by the dW contraction whose k axis is
// the token).  A [256 rows][32 k] tile of the contraction is then eight pieces of the source, one per
// 32-row block of the tile: rows (kt % 8) * 32 .. + 31 of the source block (token tile kt / 8, k-slice
// 8 * tile + piece), 2 KiB contiguous each.  The LDS tile holds the pieces one after another, i.e.
// [row block][k][row within block], and fragments come out of it through the transposing LDS read.
template <int NW>
struct TileLoaderKMajor {
  static constexpr int kLoads = kTileBytes / 1024 / NW;     // per wavefront (4 with 4 wavefronts)
  static constexpr int kPieces = kLoads / 2;                // 2 KiB pieces per wavefront
  const uint16_t* src;           // this lane's 16 bytes of the wavefront's first piece, token tile 0, rows 0..15
  int64_t tile_stride;           // elements between consecutive token tiles of the source

  __device__ __forceinline__ void init(const uint16_t* base, int tile, int kb_src, int wave, int lane) {
    src = base + (int64_t)(8 * tile + wave * kPieces) * kBlkElems + lane * 8;
    tile_stride = (int64_t)kb_src * kBlkElems;
  }
  __device__ __forceinline__ void start_at(int kt0) { src += (int64_t)(kt0 >> 3) * tile_stride; }   // kt0 % 8 == 0
  // load kIdx = 0 .. kLoads - 1 of this wavefront's share (1 KiB: half a piece)
  template <int kIdx>
  __device__ __forceinline__ void issue_one(char* lds_tile, int kt, int wave) const {
    constexpr int piece = kIdx >> 1;
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(src + (int64_t)(kt >> 3) * tile_stride + (kt & 7) * 1024 + (int64_t)piece * kBlkElems),
        (__attribute__((address_space(3))) void*)(lds_tile + (wave * kPieces + piece) * 2048), 16, (kIdx & 1) * 1024, 0);
  }
};

// The same two tiles straight from a row-major matrix (the caller's W), for batches too small to pay for repacking it:
// one instruction reads 64 bytes of 16 rows, each lane from where its place of the LDS tile wants it (16-byte chunk
// p of a tile row holds chunk p XOR bits 2..3 of the row).  Rows past the end read the last row: as vocabulary rows
// of the logits tile they are masked by the epilogue, as k of the dH contraction they meet numerators that are 0.
template <int NW>
struct TileLoaderRows {          // [256 rows][32 k]: rows of the matrix, k its columns
  static constexpr int kLoads = kTileBytes / 1024 / NW;
  const uint16_t* src[kLoads];   // this lane's chunk in k-slice 0 of each load
  __device__ __forceinline__ void init(const uint16_t* W, int tile, int rows, int ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int r = (wave * kLoads + i) * 16 + (lane >> 2), row = tile * kBM + r;
      src[i] = W + (int64_t)(row < rows ? row : rows - 1) * ld + (((lane & 3) ^ ((r >> 2) & 3)) << 3);
    }
  }
  __device__ __forceinline__ void start_at(int kt0) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) src[i] += kt0 * kBK;
  }
  template <int kIdx>
  __device__ __forceinline__ void issue_one(char* lds_tile, int kt, int wave) const {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[kIdx] + kt * kBK),
                                     (__attribute__((address_space(3))) void*)(lds_tile + (wave * kLoads + kIdx) * 1024), 16, 0, 0);
  }
  __device__ __forceinline__ void issue(char* lds_tile, int kt, int wave) const {
    static_assert(kLoads == 4, "written out for 4 wavefronts");
    issue_one<0>(lds_tile, kt, wave);
    issue_one<1>(lds_tile, kt, wave);
    issue_one<2>(lds_tile, kt, wave);
    issue_one<3>(lds_tile, kt, wave);
  }
};

template <int NW>
struct TileLoaderKMajorRows {    // [256 rows][32 k] with k the rows of the matrix: pieces of 32 k x 32 rows, as TileLoaderKMajor
  static constexpr int kLoads = kTileBytes / 1024 / NW;
  const uint16_t* src;           // this lane's chunk of row 0 of the wavefront's first piece
  int piece_step;                // elements from the wavefront's first piece to its second
  int k_rows, ld, k_lane, kt_first;
  __device__ __forceinline__ void init(const uint16_t* W, int tile, int rows, int cols, int wave, int lane) {
    static_assert(kLoads == 4, "two pieces per wavefront");
    const int c0 = tile * kBM + 64 * wave, c1 = c0 + 32;         // columns past the end (a multiple of 64 is valid): any valid ones
    const int s0 = c0 < cols ? c0 : cols - 32, s1 = c1 < cols ? c1 : cols - 32;
    k_lane = lane >> 2;
    src = W + s0 + (((lane & 3) ^ ((lane >> 4) & 3)) << 3);
    piece_step = s1 - s0;
    k_rows = rows;
    ld = cols;
    kt_first = 0;
  }
  __device__ __forceinline__ void start_at(int kt0) { kt_first = kt0; }
  template <int kIdx>
  __device__ __forceinline__ void issue_one(char* lds_tile, int kt, int wave) const {
    constexpr int piece = kIdx >> 1, half = kIdx & 1;
    const int k = (kt_first + kt) * kBK + half * 16 + k_lane;
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(src + (int64_t)(k < k_rows ? k : k_rows - 1) * ld + piece * piece_step),
        (__attribute__((address_space(3))) void*)(lds_tile + (wave * 4 + kIdx) * 1024), 16, 0, 0);
  }
};

// Per-lane byte offsets, inside a [k = 32][32 rows] piece, of the two transposing reads (q = 0, 1)
// that make one A fragment of k-substep 0.  The transposing read works on groups of 16 lanes: lane
// i of a group supplies the address of 4 consecutive 16-bit elements and receives element i % 4 of
// the lanes i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12.  With lane i pointing at k = K0 + i / 4 and rows
// 16 g + 4 (i % 4) .. + 3, lane i ends up with row 16 g + i and k = K0 .. K0 + 3: the MFMA's A layout
// (row = lane % 32, 8 consecutive k from 8 * (lane / 32)) after two reads, K0 = 8 * (lane / 32) + 4 q.
// The 16-byte chunks of a source row are stored XOR-ed with bits 2..3 of the row (see blk_off); for
// these k values that is 2 * (lane / 32) + q.  The 32 lanes of a half-wavefront then cover all 64
// LDS banks exactly once.
struct KMajorFragOffsets {
  int off[2];
  __device__ __forceinline__ void init(int lane) {
    const int i = lane & 15, g = (lane >> 4) & 1, lhi = lane >> 5, a = i & 3;
#pragma unroll
    for (int q = 0; q < 2; ++q)
      off[q] = (8 * lhi + 4 * q + (i >> 2)) * 64 + ((((2 * g + (a >> 1)) ^ (2 * lhi + q)) & 3) << 4) + (a & 1) * 8;
  }
};

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// One k-substep of the row-major loop, instruction slot by slot (the compiler may not move anything
// across a slot's end): slot m holds MFMA m on the fragments (au, bu); behind each of the first 4 + NB
// MFMAs one fragment read of k-substep ks_load from (a_s, b_s) into (al, bl); the remaining MFMAs carry
// the direct-to-LDS loads of this wavefront's share of slice k into lds_dst, evenly spaced (mixing them
// with the fragment reads measured slower).
template <int NW, int NB, int M = 0, class Loader>
__device__ __forceinline__ void substep_slots(f32x16 (&acc)[4][NB], const bf16x8 (&au)[4], const bf16x8 (&bu)[NB],
                                              bf16x8 (&al)[4], bf16x8 (&bl)[NB], const char* a_s, const char* b_s,
                                              int a_row0, int b_row0, int l32, int lhi, int ks_load,
                                              const Loader& ld, char* lds_dst, int k, int wave) {
  constexpr int kLoadFirst = 4 + NB, kLoadEvery = (4 * NB - kLoadFirst) / TileLoader<NW>::kLoads;
  static_assert(kLoadEvery >= 1, "every load needs a slot");
  if constexpr (M < 4 * NB) {
    constexpr int i = M / NB, j = M % NB;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(au[i], bu[j], acc[i][j], 0, 0, 0);
    if constexpr (M < 4) al[M] = *(const bf16x8*)(a_s + lds_chunk_off(a_row0 + M * 32 + l32, ks_load * 2 + lhi));
    else if constexpr (M < 4 + NB) bl[M - 4] = *(const bf16x8*)(b_s + lds_chunk_off(b_row0 + (M - 4) * 32 + l32, ks_load * 2 + lhi));
    if constexpr (M >= kLoadFirst && (M - kLoadFirst) % kLoadEvery == 0 && (M - kLoadFirst) / kLoadEvery < TileLoader<NW>::kLoads)
      ld.template issue_one<(M - kLoadFirst) / kLoadEvery>(lds_dst, k, wave);
    __builtin_amdgcn_sched_barrier(0);
    substep_slots<NW, NB, M + 1>(acc, au, bu, al, bl, a_s, b_s, a_row0, b_row0, l32, lhi, ks_load, ld, lds_dst, k, wave);
  }
}

// The same for the loop that reads its A tiles from rows (TileLoaderRows), which refills two slices' A tiles at once:
// kRefill 0: the loads of B, one every second MFMA as above; 1: eight loads of A, the two halves of each 128-byte
// line one right after the other; 2: none.  NB = 2 (a tile of 128 columns): eight MFMAs, the loads behind the last two.
template <int NB, int kRefill, int M = 0, class LoaderB>
__device__ __forceinline__ void substep_slots_rows(f32x16 (&acc)[4][NB], const bf16x8 (&au)[4], const bf16x8 (&bu)[NB],
                                                   bf16x8 (&al)[4], bf16x8 (&bl)[NB], const char* a_s, const char* b_s,
                                                   int a_row0, int b_row0, int l32, int lhi, int ks_load,
                                                   const TileLoaderRows<4>& la, const LoaderB& lb, char* lds0, char* lds1,
                                                   int k0, int k1, int wave) {
  constexpr int kFirst = 4 + NB, kSlots = 4 * NB - kFirst;     // slots behind the fragment reads: 8, or 2
  if constexpr (M < 4 * NB) {
    constexpr int i = M / NB, j = M % NB, q = M - kFirst;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(au[i], bu[j], acc[i][j], 0, 0, 0);
    if constexpr (M < 4) al[M] = *(const bf16x8*)(a_s + lds_chunk_off(a_row0 + M * 32 + l32, ks_load * 2 + lhi));
    else if constexpr (M < kFirst) bl[M - 4] = *(const bf16x8*)(b_s + lds_chunk_off(b_row0 + (M - 4) * 32 + l32, ks_load * 2 + lhi));
    else if constexpr (kRefill == 0) {
      if constexpr (q * LoaderB::kLoads % kSlots == 0) lb.template issue_one<q * LoaderB::kLoads / kSlots>(lds0, k0, wave);
    } else if constexpr (kRefill == 1) {
      if constexpr (NB == 4) {
        if constexpr ((q & 1) == 0) la.template issue_one<q / 2>(lds0, k0, wave);
        else la.template issue_one<q / 2>(lds1, k1, wave);
      } else {
        la.template issue_one<2 * q>(lds0, k0, wave);
        la.template issue_one<2 * q>(lds1, k1, wave);
        la.template issue_one<2 * q + 1>(lds0, k0, wave);
        la.template issue_one<2 * q + 1>(lds1, k1, wave);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    substep_slots_rows<NB, kRefill, M + 1>(acc, au, bu, al, bl, a_s, b_s, a_row0, b_row0, l32, lhi, ks_load, la, lb, lds0, lds1, k0, k1, wave);
  }
}

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

// The transposing read as inline assembly (byte offset as an immediate): invisible to the compiler's wait-count
// pass, which would otherwise put a wait for all direct-to-LDS loads in front of it; the caller waits
// (lgkmcnt) before it uses what was read.
__device__ __forceinline__ s16x4 lds_read_tr16_b64(uint32_t addr, int off) {
  s16x4 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(off) : "memory");
  return v;
}

// One k-substep of the k-major loop with 4 wavefronts of 128 x 128, slot by slot (see substep_slots): MFMA m on
// (au, bu); behind the first 8 MFMAs one transposing read each (halves q = m % 2 of A block m / 2, from the
// piece bases a_rd[q]) and behind the first 4 also one 16-byte read of B; behind MFMAs 8, 10, 12, 14 one
// direct-to-LDS load of the refill (the A tile's when kRefillA, else the B tile's).  NB = 2 (a tile of 128 columns):
// eight MFMAs, two transposing reads behind each of the first four, the two reads of B, then the loads.
template <int NB, bool kRefillA, int M = 0, class LoaderA, class LoaderB>
__device__ __forceinline__ void substep_slots_kmajor4(f32x16 (&acc)[4][NB], const bf16x8 (&au)[4], const bf16x8 (&bu)[NB],
                                                      s16x4 (&al)[8], bf16x8 (&bl)[NB], const uint32_t (&a_rd)[2], const char* b_rd,
                                                      const LoaderA& la, const LoaderB& lb, char* lds_dst,
                                                      int k, int wave) {
  if constexpr (M < 4 * NB) {
    constexpr int i = M / NB, j = M % NB;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(au[i], bu[j], acc[i][j], 0, 0, 0);
    if constexpr (NB == 4) {
      if constexpr (M < 4) bl[M] = *(const bf16x8*)(b_rd + M * 2048);
      if constexpr (M < 8) al[M] = lds_read_tr16_b64(a_rd[M & 1], (M / 2) * 2048);
      if constexpr (M >= 8 && (M & 1) == 0) {
        if constexpr (kRefillA) la.template issue_one<(M - 8) / 2>(lds_dst, k, wave);
        else lb.template issue_one<(M - 8) / 2>(lds_dst, k, wave);
      }
    } else if constexpr (M < 4) {
      al[2 * M] = lds_read_tr16_b64(a_rd[0], M * 2048);
      al[2 * M + 1] = lds_read_tr16_b64(a_rd[1], M * 2048);
    } else if constexpr (M < 6) {
      bl[M - 4] = *(const bf16x8*)(b_rd + (M - 4) * 2048);
    } else if constexpr (kRefillA) {
      la.template issue_one<2 * (M - 6)>(lds_dst, k, wave);
      la.template issue_one<2 * (M - 6) + 1>(lds_dst, k, wave);
    } else {
      lb.template issue_one<M - 6>(lds_dst, k, wave);
    }
    __builtin_amdgcn_sched_barrier(0);
    substep_slots_kmajor4<NB, kRefillA, M + 1>(acc, au, bu, al, bl, a_rd, b_rd, la, lb, lds_dst, k, wave);
  }
}

// fragments of k-substep ks: four 32-row blocks of A from row a_row0, NB 32-row blocks of B from b_row0
template <int NB>
__device__ __forceinline__ void load_frags(const char* a_s, const char* b_s, int a_row0, int b_row0, int l32, int lhi,
                                           int ks, bf16x8 (&af)[4], bf16x8 (&bfr)[NB]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) af[i] = *(const bf16x8*)(a_s + lds_chunk_off(a_row0 + i * 32 + l32, ks * 2 + lhi));
#pragma unroll
  for (int j = 0; j < NB; ++j) bfr[j] = *(const bf16x8*)(b_s + lds_chunk_off(b_row0 + j * 32 + l32, ks * 2 + lhi));
}

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }

// NW wavefronts in a 2 x (NW/2) grid over the 256 x 256 tile: wavefront (wm, wn) owns rows
// wm*128.. and columns wn*(NB*32).. with NB = 16/NW (4 wavefronts: 128 columns, 8: 64 columns).
// acc[mb][nb] element r of lane l is C[row0 + mb*32 + 8*(r/4) + 4*(l/32) + r%4][col0 + nb*32 + l%32]
// kA: how the A operand is stored.  k-major: along this contraction's k axis (g.kb_a_src is then the number of
// k-slices of that source); rows: a row-major matrix of g.src_rows x g.src_cols, read as it is.
enum class ASource { kBlocked, kKMajorBlocked, kRows, kKMajorRows };
// one LDS object (with a second one the compiler's wait-count pass orders every fragment read behind all
// direct-to-LDS loads in flight): the ring, and behind it the words the epilogue parks across the k-loop
template <int kStashWords>
struct GemmShared {
  char ring[kStages][2][kTileBytes];
  int stash[kStashWords > 0 ? kStashWords : 1];
};

// One tile.  NB: 32-column blocks per wavefront, 16 / NW; or 2 with 4 wavefronts: a tile of which only the first 128
// columns are computed.
template <class Epilogue, int NW, ASource kA, int NB, class Shared>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, const Epilogue& epi, Shared& sm, int tm, int tn, int range, int slab) {
  constexpr bool AT = kA == ASource::kKMajorBlocked || kA == ASource::kKMajorRows;
  constexpr bool kHalf = NB * NW < 16;
  constexpr int kLoadsA = kTileBytes / 1024 / NW, kLoadsB = kHalf ? HalfTileLoader::kLoads : kLoadsA;   // per wavefront and slice
  constexpr int kLoadsPerWave = kLoadsA + kLoadsB;
  auto& lds = sm.ring;
  int* pre_stash = sm.stash;
  const int m0 = tm * kBM, n0 = tn * kBN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / (NW / 2), wn = wave % (NW / 2);
  const int a_row0 = wm * 128, b_row0 = wn * (NB * 32);
  const int l32 = lane & 31, lhi = lane >> 5;

  f32x16 acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // per-column scalars the epilogue needs (token id, exponent shift): fetched into LDS now, read after the k-loop
  typename Epilogue::template Pre<NB> pre;
  epi.template prefetch<NB>(pre_stash, NW * 64, n0 + b_row0, lane, wave);

  using Blocked = typename std::conditional<AT, TileLoaderKMajor<NW>, TileLoader<NW>>::type;
  using Rows = typename std::conditional<AT, TileLoaderKMajorRows<NW>, TileLoaderRows<NW>>::type;
  constexpr bool kDirect = kA == ASource::kRows || kA == ASource::kKMajorRows;
  typename std::conditional<kDirect, Rows, Blocked>::type la;
  typename std::conditional<kHalf, HalfTileLoader, TileLoader<NW>>::type lb;
  const int kt_all = g.K / kBK;
  if constexpr (kDirect) la.init(g.A, tm, g.src_rows, g.src_cols, wave, lane);
  else la.init(g.A, tm, AT ? g.kb_a_src : kt_all, wave, lane);
  lb.init(g.B, tn, g.kb_b, wave, lane);
  int kt_n = kt_all;                                           // k-slices this workgroup contracts over
  if (range >= 0) {
    const int kt0 = range * g.kt_per_split;                    // with a blocked k-major A a multiple of 8 (TileLoaderKMajor::start_at)
    kt_n = kt_all - kt0 < g.kt_per_split ? kt_all - kt0 : g.kt_per_split;
    la.start_at(kt0);
    lb.start_at(kt0);
  }

  if constexpr (AT) {
    // k-major A: the row-major pipeline below (refill in two halves), with 4 wavefronts of 128 x 128, every
    // instruction of the loop placed by hand (substep_slots_kmajor4), and the A fragments through the transposing
    // read issued as inline assembly.  (The compiler's builtin for that read carries no memory operand, so its
    // wait-count pass puts a wait for ALL direct-to-LDS loads in flight in front of every such read: vmcnt(0)
    // inside the k-loop, 20-30 % slower.  As inline assembly the read is invisible to that pass; the kernel
    // waits for it itself, lgkmcnt(0) before the next substep uses what was read.  An earlier variant kept the
    // builtin read and hid the loads instead, with 8 wavefronts and compiler-scheduled reads: 3.5 % slower.)
    static_assert(NW == 4, "the k-major loop is written for 4 wavefronts");
    KMajorFragOffsets fo;
    fo.init(lane);
    const int a_blk0 = a_row0 / 32;
#pragma unroll
    for (int st = 0; st < kStages; ++st) {
      const int k = st < kt_n ? st : kt_n - 1;
      la.template issue_one<0>(lds[st][0], k, wave);
      la.template issue_one<1>(lds[st][0], k, wave);
      la.template issue_one<2>(lds[st][0], k, wave);
      la.template issue_one<3>(lds[st][0], k, wave);
      if (st < kStages - 1) lb.issue(lds[st][1], k, wave);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((kStages - 1) * kLoadsA + (kStages - 2) * kLoadsB));   // slice 0 has landed
    __syncthreads();
    s16x4 ah[2][8];
    bf16x8 bfr[2][NB];
    auto a_bases = [&](int stage, int ks, uint32_t (&out)[2]) {
      const uint32_t piece0 = lds_addr(lds[stage][0] + a_blk0 * 2048 + ks * 1024);
      out[0] = piece0 + fo.off[0];
      out[1] = piece0 + fo.off[1];
    };
    auto join = [&](const s16x4 (&h)[8], bf16x8 (&out)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const s16x8 both = {h[2 * i][0], h[2 * i][1], h[2 * i][2], h[2 * i][3], h[2 * i + 1][0], h[2 * i + 1][1], h[2 * i + 1][2], h[2 * i + 1][3]};
        out[i] = __builtin_bit_cast(bf16x8, both);
      }
    };
    {
      uint32_t ar[2];
      a_bases(0, 0, ar);
#pragma unroll
      for (int m = 0; m < 8; ++m) ah[0][m] = lds_read_tr16_b64(ar[m & 1], (m / 2) * 2048);
#pragma unroll
      for (int j = 0; j < NB; ++j) bfr[0][j] = *(const bf16x8*)(lds[0][1] + lds_chunk_off(b_row0 + j * 32 + l32, lhi));
    }
    for (int kt = 0; kt < kt_n; ++kt) {
      const int cur = kt % kStages, nxt = (kt + 1) % kStages, last = (kt + kStages - 1) % kStages;
      int k1 = kt + kStages - 1;
      k1 = k1 < kt_n ? k1 : kt_n - 1;
      int k2 = kt + kStages;
      k2 = k2 < kt_n ? k2 : kt_n - 1;
      uint32_t ar[2];
      bf16x8 au[4];
      // first k-substep of slice kt: reads its second substep's fragments, refills the B tile of slice kt + 3
      a_bases(cur, 1, ar);
      __builtin_amdgcn_s_waitcnt(0xc07f);                      // lgkmcnt(0): the fragments read under the last substep
      join(ah[0], au);
      __builtin_amdgcn_sched_barrier(0);
      substep_slots_kmajor4<NB, false>(acc, au, bfr[0], ah[1], bfr[1], ar, lds[cur][1] + lds_chunk_off(b_row0 + l32, 2 + lhi),
                                   la, lb, lds[last][1], k1, wave);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm((kStages - 2) * kLoadsPerWave) & 0xf0ff);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      // second k-substep: reads the first fragments of slice kt + 1, refills the A tile of lds[cur] with slice kt + 4
      a_bases(nxt, 0, ar);
      join(ah[1], au);
      __builtin_amdgcn_sched_barrier(0);
      substep_slots_kmajor4<NB, true>(acc, au, bfr[1], ah[0], bfr[0], ar, lds[nxt][1] + lds_chunk_off(b_row0 + l32, lhi),
                                  la, lb, lds[cur][0], k2, wave);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // no direct-to-LDS load may outlive the block
    __syncthreads();
    epi(acc, pre, m0 + a_row0, n0 + b_row0, lane, wave, &lds[0][0][0], slab);
    return;
  } else if constexpr (kA == ASource::kRows) {
    // A from rows: the pipeline below, two slices per turn.  A slice is 64 bytes of a row, half a cache line; fetched
    // a slice apart, the halves cost the line twice on the way from the L2 (12289 tokens at H = 4096: 11.92 ms, 11.55 as
    // below, 11.48 from the repacked copy).  So both A tiles of slices
    // kt + 3 and kt + 4 are refilled under the second k-substep of an odd slice kt, half after half; B as below.  Issue order:
    // [even kt] B(kt + 3) [odd kt] B(kt + 3) A(kt + 3) A(kt + 4).  "Slice kt + 1 has landed" is then eight loads of A and two Bs
    // at the barrier of an even slice (B A A of slice kt - 1, B of kt), two Bs at that of an odd one (of kt - 1 and kt).  H is a multiple of 64: the number of slices is even.
    static_assert(NW == 4, "the loop is written for 4 wavefronts");
    auto clamp = [&](int k) { return k < kt_n ? k : kt_n - 1; };
    auto pair = [&](int st, int k) {
      la.template issue_one<0>(lds[st][0], clamp(k), wave);
      la.template issue_one<0>(lds[st + 1][0], clamp(k + 1), wave);
      la.template issue_one<1>(lds[st][0], clamp(k), wave);
      la.template issue_one<1>(lds[st + 1][0], clamp(k + 1), wave);
      la.template issue_one<2>(lds[st][0], clamp(k), wave);
      la.template issue_one<2>(lds[st + 1][0], clamp(k + 1), wave);
      la.template issue_one<3>(lds[st][0], clamp(k), wave);
      la.template issue_one<3>(lds[st + 1][0], clamp(k + 1), wave);
    };
    pair(0, 0);
    lb.issue(lds[0][1], 0, wave);
    lb.issue(lds[1][1], clamp(1), wave);
    pair(2, 2);
    lb.issue(lds[2][1], clamp(2), wave);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kLoadsA + 2 * kLoadsB));   // slice 0 has landed (younger: B1, A2, A3, B2)
    __syncthreads();
    bf16x8 af[2][4], bfr[2][NB];
    load_frags<NB>(lds[0][0], lds[0][1], a_row0, b_row0, l32, lhi, 0, af[0], bfr[0]);
    for (int kt = 0; kt < kt_n; kt += 2) {
      const int c0 = kt % kStages, c1 = c0 + 1, c2 = (c0 + 2) % kStages, c3 = c2 + 1;    // buffers of slices kt .. kt + 3
      __builtin_amdgcn_sched_barrier(0);
      substep_slots_rows<NB, 0>(acc, af[0], bfr[0], af[1], bfr[1], lds[c0][0], lds[c0][1], a_row0, b_row0, l32, lhi, 1, la, lb,
                            lds[c3][1], nullptr, clamp(kt + 3), 0, wave);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kLoadsA + 2 * kLoadsB) & 0xf0ff);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      substep_slots_rows<NB, 2>(acc, af[1], bfr[1], af[0], bfr[0], lds[c1][0], lds[c1][1], a_row0, b_row0, l32, lhi, 0, la, lb,
                            nullptr, nullptr, 0, 0, wave);
      substep_slots_rows<NB, 0>(acc, af[0], bfr[0], af[1], bfr[1], lds[c1][0], lds[c1][1], a_row0, b_row0, l32, lhi, 1, la, lb,
                            lds[c0][1], nullptr, clamp(kt + 4), 0, wave);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kLoadsB) & 0xf0ff);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      substep_slots_rows<NB, 1>(acc, af[1], bfr[1], af[0], bfr[0], lds[c2][0], lds[c2][1], a_row0, b_row0, l32, lhi, 0, la, lb,
                            lds[c0][0], lds[c1][0], clamp(kt + 4), clamp(kt + 5), wave);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // no direct-to-LDS load may outlive the block
    __syncthreads();
    epi.unstash(pre, pre_stash, NW * 64);
    epi(acc, pre, m0 + a_row0, n0 + b_row0, lane, wave, &lds[0][0][0], slab);
  } else {
  // Software pipeline over k-slices of 32.  Slice kt lives in lds[kt % 4]; three slices are
  // in flight while one is consumed, so a load has two to three iterations to land.  The barrier
  // sits between the two k-substeps of a slice; once it is passed, every wavefront has finished
  // reading slice kt and its buffer may be refilled.  The refill is issued in two halves so that
  // the loads of the NW wavefronts (which run in step) do not reach the CU's one address unit
  // all within a few hundred cycles: the A tile under the second substep of slice kt, the B tile
  // under the first substep of slice kt+1, each load one or two MFMAs after the previous one.
  // Loads complete in issue order (A0 B0 A1 B1 ...), hence "slice kt+1 has landed" at the barrier of
  // slice kt is vmcnt(2 * kLoadsPerWave): the halves of the two younger slices may be outstanding.
  // Slices past the end re-load the last one (into a buffer nobody reads again) to keep the body
  // branch-free and the count fixed.
  static_assert(!kHalf, "half tiles are read from rows");
  constexpr int kHalfLoads = kLoadsPerWave / 2;                // loads per wavefront and operand tile
#pragma unroll
  for (int st = 0; st < kStages; ++st) {
    const int k = st < kt_n ? st : kt_n - 1;
    la.issue(lds[st][0], k, wave);
    if (st < kStages - 1) lb.issue(lds[st][1], k, wave);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm((2 * kStages - 3) * kHalfLoads));   // slice 0 has landed
  __syncthreads();
  bf16x8 af[2][4], bfr[2][NB];
  load_frags<NB>(lds[0][0], lds[0][1], a_row0, b_row0, l32, lhi, 0, af[0], bfr[0]);

  for (int kt = 0; kt < kt_n; ++kt) {
    const int cur = kt % kStages, nxt = (kt + 1) % kStages, last = (kt + kStages - 1) % kStages;
    // first k-substep of slice kt; under its MFMAs: the second substep's fragments and the B half of
    // the refill of the buffer released at the previous barrier (slice kt + 3)
    int k1 = kt + kStages - 1;
    k1 = k1 < kt_n ? k1 : kt_n - 1;
    __builtin_amdgcn_sched_barrier(0);
    substep_slots<NW, NB>(acc, af[0], bfr[0], af[1], bfr[1], lds[cur][0], lds[cur][1], a_row0, b_row0, l32, lhi, 1,
                          lb, lds[last][1], k1, wave);
    // slice kt+1 has landed (this wavefront's share; the barrier covers the others) and this
    // wavefront has finished reading slice kt, whose buffer is refilled from here on
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((kStages - 2) * kLoadsPerWave) & 0xf0ff);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // second k-substep; under it: first fragments of slice kt+1 and the A half of the refill of lds[cur]
    int k2 = kt + kStages;
    k2 = k2 < kt_n ? k2 : kt_n - 1;
    substep_slots<NW, NB>(acc, af[1], bfr[1], af[0], bfr[0], lds[nxt][0], lds[nxt][1], a_row0, b_row0, l32, lhi, 0,
                          la, lds[cur][0], k2, wave);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // no direct-to-LDS load may outlive the block
  __syncthreads();

  epi.unstash(pre, pre_stash, NW * 64);
  epi(acc, pre, m0 + a_row0, n0 + b_row0, lane, wave, &lds[0][0][0], slab);
  }
}

template <class Epilogue, int NW, ASource kA = ASource::kBlocked>
__global__ void __launch_bounds__(NW * 64, 1)
gemm_nt_kernel(GemmArgs g, Epilogue epi) {
  __shared__ __attribute__((aligned(1024))) GemmShared<Epilogue::template stash_words<16 / NW>() * NW * 64> sm;
  int tm, tn;
  const int n_tiles = g.tiles_m * g.tiles_n;
  int pid = (int)blockIdx.x, range = -1, slab = -1;           // range of the contraction axis / slab (-1: whole axis)
  if (g.k_splits > 1 && pid >= n_tiles - g.tail_tiles) {
    const int r = pid - (n_tiles - g.tail_tiles);
    range = r / g.tail_tiles;
    const int pos = r - range * g.tail_tiles;
    pid = n_tiles - g.tail_tiles + pos;
    slab = pos * g.k_splits + range;
  }
  tile_of_block(g, pid, tm, tn);
  // Where W is read as it is the batch is short and the columns are its tokens: a last tile with at most 128 of them
  // computes only those (301 log-probs at the 0.6B head: logits 153 -> 132 us; 59 tokens at the 8B head: call 1155 -> 1067 us).
  if constexpr (kA == ASource::kRows || kA == ASource::kKMajorRows) {
    if (epi.n_valid - tn * kBN <= kBN / 2) {
      gemm_tile<Epilogue, NW, kA, 2>(g, epi, sm, tm, tn, range, slab);
      return;
    }
  }
  gemm_tile<Epilogue, NW, kA, 16 / NW>(g, epi, sm, tm, tn, range, slab);
}

// ------------------------------------------------------------- epilogues ----

// Logits tile: rows = vocabulary (A = W), columns = tokens of the chunk (B = H_chunk).
template <bool kEntropy, bool kStoreE = true>
struct LogitsEpilogue {
  int V, n_valid;                  // vocabulary size, valid tokens in the chunk
  int64_t ld_part;                 // leading dimension (tokens) of the partial sums
  int kb_z;                        // k-slices of Eb (Vp / 32)
  uint16_t* Eb;                    // blocked, rows = token, k = vocabulary: E = exp(z - ref), stored once
  float* s_part;                   // [Vp/128, ld_part] partial sums of E
  float* t_part;                   // [Vp/128, ld_part] partial sums of E (z - ref) (entropy), kEntropy only
  float* z_target;                 // [ld_part] exact target logits
  const int32_t* ids;              // target ids of the chunk's tokens
  const float* ref;                // [ld_part] exponent shift per token

  static constexpr int kStageRow = 272;        // bytes per token row of the LDS staging tile (128 bf16 + pad)

  // The per-column scalars the epilogue needs (token id, exponent shift) are fetched before the k-loop
  // straight into LDS (direct-to-LDS loads of 4 bytes per lane, from a clamped index; n_valid >= 1 in
  // every launch) and read back after it: they wait for nothing, hold no registers across the loop, and
  // are older than every operand load, so the loop's load counting is unchanged.  (Fetched into registers
  // they either cost a wait before the first operand loads, or live across the loop, where the compiler
  // spilled some of them and each reload in the epilogue waited for the stores in flight.)
  template <int NB> struct Pre { int y[NB]; float shift[NB]; };
  template <int NB> static constexpr int stash_words() { return 2 * NB; }
  template <int NB>
  __device__ __forceinline__ void prefetch(int* words, int n_threads, int k0, int lane, int wave) const {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int kk = k0 + nb * 32 + (lane & 31);
      const int kc = kk < n_valid ? kk : n_valid - 1;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(ids + kc),
                                       (__attribute__((address_space(3))) void*)(words + (2 * nb) * n_threads + wave * 64), 4, 0, 0);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(ref + kc),
                                       (__attribute__((address_space(3))) void*)(words + (2 * nb + 1) * n_threads + wave * 64), 4, 0, 0);
    }
  }
  template <int NB>
  __device__ __forceinline__ void unstash(Pre<NB>& pre, const int* words, int n_threads) const {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      pre.y[nb] = words[(2 * nb) * n_threads + threadIdx.x];
      pre.shift[nb] = __builtin_bit_cast(float, words[(2 * nb + 1) * n_threads + threadIdx.x]);
    }
  }

  template <int NB>
  __device__ __forceinline__ void operator()(f32x16 (&acc)[4][NB], const Pre<NB>& pre, int v0, int k0, int lane, int wave,
                                             char* lds, int) const {
    constexpr int kTok = NB * 32;                          // token columns of this wavefront
    const int l32 = lane & 31, lhi = lane >> 5;
    const int granule = v0 / kGranule;
    const bool all_rows_valid = v0 + kGranule <= V;
    constexpr float kLog2e = 1.44269504088896340736f, kLn2 = 0.69314718055994530942f;

    int y_of[NB];                  // target id of this lane's token per column block; -1: padding column, or
    float shift_of[NB];            // an id outside the vocabulary (matches no row)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const bool tok_valid = k0 + nb * 32 + l32 < n_valid;
      y_of[nb] = (tok_valid && pre.y[nb] >= 0 && pre.y[nb] < V) ? pre.y[nb] : -1;
      shift_of[nb] = tok_valid ? pre.shift[nb] : 0.f;
    }

    // exact target logit, if the target row lies in this granule and in this lane's half
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int yrel = y_of[nb] - v0;
      if (__any(yrel >= 0 && yrel < kGranule)) {
        if (yrel >= 0 && yrel < kGranule && ((yrel >> 2) & 1) == lhi) {
          float zt = 0.f;
#pragma unroll
          for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (yrel == mb * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3)) zt = acc[mb][nb][r];
          z_target[k0 + nb * 32 + l32] = zt;
        }
      }
    }

    // One pass over the accumulators, 32 token columns (all 128 vocabulary rows of the wavefront) at a
    // time: E = exp(min(z - shift, 70)) as 2^(min(z * log2(e) - shift * log2(e), 70 * log2(e))) (one fma,
    // one min and the hardware exponential per logit, sixteen at a time with independent temporaries),
    // its running sums, and at once the store of those columns, so that the stores of one group are in
    // flight under the exponentials of the next.  E is stored once, rows = token, k = vocabulary (the
    // dH contraction reads it as it is, the dW contraction through the transposing LDS read): a lane
    // holds 4 consecutive vocabulary entries of its token; the 32 x 128 group is staged through this
    // wavefront's own part of the LDS ring (free after the k-loop) and leaves as 16-byte stores, 1 KiB
    // (16 token rows of one 32-wide vocabulary slice) contiguous per instruction.  The staging area is
    // private to the wavefront and LDS operations of one wavefront execute in order, so no barrier is
    // needed between its writes, its reads and the next group's writes.
    char* stage = lds + wave * (32 * kStageRow);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const float nshift2 = -shift_of[nb] * kLog2e;
      float s2[2] = {0.f, 0.f}, t2[2] = {0.f, 0.f};        // two independent chains per sum
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        float x2[16], e[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x2[r] = fminf(fmaf(acc[mb][nb][r], kLog2e, nshift2), 70.f * kLog2e);
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = __builtin_amdgcn_exp2f(x2[r]);
        if (!all_rows_valid) {                             // only the last vocabulary tile pays for the row check
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (v0 + mb * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3) >= V) e[r] = 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          s2[r & 1] += e[r];
          if (kEntropy) t2[r & 1] = fmaf(e[r], x2[r], t2[r & 1]);
        }
        if (kStoreE) {
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            uint2 w;
            w.x = pack_bf16x2(e[4 * r4], e[4 * r4 + 1]);
            w.y = pack_bf16x2(e[4 * r4 + 2], e[4 * r4 + 3]);
            *(uint2*)(stage + l32 * kStageRow + (mb * 32 + 8 * r4 + 4 * lhi) * 2) = w;
          }
        }
      }
      if (kStoreE) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {                      // vocabulary slice i / 2, token rows (i % 2) * 16 .. + 15
          const int sl = i >> 1, tok = (i & 1) * 16 + (lane >> 2), ch = lane & 3;
          const uint4 val = *(const uint4*)(stage + tok * kStageRow + sl * 64 + ch * 16);
          NAT_E_STORE((u32x4v*)(Eb + blk_off(k0 + nb * 32 + tok, v0 + sl * 32 + ch * 8, kb_z)), __builtin_bit_cast(u32x4v, val));
        }
      }
      const int kk = k0 + nb * 32 + l32;                   // token column (always inside the padded chunk)
      float sum = s2[0] + s2[1];
      sum += __shfl_xor(sum, 32);
      if (lhi == 0) s_part[(int64_t)granule * ld_part + kk] = sum;
      if (kEntropy) {
        float t = (t2[0] + t2[1]) * kLn2;                  // back to natural-log units
        t += __shfl_xor(t, 32);
        if (lhi == 0) t_part[(int64_t)granule * ld_part + kk] = t;
      }
    }
  }
};

// dH tile: rows = tokens of the chunk (A = E), columns = hidden units (B = W^T); rows scaled by beta.
struct DHiddenEpilogue {
  int n_valid, H;
  uint16_t* dH;                    // rows of this chunk, [n_valid, H] bf16
  const float* beta;               // [n_valid]
  float* partial;                  // tiles whose contraction is cut into ranges: [slab][256][256] fp32 raw sums

  template <int NB> struct Pre {};
  template <int NB> static constexpr int stash_words() { return 0; }
  template <int NB> __device__ __forceinline__ void prefetch(int*, int, int, int, int) const {}
  template <int NB> __device__ __forceinline__ void unstash(Pre<NB>&, const int*, int) const {}
  template <int NB>
  __device__ __forceinline__ void operator()(f32x16 (&acc)[4][NB], const Pre<NB>&, int k0, int h0, int lane, int wave,
                                             char* lds, int slab_id) const {
    const int l32 = lane & 31, lhi = lane >> 5;
    if (slab_id >= 0) {            // this workgroup's range of the vocabulary: the raw sums go to its slab
      float* slab = partial + (int64_t)slab_id * (kBM * kBN);
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int k = k0 + mb * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
          if (k >= n_valid) continue;                          // padding rows of a short batch are not read back
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) slab[(k & (kBM - 1)) * kBN + (h0 & (kBN - 1)) + nb * 32 + l32] = acc[mb][nb][r];
        }
      return;
    }
    // 32 token rows at a time: beta_k * acc rounded to bf16 goes through this wavefront's own part of the LDS
    // ring (free after the k-loop; rows of NB * 64 + 16 bytes) and leaves as 16-byte stores, whole rows of the
    // wavefront's NB * 32 columns contiguous (2-byte stores straight from the accumulators took 80 k cycles
    // per tile).  LDS operations of one wavefront execute in order: no barrier between its writes and reads.
    constexpr int kRowBytes = NB * 64, kStageRow = kRowBytes + 16;
    constexpr int kChunks = kRowBytes / 16, kRowsPerStore = 64 / kChunks;
    char* stage = lds + wave * (32 * kStageRow);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * lhi + (r & 3);
        const int k = k0 + mb * 32 + row;
        const float b = k < n_valid ? beta[k] : 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          *(uint16_t*)(stage + row * kStageRow + (nb * 32 + l32) * 2) = f32_to_bf16_bits(b * acc[mb][nb][r]);
      }
#pragma unroll
      for (int i = 0; i < 32 / kRowsPerStore; ++i) {
        const int row = i * kRowsPerStore + lane / kChunks, ch = lane % kChunks;
        const uint4 val = *(const uint4*)(stage + row * kStageRow + ch * 16);
        const int k = k0 + mb * 32 + row, h = h0 + ch * 8;
        if (k < n_valid && h < H) *(uint4*)(dH + (int64_t)k * H + h) = val;     // H is a multiple of 8: whole chunks
      }
    }
  }
};

// dH^T tile of the contraction that reads W as it is: rows = hidden units (A = W^T, k-major), columns = tokens (B = E).
// A lane holds four consecutive hidden units of its token: 8-byte LDS writes, then the same 16-byte stores of whole rows.
// (11 registers go to scratch, 9 in the epilogue of the repacked path: the accumulators fill the file.)
struct DHiddenTEpilogue {
  int n_valid, H;
  uint16_t* dH;                    // rows of this chunk, [n_valid, H] bf16
  const float* beta;               // [n_valid]
  float* partial;                  // tiles whose contraction is cut into ranges: [slab][256 tokens][256 hidden] fp32 raw sums

  template <int NB> struct Pre {};
  template <int NB> static constexpr int stash_words() { return 0; }
  template <int NB> __device__ __forceinline__ void prefetch(int*, int, int, int, int) const {}
  template <int NB> __device__ __forceinline__ void unstash(Pre<NB>&, const int*, int) const {}
  template <int NB>
  __device__ __forceinline__ void operator()(f32x16 (&acc)[4][NB], const Pre<NB>&, int h0, int k0, int lane, int wave,
                                             char* lds, int slab_id) const {
    const int l32 = lane & 31, lhi = lane >> 5;
    if (slab_id >= 0) {
      float* slab = partial + (int64_t)slab_id * (kBM * kBN);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int k = k0 + nb * 32 + l32;
        if (k >= n_valid) continue;
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4)
            *(float4*)(slab + (k & (kBN - 1)) * kBM + (h0 & (kBM - 1)) + mb * 32 + 8 * r4 + 4 * lhi) =
                make_float4(acc[mb][nb][4 * r4], acc[mb][nb][4 * r4 + 1], acc[mb][nb][4 * r4 + 2], acc[mb][nb][4 * r4 + 3]);
      }
      return;
    }
    constexpr int kStageRow = 128 * 2 + 16;                    // 128 hidden units of a token, and 16 bytes of padding
    char* stage = lds + wave * (32 * kStageRow);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int kk = k0 + nb * 32 + l32;
      const float b = kk < n_valid ? beta[kk] : 0.f;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          uint2 w;
          w.x = pack_bf16x2(b * acc[mb][nb][4 * r4], b * acc[mb][nb][4 * r4 + 1]);
          w.y = pack_bf16x2(b * acc[mb][nb][4 * r4 + 2], b * acc[mb][nb][4 * r4 + 3]);
          *(uint2*)(stage + l32 * kStageRow + (mb * 32 + 8 * r4 + 4 * lhi) * 2) = w;
        }
#pragma unroll
      for (int i = 0; i < 8; ++i) {                            // four token rows of 256 bytes per instruction
        const int row = i * 4 + (lane >> 4), ch = lane & 15;
        const uint4 val = *(const uint4*)(stage + row * kStageRow + ch * 16);
        const int k = k0 + nb * 32 + row, h = h0 + ch * 8;
        if (k < n_valid && h < H) *(uint4*)(dH + (int64_t)k * H + h) = val;
      }
    }
  }
};

// dW tile: rows = vocabulary (A = E^T), columns = hidden units (B = (diag(beta) H_chunk)^T).
struct DWeightEpilogue {
  int V, H, accumulate;
  float* dW;                       // [V, H] fp32
  float* partial;                  // tiles whose contraction is cut into ranges: [slab][256][256] fp32 raw sums

  template <int NB> struct Pre {};
  template <int NB> static constexpr int stash_words() { return 0; }
  template <int NB> __device__ __forceinline__ void prefetch(int*, int, int, int, int) const {}
  template <int NB> __device__ __forceinline__ void unstash(Pre<NB>&, const int*, int) const {}
  // the wavefront's tile is MA x NB blocks of 32 x 32
  template <int MA, int NB, class P>
  __device__ __forceinline__ void operator()(f32x16 (&acc)[MA][NB], const P&, int v0, int h0, int lane, int,
                                             char*, int slab_id) const {
    const int l32 = lane & 31, lhi = lane >> 5;
    if (slab_id >= 0) {            // one range of this tile's tokens: raw sums to the slab, added up by dw_tail_reduce_kernel
      float* slab = partial + (int64_t)slab_id * (kBM * kBN);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MA; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            slab[((v0 & (kBM - 1)) + mb * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3)) * kBN + (h0 & (kBN - 1)) + nb * 32 + l32] = acc[mb][nb][r];
      return;
    }
    // One owner per element and launch, launches in stream order: the atomic sum is that of a
    // read-modify-write, but the addition happens at the L2 and the workgroup does not wait for it.
    // Addresses are a wave-uniform row pointer plus one per-lane offset (rows 4 * lhi further down, column
    // l32), and the two launch-wide conditions (accumulate or overwrite, every row inside the vocabulary or
    // the last tile's row check) are taken once, outside the loops: per element that leaves the store or
    // atomic and a scalar add (per-element branches and 64-bit vector address arithmetic made this epilogue
    // 31 k cycles per tile).
    const uint32_t lane_off = (uint32_t)(4 * lhi) * (uint32_t)H + (uint32_t)l32;   // elements
    const bool rows_ok = v0 + MA * 32 <= V;
    auto sweep = [&](auto acc_mode, auto checked) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        if (h0 + nb * 32 >= H) continue;                     // H is a multiple of 64: a 32-column block is in or out
#pragma unroll
        for (int mb = 0; mb < MA; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int v = v0 + mb * 32 + 8 * (r >> 2) + (r & 3);   // row of lanes 0..31 (wave-uniform)
            if (decltype(checked)::value && v + 4 * lhi >= V) continue;
            float* p = dW + (int64_t)v * H + (h0 + nb * 32) + lane_off;
            if (decltype(acc_mode)::value) unsafeAtomicAdd(p, acc[mb][nb][r]);
            else *p = acc[mb][nb][r];
          }
      }
    };
    if (accumulate) {
      if (rows_ok) sweep(std::true_type{}, std::false_type{});
      else sweep(std::true_type{}, std::true_type{});
    } else {
      if (rows_ok) sweep(std::false_type{}, std::false_type{});
      else sweep(std::false_type{}, std::true_type{});
    }
  }
};

// The same tile added to dW by reading, adding and storing, for short contractions: the fp32 memory atomics above run at
// 28 cycles an instruction, 1024 per tile, i.e. 1.9 ms for the whole of a 151936 x 4096 dW however few tokens are added to
// it.  32 rows of the wavefront's tile at a time go through its own part of the LDS ring (free after the k-loop), so that
// old values come and sums leave 16 bytes per lane, two whole rows of its columns per instruction; the old values are loaded
// two blocks ahead of their use and before the stores of the block in hand (the load counter would wait for those
// first).  One fp32 addition old + sum per element, as with the atomics.  See kReadAddSlices.  Two blocks of old values
// (128 registers), the results and the accumulators do not fit: 65 registers go to scratch in this epilogue, none in the k-loop.
struct DWeightAddEpilogue {
  DWeightEpilogue whole;           // ranges of cut tiles still go to their slabs

  template <int NB> struct Pre {};
  template <int NB> static constexpr int stash_words() { return 0; }
  template <int NB> __device__ __forceinline__ void prefetch(int*, int, int, int, int) const {}
  template <int NB> __device__ __forceinline__ void unstash(Pre<NB>&, const int*, int) const {}
  template <int MA, int NB, class P>
  __device__ __forceinline__ void operator()(f32x16 (&acc)[MA][NB], const P& pre, int v0, int h0, int lane, int wave,
                                             char* lds, int slab_id) const {
    if (slab_id >= 0) {
      whole(acc, pre, v0, h0, lane, wave, lds, slab_id);
      return;
    }
    constexpr int kCols = NB * 32, kLanesPerRow = kCols / 4, kRowsPer = 64 / kLanesPerRow, kN = 32 / kRowsPer;
    constexpr int kStageRow = kCols + 8;                       // floats: the two half-wavefronts' rows fall on different banks
    const int l32 = lane & 31, lhi = lane >> 5, H = whole.H;
    const int row = lane / kLanesPerRow, col = (lane % kLanesPerRow) * 4;
    float* stage = (float*)lds + wave * (32 * kStageRow);
    const int rows = whole.V - v0;                             // valid rows from v0 on (may be <= 0)
    const bool col_ok = h0 + col < H;                          // H is a multiple of 64: a lane's four columns are in or out
    float* dst = whole.dW + (int64_t)(v0 + row) * H + h0 + col;
    auto sweep = [&](auto all_valid) {
      constexpr bool kAll = decltype(all_valid)::value;        // no row or column to leave out
      float4 old[2][kN];
      auto fetch = [&](int mb) {
#pragma unroll
        for (int i = 0; i < kN; ++i) {
          const int r = mb * 32 + i * kRowsPer;
          if (kAll || (col_ok && r + row < rows)) old[mb & 1][i] = *(const float4*)(dst + (int64_t)r * H);
          else old[mb & 1][i] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      };
      fetch(0);
      fetch(1);
#pragma unroll
      for (int mb = 0; mb < MA; ++mb) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            stage[(8 * (r >> 2) + 4 * lhi + (r & 3)) * kStageRow + nb * 32 + l32] = acc[mb][nb][r];
        float4 out[kN];
#pragma unroll
        for (int i = 0; i < kN; ++i) {
          const float4 o = old[mb & 1][i], x = *(const float4*)(stage + (i * kRowsPer + row) * kStageRow + col);
          out[i] = make_float4(o.x + x.x, o.y + x.y, o.z + x.z, o.w + x.w);
        }
        if (mb + 2 < MA) fetch(mb + 2);
#pragma unroll
        for (int i = 0; i < kN; ++i) {
          const int r = mb * 32 + i * kRowsPer;
          if (kAll || (col_ok && r + row < rows)) *(float4*)(dst + (int64_t)r * H) = out[i];
        }
      }
    };
    if (rows >= MA * 32 && h0 + kCols <= H) sweep(std::true_type{});
    else sweep(std::false_type{});
  }
};

// dH tiles of a launch whose last tail_tiles tiles (in launch order) were cut into k_splits ranges of the vocabulary:
// dH[k][h] = beta_k * (slab 0 + slab 1 + ...) of the tile, in range order.  One block per 1024 elements of a tile.
__global__ void __launch_bounds__(256)
dh_tail_reduce_kernel(const float* __restrict__ partial, GemmArgs g, bool transposed, const float* __restrict__ beta,
                      int n_valid, int H, uint16_t* __restrict__ dH) {
  const int pos = blockIdx.y;
  int tm, tn;                                                          // tile of tokens, of hidden units
  if (transposed) tile_of_block(g, g.tiles_m * g.tiles_n - g.tail_tiles + pos, tn, tm);
  else tile_of_block(g, g.tiles_m * g.tiles_n - g.tail_tiles + pos, tm, tn);
  const int e = (blockIdx.x * 256 + threadIdx.x) * 4;                  // four hidden units of a token
  const int k = tm * kBM + e / kBN, h = tn * kBN + e % kBN;
  if (k >= n_valid || h >= H) return;                                  // H is a multiple of 64
  const float* slab = partial + (int64_t)pos * g.k_splits * (kBM * kBN) + e;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int r = 0; r < g.k_splits; ++r) {
    const float4 x = *reinterpret_cast<const float4*>(slab + (int64_t)r * (kBM * kBN));
    s.x += x.x; s.y += x.y; s.z += x.z; s.w += x.w;
  }
  const float b = beta[k];
  uint2 w;
  w.x = pack_bf16x2(b * s.x, b * s.y);
  w.y = pack_bf16x2(b * s.z, b * s.w);
  *reinterpret_cast<uint2*>(dH + (int64_t)k * H + h) = w;
}

// dW tiles of a launch whose last tail_tiles tiles (in launch order) were cut into k_splits ranges of tokens:
// dW[v][h] (+)= slab 0 + slab 1 + ... of the tile, in range order.  One block per 1024 elements of a tile.
__global__ void __launch_bounds__(256)
dw_tail_reduce_kernel(const float* __restrict__ partial, GemmArgs g, int V, int H, int accumulate, float* __restrict__ dW) {
  const int pos = blockIdx.y;
  int tm, tn;
  tile_of_block(g, g.tiles_m * g.tiles_n - g.tail_tiles + pos, tm, tn);
  const float* slab = partial + (int64_t)pos * g.k_splits * (kBM * kBN);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = (blockIdx.x * 4 + q) * 256 + threadIdx.x;
    const int v = tm * kBM + e / kBN, h = tn * kBN + e % kBN;
    if (v >= V || h >= H) continue;
    float sum = 0.f;
    for (int r = 0; r < g.k_splits; ++r) sum += slab[(int64_t)r * (kBM * kBN) + e];
    float* p = dW + (int64_t)v * H + h;
    *p = accumulate ? *p + sum : sum;
  }
}

// ----------------------------------------------------- reference logit ----
// ref[kk] = h_k . W[ids_k] in fp32, one wavefront per token (row-major caller arrays).
// An id outside [0, V) reads no row of W and gets the shift 0.
__device__ __forceinline__ void target_logit(const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ W,
                                             const int32_t* __restrict__ ids, int n_valid, int H, int V,
                                             float* __restrict__ ref, int block) {
  const int kk = block * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (kk >= n_valid) return;
  const int y = ids[kk];
  if (y < 0 || y >= V) {
    if (lane == 0) ref[kk] = 0.f;
    return;
  }
  const uint4* hp = (const uint4*)(hidden + (int64_t)kk * H);
  const uint4* wp = (const uint4*)(W + (int64_t)y * H);
  float s = 0.f;
  for (int j = lane; j < H / 8; j += 64) {
    const uint4 a = hp[j], b = wp[j];
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s = fmaf(__builtin_bit_cast(float, aw[q] << 16), __builtin_bit_cast(float, bw[q] << 16), s);
      s = fmaf(__builtin_bit_cast(float, aw[q] & 0xffff0000u), __builtin_bit_cast(float, bw[q] & 0xffff0000u), s);
    }
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) ref[kk] = s;
}

// H_chunk in the blocked layout (the first pack_blocks blocks, H / 64 of them to 64 rows) and the exponent shifts (the
// others): one launch, both read the same rows.
__global__ void __launch_bounds__(256)
hidden_prep_kernel(const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ W, const int32_t* __restrict__ ids,
                   int n_valid, int H, int V, uint16_t* __restrict__ Hb, float* __restrict__ ref, int pack_blocks) {
  const int block = (int)blockIdx.x;
  if (block >= pack_blocks) {
    target_logit(hidden, W, ids, n_valid, H, V, ref, block - pack_blocks);
    return;
  }
  const int cb = H / 64, r0 = block / cb * 64, c0 = block % cb * 64, kb = H >> 5;
  const int c = c0 + 8 * (threadIdx.x & 7);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = r0 + (threadIdx.x >> 3) + 32 * i;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (r < n_valid) x = *reinterpret_cast<const uint4*>(hidden + (int64_t)r * H + c);
    *reinterpret_cast<uint4*>(Hb + blk_off(r, c, kb)) = x;
  }
}

// ------------------------------------------------- per-token statistics ----
// A granule's partial sum at or above e^70 means some numerator reached the range in which the
// clamp of the exponent shift acts (a clamped numerator alone makes its granule's sum that large).
constexpr float kShiftRangeLimit = 2.5154386709191669e30f;     // e^70

// Per-token sums of the per-granule partials: kStatTokens tokens per workgroup; the granules of a
// token are split over kStatParts groups of threads (granule gi goes to group gi % kStatParts), each
// of which walks its granules in order, and the groups' sums are added in a fixed tree, so the result
// does not depend on timing.  Bound by the latency of the walk (149 granules per group at V = 151936): with 32
// loads in flight instead of 8 a launch over 3000 tokens takes 14 us instead of 19.  Returns to the first kStatTokens threads only.
constexpr int kStatTokens = 32, kStatParts = 8, kStatBatch = 32;
struct TokenSums { float S, TZ; bool in_shift_range; };
struct StatShared { float s[kStatParts][kStatTokens], t[kStatParts][kStatTokens], m[kStatParts][kStatTokens]; };

__device__ __forceinline__ TokenSums token_sums(const float* __restrict__ s_part, const float* __restrict__ t_part,
                                                int n_granules, int64_t ld, int kk, bool valid, StatShared& sh) {
  const int t = threadIdx.x % kStatTokens, part = threadIdx.x / kStatTokens;
  float s = 0.f, tz = 0.f, mx = 0.f;
  // kStatBatch loads in flight, added in granule order (0 past the end leaves the sums as they are)
  auto walk = [&](const float* __restrict__ p, auto use) {
    for (int g0 = part; g0 < n_granules; g0 += kStatParts * kStatBatch) {
      float v[kStatBatch];
#pragma unroll
      for (int e = 0; e < kStatBatch; ++e) {
        const int gi = g0 + e * kStatParts;
        v[e] = gi < n_granules ? p[(int64_t)gi * ld + kk] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < kStatBatch; ++e) use(v[e]);
    }
  };
  if (valid) {
    walk(s_part, [&](float v) { s += v; mx = fmaxf(mx, v); });
    if (t_part) walk(t_part, [&](float v) { tz += v; });
  }
  sh.s[part][t] = s;
  sh.t[part][t] = tz;
  sh.m[part][t] = mx;
  __syncthreads();
  TokenSums out;
  out.S = ((sh.s[0][t] + sh.s[1][t]) + (sh.s[2][t] + sh.s[3][t])) + ((sh.s[4][t] + sh.s[5][t]) + (sh.s[6][t] + sh.s[7][t]));
  out.TZ = ((sh.t[0][t] + sh.t[1][t]) + (sh.t[2][t] + sh.t[3][t])) + ((sh.t[4][t] + sh.t[5][t]) + (sh.t[6][t] + sh.t[7][t]));
  float m = sh.m[0][t];
  for (int q = 1; q < kStatParts; ++q) m = fmaxf(m, sh.m[q][t]);
  out.in_shift_range = m >= kShiftRangeLimit;
  return out;
}

__global__ void __launch_bounds__(256)
token_stats_kernel(const float* __restrict__ s_part, const float* __restrict__ t_part, int n_granules, int64_t ld,
                   const float* __restrict__ ref, const float* __restrict__ z_target, int n_valid, int chunk_start,
                   const int32_t* __restrict__ ids, int V,
                   const float* __restrict__ old_logp, const float* __restrict__ adv,
                   const int32_t* __restrict__ kept_seq, const float* __restrict__ kept_w,
                   float eps_lo, float eps_hi, float grad_scale, KlArgs klp,
                   float* __restrict__ beta_out, uint16_t* __restrict__ Eb, int kb_z,
                   float* __restrict__ logp_out, float* __restrict__ kl_out, float* __restrict__ entropy_out,
                   float* __restrict__ term, int32_t* __restrict__ diag) {
  __shared__ StatShared sh;
  const int kk = blockIdx.x * kStatTokens + threadIdx.x % kStatTokens;
  const bool valid = kk < n_valid;
  const TokenSums sums = token_sums(s_part, t_part, n_granules, ld, kk, valid, sh);
  if (threadIdx.x >= kStatTokens) return;                // the first threads finish the tokens
  bool bad_id = false, clipped = false, nonzero_adv = false;
  if (valid) {
    const float S = sums.S;
    const int k = chunk_start + kk;
    const int y = ids[kk];
    bad_id = y < 0 || y >= V;
    if (entropy_out) entropy_out[k] = logf(S) - sums.TZ / S;   // -sum_v p_v log p_v, p_v = E_v / S
    if (bad_id) {                                        // left out: no loss term, zero gradient
      beta_out[kk] = 0.f;
      if (logp_out) logp_out[k] = __builtin_nanf("");
      if (kl_out) kl_out[k] = __builtin_nanf("");
      term[k] = 0.f;
    } else {
      const float lse = ref[kk] + logf(S);
      const float logp = z_target[kk] - lse;
      const float w = kept_w[k];
      const float A = adv[kept_seq[k]];
      const TokenScalars ts = grpo_token_scalars(logp, old_logp[k], A, w, eps_lo, eps_hi, grad_scale,
                                                 klp.beta, klp.kind, klp.beta != 0.f ? klp.ref_logp[k] : 0.f);
      clipped = ts.clipped;
      nonzero_adv = A != 0.f;
      beta_out[kk] = -ts.c / S;                          // dz_kv = beta_k E_kv off the target
      // the target entry of E is replaced by E' with beta_k E' = c_k (1 - p_target): the two backward
      // contractions then need no separate one-hot term
      Eb[blk_off(kk, y, kb_z)] = f32_to_bf16_bits(-S * (1.f - __expf(logp)));
      if (logp_out) logp_out[k] = logp;
      if (kl_out) kl_out[k] = ts.kl;
      term[k] = w * ts.L;
    }
  }
  if (diag) {
    wave_count(bad_id, diag + NAT_DIAG_BAD_ID);
    wave_count(valid && sums.in_shift_range, diag + NAT_DIAG_SHIFT_RANGE);
    wave_count(clipped, diag + NAT_DIAG_CLIPPED);
    wave_count(nonzero_adv, diag + NAT_DIAG_NONZERO_ADV);
  }
}

// Forward pass alone: log-prob of the target (and the entropy) from the per-granule sums.
__global__ void __launch_bounds__(256)
logp_stats_kernel(const float* __restrict__ s_part, const float* __restrict__ t_part, int n_granules, int64_t ld,
                  const float* __restrict__ ref, const float* __restrict__ z_target, int n_valid, int chunk_start,
                  const int32_t* __restrict__ ids, int V,
                  float* __restrict__ logp_out, float* __restrict__ entropy_out, int32_t* __restrict__ diag) {
  __shared__ StatShared sh;
  const int kk = blockIdx.x * kStatTokens + threadIdx.x % kStatTokens;
  const bool valid = kk < n_valid;
  const TokenSums sums = token_sums(s_part, t_part, n_granules, ld, kk, valid, sh);
  if (threadIdx.x >= kStatTokens) return;
  bool bad_id = false;
  if (valid) {
    const int k = chunk_start + kk;
    const int y = ids[kk];
    bad_id = y < 0 || y >= V;
    logp_out[k] = bad_id ? __builtin_nanf("") : z_target[kk] - (ref[kk] + logf(sums.S));
    if (entropy_out) entropy_out[k] = logf(sums.S) - sums.TZ / sums.S;
  }
  if (diag) {
    wave_count(bad_id, diag + NAT_DIAG_BAD_ID);
    wave_count(valid && sums.in_shift_range, diag + NAT_DIAG_SHIFT_RANGE);
  }
}

// -------------------------------------------------------------- host side ----
static inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

struct Bf16Plan {
  int64_t Vp, Hp; int n_granules; int cap;      // padded vocabulary / hidden size, granules, chunk capacity (tokens)
  size_t off_Wb, off_Wtb, off_Hb, off_Hktb, off_Eb, off_s, off_t, off_zt, off_ref, off_beta, off_term, off_dh_part, total;
};

static Bf16Plan make_plan(int32_t N_k, int32_t H, int32_t V, int cap) {
  Bf16Plan p;
  p.Vp = round_up(V, kBM);
  p.Hp = round_up(H, kBN);
  p.n_granules = (int)(p.Vp / kGranule);
  p.cap = cap;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) / 256 * 256; return o; };
  p.off_Wb = take((size_t)p.Vp * H * 2);        // W:    rows = vocabulary, k = hidden
  p.off_Wtb = take((size_t)p.Hp * p.Vp * 2);    // W^T:  rows = hidden,     k = vocabulary
  p.off_Hb = take((size_t)cap * H * 2);         // H_chunk:   rows = tokens, k = hidden
  p.off_Hktb = take((size_t)p.Hp * cap * 2);    // H_chunk^T: rows = hidden, k = tokens
  p.off_Eb = take((size_t)cap * p.Vp * 2);      // E: rows = tokens, k = vocabulary (its one copy)
  p.off_s = take((size_t)p.n_granules * cap * 4);
  p.off_t = take((size_t)p.n_granules * cap * 4);
  p.off_zt = take((size_t)cap * 4);
  p.off_ref = take((size_t)cap * 4);
  p.off_beta = take((size_t)cap * 4);
  p.off_term = take((size_t)(N_k > 0 ? N_k : 1) * 4);
  p.off_dh_part = take((size_t)kNumCU * kBM * kBN * 4);   // raw fp32 tiles of a contraction cut into ranges (dH, or the last dW tiles): 64 MiB
  p.total = off;
  return p;
}

// Token rows per launch of the logits and dH contractions inside a chunk of `cap` rows: the smallest
// multiple of kSubChunk whose dH launch (rows / 256 x Hp / 256 tiles) fills whole waves of kNumCU
// workgroups to at least 97 %; the whole chunk if none does.  (Hp = 4096: 8192 rows = 512 tiles;
// Hp = 5120: 16384 rows = 1280 tiles; Hp = 3584 and 1024: the whole chunk.)
static int sub_chunk_rows(int cap, int Hp) {
  if (kSubChunk < 8192) return kSubChunk < cap ? kSubChunk : cap;   // a test build: the sub-chunk logic on small shapes
  const int n_col = Hp / kBN;
  for (int rows = kSubChunk; rows < cap; rows += kSubChunk) {
    const int tiles = rows / kBM * n_col;
    const int waves = (tiles + kNumCU - 1) / kNumCU;
    if (tiles * 100 >= waves * kNumCU * 97) return rows;
  }
  return cap;
}

// Chunk capacity of the recommended workspace.  Forward pass alone: kMaxChunk.  With the backward pass the
// chunk also sizes the stored soft-max numerators (cap x Vp x 2 bytes), and the dW contraction, whose
// contraction axis is the chunk, is within 0.2 % of its 32768-token speed at 16384 (measured): the
// smallest of 16384 / 24576 / 32768 rows whose dH launch fills whole rounds of workgroups to 97 %.
static int recommended_cap(int32_t N_k, int32_t H, bool backward) {
  const int64_t all = round_up(N_k > 0 ? N_k : 1, kBN);
  if (!backward) return (int)(all > kMaxChunk ? kMaxChunk : all);
  if (all <= kMaxChunk / 2) return (int)all;
  const int n_col = (int)(round_up(H, kBN) / kBN);
  for (int cap = kMaxChunk / 2; cap < kMaxChunk; cap += kMaxChunk / 4) {
    const int tiles = cap / kBM * n_col;
    const int waves = (tiles + kNumCU - 1) / kNumCU;
    if (tiles * 100 >= waves * kNumCU * 97) return (int)(all < cap ? all : cap);
  }
  return (int)(all > kMaxChunk ? kMaxChunk : all);
}

size_t loss_bf16_workspace_bytes(int32_t N_k, int32_t H, int32_t V, bool minimal) {
  return make_plan(N_k, H, V, minimal ? kBN : recommended_cap(N_k, H, true)).total;
}

// workspace of the forward pass alone: W and H_chunk blocked, the partial sums, two per-token vectors
struct FwdPlan { int64_t Vp; int n_granules; int cap; size_t off_Wb, off_Hb, off_s, off_t, off_zt, off_ref, total; };

static FwdPlan make_fwd_plan(int32_t H, int32_t V, int cap) {
  FwdPlan p;
  p.Vp = round_up(V, kBM);
  p.n_granules = (int)(p.Vp / kGranule);
  p.cap = cap;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) / 256 * 256; return o; };
  p.off_Wb = take((size_t)p.Vp * H * 2);
  p.off_Hb = take((size_t)cap * H * 2);
  p.off_s = take((size_t)p.n_granules * cap * 4);
  p.off_t = take((size_t)p.n_granules * cap * 4);
  p.off_zt = take((size_t)cap * 4);
  p.off_ref = take((size_t)cap * 4);
  p.total = off;
  return p;
}

size_t logp_bf16_workspace_bytes(int32_t N_k, int32_t H, int32_t V, bool minimal) {
  return make_fwd_plan(H, V, minimal ? kBN : recommended_cap(N_k, H, false)).total;
}

// How a launch of `tiles` output tiles and `kt_all` k-slices uses the compute units.  Full rounds of one tile per
// compute unit run whole; the tiles left over (at most half a round: with more, two ranges each would not fit one
// round) are cut into as many ranges of the contraction axis as fill the chip once, of at least kMinSlicesPerRange
// on average (a workgroup's load ring and epilogue cost about ten slices), starts multiples of `align`; the last range takes
// what that rounding leaves (1256 slices in 39 ranges: 38 of 33 and one of 2).
// 5003 tokens at the 7B head: 280 dH tiles took a second round for 24 of them, 6.26 ms; cut into ten ranges, 3.96 ms.
struct RangeCut { int splits, kt_per, tail, grid; };
static RangeCut range_cut(int tiles, int kt_all, int align) {
  RangeCut c{1, kt_all, 0, tiles};
  const int tail = tiles % kNumCU;
  if (tail == 0 || tail * 2 > kNumCU) return c;
  int splits = kNumCU / tail;
  if (splits > kt_all / kMinSlicesPerRange) splits = kt_all / kMinSlicesPerRange;
  if (splits <= 1) return c;
  c.kt_per = (int)round_up((kt_all + splits - 1) / splits, align);
  c.splits = (kt_all + c.kt_per - 1) / c.kt_per;                   // every range non-empty
  if (c.splits <= 1) return RangeCut{1, kt_all, 0, tiles};
  c.tail = tail;
  c.grid = tiles - tail + tail * c.splits;
  return c;
}

// Up to how many tokens a call reads W as it is instead of repacking it first.  The repack moves W three times with the
// backward pass (0.77 ms at V x H = 151936 x 4096, 0.21 ms at H = 1024), twice without (0.50 / 0.12 ms), whatever the
// batch; reading rows costs the logits contraction 1 to 2 % and the dH contraction, with its transposing reads, 3 to
// 5 %, so the gain shrinks with the batch.  The lines are where it ends for the last of the hidden sizes; repacked against
// direct in alternating runs, whole call, ms at V = 151936 unless stated.  H a multiple of the 256-wide dH tile: 1500 tokens
// 5.56 / 4.99 (H = 4096), 1.55 / 1.41 (1024); 5000: 15.1 / 14.6, 4.17 / 4.07; 7168: 21.7 / 21.2 (4096), 5.75 / 5.66 (1024), 27.08 / 26.96
// (5120); 8192: 23.5 / 23.2 (4096) but 29.4 / 29.7 (5120).  Other H, whose dH tiles are padded (the work grows with the
// tiles, the repack with H): 1500: 1.08 / 0.97 (576), 0.80 / 0.72 (320); 5000: 2.88 / 2.87, 2.03 / 2.00; 6144: 3.46 / 3.48, 2.39 / 2.39; 7168: 3.97 / 4.01, 2.77 / 2.81;
// 8192 at V = 50000: 1.08 / 1.10 (320).  Forward pass alone: 2000 tokens 2.42 / 1.98 (4096), 0.68 / 0.59 (1024); 12289 with the
// entropy: 12.02 / 11.79, 3.52 / 3.38; 24576: 24.4 / 24.1, 6.42 / 6.37, 29.9 / 29.7 (5120); 49152: 45.7 / 45.7, 12.9 / 12.9, 57.0 / 57.8; with
// contractions of a few slices 5000: 0.386 / 0.386 (H = 64, V = 160000), 16384: 1.19 / 1.20.
static int direct_tokens(int H) { return H % kBN == 0 ? 7168 : 6144; }
static int direct_tokens_forward(int H) { return H >= kBN ? 24576 : 8192; }

// Up to how many k-slices (32 tokens) a chunk is added to dW by reading, adding and storing instead of by atomics.
// Accumulating call, atomics against read-add-store, ms at V x H = 151936 x 4096: 59 tokens 2.47 / 1.66, 300: 2.88 / 2.23,
// 1237: 4.76 / 4.58, 2500: 8.70 / 8.74, 4096: 12.04 / 12.18; at H = 1024: 59 tokens 0.68 / 0.50, 600: 1.03 / 0.90, 4096: equal.
constexpr int kReadAddSlices = 64;

// logits contraction: rows = vocabulary, columns = tokens (tiles_n tiles), contraction over the hidden size; W either
// repacked (Wb) or read as it is (Wb NULL)
template <class Epi>
static nat_status launch_logits(const uint16_t* W, const uint16_t* Wb, const uint16_t* Hb, int V, int H, int Vp, int tiles_n,
                                const Epi& epi, hipStream_t s) {
  ProfScope prof(PC_LOGITS, s);
  GemmArgs g{Wb ? Wb : W, Hb, H, Vp / kBM, tiles_n, NAT_GROUP_LOGITS, 0, H / kBK, 1, 0, 0, V, H};
  const int grid = g.tiles_m * g.tiles_n;
  if (Wb) gemm_nt_kernel<Epi, NAT_WAVES_LOGITS><<<grid, NAT_WAVES_LOGITS * 64, 0, s>>>(g, epi);
  else gemm_nt_kernel<Epi, NAT_WAVES_LOGITS, ASource::kRows><<<grid, NAT_WAVES_LOGITS * 64, 0, s>>>(g, epi);
  NAT_LAUNCH_CHECK();
  return NAT_OK;
}

nat_status loss_bf16_run(const LossArgs& a) {
  // largest chunk capacity (multiple of 256 tokens) whose plan fits the workspace
  int cap = recommended_cap(a.N_k, a.H, true);
  while (cap > kBN && make_plan(a.N_k, a.H, a.V, cap).total > a.ws_bytes) cap -= kBN;
  const Bf16Plan p = make_plan(a.N_k, a.H, a.V, cap);
  if (p.total > a.ws_bytes) return NAT_WORKSPACE_TOO_SMALL;
  hipStream_t s = a.stream;
  char* ws = (char*)a.ws;
  uint16_t* Wb = (uint16_t*)(ws + p.off_Wb);
  uint16_t* Wtb = (uint16_t*)(ws + p.off_Wtb);
  uint16_t* Hb = (uint16_t*)(ws + p.off_Hb);
  uint16_t* Hktb = (uint16_t*)(ws + p.off_Hktb);
  uint16_t* Eb = (uint16_t*)(ws + p.off_Eb);
  float* s_part = (float*)(ws + p.off_s);
  float* t_part = a.entropy_out ? (float*)(ws + p.off_t) : nullptr;
  float* zt = (float*)(ws + p.off_zt);
  float* ref = (float*)(ws + p.off_ref);
  float* beta = (float*)(ws + p.off_beta);
  float* term = (float*)(ws + p.off_term);
  float* dh_part = (float*)(ws + p.off_dh_part);
  const uint16_t* W = (const uint16_t*)a.W;
  const uint16_t* hidden = (const uint16_t*)a.hidden;
  const int H = a.H, V = a.V;
  const int Vp = (int)p.Vp, Hp = (int)p.Hp;

  const bool direct = a.N_k <= direct_tokens(H);
  if (!direct) {  // W and W^T in the blocked layout, padding zero-filled
    ProfScope prof(PC_TRANSPOSE, s);
    pack_blocked_kernel<<<dim3(Vp / 64, Hp / 64), 256, 0, s>>>(W, H, V, H, Vp, Hp, Wb, Wtb, Vp / 32, nullptr);
    NAT_LAUNCH_CHECK();
  }
  const int sub = sub_chunk_rows(cap, Hp);
  for (int c0 = 0; c0 < a.N_k; c0 += cap) {
    const int nv = a.N_k - c0 < cap ? a.N_k - c0 : cap;
    const int np = (int)round_up(nv, kBN);
    const uint16_t* hid_c = hidden + (int64_t)c0 * H;
    {  // H_chunk in the blocked layout; exponent shift = target logit
      ProfScope prof(PC_TRANSPOSE, s);
      const int pack_blocks = np / 64 * (H / 64);
      hidden_prep_kernel<<<pack_blocks + (nv + 3) / 4, 256, 0, s>>>(hid_c, W, a.ids + c0, nv, H, V, Hb, ref, pack_blocks);
      NAT_LAUNCH_CHECK();
    }
    // The forward sweep and the dH contraction go over the chunk in sub-chunks: shorter launches of
    // the three contractions alternate, which this power-limited part rewards with a higher clock
    // (measured: both run faster on 8192 tokens than on 32768), while the dW contraction below keeps
    // the whole chunk as its contraction axis (it is the one that loses on short axes).
    for (int s0 = 0; s0 < nv; s0 += sub) {
      const int snv = nv - s0 < sub ? nv - s0 : sub;
      const int snp = (int)round_up(snv, kBN);
      uint16_t* Eb_s = Eb + (int64_t)(s0 / 256) * (Vp / 32) * kBlkElems;    // token tile s0 / 256
      const int32_t* ids_s = a.ids + c0 + s0;
      {  // logits: rows = vocabulary, columns = tokens, contraction over the hidden size
        const uint16_t* Hb_s = Hb + (int64_t)(s0 / 256) * (H / 32) * kBlkElems;
        nat_status st;
        if (t_part) {
          LogitsEpilogue<true> e{V, snv, cap, Vp / 32, Eb_s, s_part + s0, t_part + s0, zt + s0, ids_s, ref + s0};
          st = launch_logits(W, direct ? nullptr : Wb, Hb_s, V, H, Vp, snp / kBN, e, s);
        } else {
          LogitsEpilogue<false> e{V, snv, cap, Vp / 32, Eb_s, s_part + s0, nullptr, zt + s0, ids_s, ref + s0};
          st = launch_logits(W, direct ? nullptr : Wb, Hb_s, V, H, Vp, snp / kBN, e, s);
        }
        if (st != NAT_OK) return st;
      }
      {
        ProfScope prof(PC_TOKEN_STATS, s);
        token_stats_kernel<<<(snv + kStatTokens - 1) / kStatTokens, kStatTokens * kStatParts, 0, s>>>(
            s_part + s0, t_part ? t_part + s0 : nullptr, p.n_granules, cap, ref + s0, zt + s0, snv, c0 + s0, ids_s, V,
            a.old_logp, a.adv, a.kept_seq, a.kept_w, a.eps_lo, a.eps_hi, a.grad_scale,
            KlArgs{a.ref_logp, a.beta_kl, a.kl_kind}, beta + s0, Eb_s, Vp / 32, a.logp, a.kl_out, a.entropy_out, term, a.diag);
        NAT_LAUNCH_CHECK();
      }
      {  // (diag(beta) H)^T of the sub-chunk into its k-slices of the chunk's blocked operand
        ProfScope prof(PC_TRANSPOSE, s);
        pack_blocked_kernel<<<dim3(snp / 64, Hp / 64), 256, 0, s>>>(hid_c + (int64_t)s0 * H, H, snv, H, snp, Hp, nullptr,
                                                                   Hktb + (int64_t)(s0 / 32) * kBlkElems, np / 32, beta + s0);
        NAT_LAUNCH_CHECK();
      }
      {  // dH: rows = tokens, columns = hidden units, contraction over the padded vocabulary
        // The tiles left over after the last full round of one tile per compute unit (all of them in a short batch)
        // are cut into ranges of the vocabulary: see range_cut.
        const int tiles = (snp / kBM) * (Hp / kBN);
        const RangeCut cut = range_cut(tiles, Vp / kBK, 1);
        uint16_t* dH_s = (uint16_t*)a.dH + (int64_t)(c0 + s0) * H;
        ProfScope prof(PC_DHIDDEN, s);
        GemmArgs g{Eb_s, Wtb, Vp, snp / kBM, Hp / kBN, NAT_GROUP_DHIDDEN, 0, Vp / kBK, cut.splits, cut.kt_per, cut.tail, V, H};
        if (direct) {            // dH^T = W^T E^T from W as it is
          g.A = W;
          g.B = Eb_s;
          g.tiles_m = Hp / kBM;
          g.tiles_n = snp / kBN;
          DHiddenTEpilogue e{snv, H, dH_s, beta + s0, dh_part};
          gemm_nt_kernel<DHiddenTEpilogue, NAT_WAVES_DHIDDEN, ASource::kKMajorRows><<<cut.grid, NAT_WAVES_DHIDDEN * 64, 0, s>>>(g, e);
        } else {
          DHiddenEpilogue e{snv, H, dH_s, beta + s0, dh_part};
          gemm_nt_kernel<DHiddenEpilogue, NAT_WAVES_DHIDDEN><<<cut.grid, NAT_WAVES_DHIDDEN * 64, 0, s>>>(g, e);
        }
        NAT_LAUNCH_CHECK();
        if (cut.splits > 1) {
          dh_tail_reduce_kernel<<<dim3(kBM * kBN / 1024, cut.tail), 256, 0, s>>>(dh_part, g, direct, beta + s0, snv, H, dH_s);
          NAT_LAUNCH_CHECK();
        }
      }
    }
    {  // dW: rows = vocabulary, columns = hidden units, contraction over the chunk's (padded) tokens
      // A = E from its one copy (rows = token), i.e. stored along this contraction's k axis
      // The leftover tiles of the last round are cut into ranges of tokens (multiples of the 8 k-slices that the
      // k-major loader starts at): see range_cut.
      const int kt = (nv + kBK - 1) / kBK;                       // only the slices that hold tokens
      const RangeCut cut = range_cut((Vp / kBM) * (Hp / kBN), kt, 8);
      const int accumulate = (c0 > 0 || a.accumulate_dw) ? 1 : 0;
      GemmArgs g{Eb, Hktb, kt * kBK, Vp / kBM, Hp / kBN, NAT_GROUP_DWEIGHT, Vp / 32, np / kBK, cut.splits, cut.kt_per, cut.tail};
      DWeightEpilogue e{V, H, accumulate, a.dW, dh_part};
      {
        ProfScope prof(PC_DWEIGHT, s);
        if (accumulate && kt <= kReadAddSlices)
          gemm_nt_kernel<DWeightAddEpilogue, NAT_WAVES_DWEIGHT, ASource::kKMajorBlocked><<<cut.grid, NAT_WAVES_DWEIGHT * 64, 0, s>>>(g, DWeightAddEpilogue{e});
        else
          gemm_nt_kernel<DWeightEpilogue, NAT_WAVES_DWEIGHT, ASource::kKMajorBlocked><<<cut.grid, NAT_WAVES_DWEIGHT * 64, 0, s>>>(g, e);
        NAT_LAUNCH_CHECK();
        if (cut.splits > 1) {
          dw_tail_reduce_kernel<<<dim3(kBM * kBN / 1024, cut.tail), 256, 0, s>>>(dh_part, g, V, H, accumulate, a.dW);
          NAT_LAUNCH_CHECK();
        }
      }
    }
  }
  ProfScope prof(PC_LOSS_REDUCE, s);
  loss_reduce_kernel<<<1, 1024, 0, s>>>(term, a.N_k, a.loss);
  NAT_LAUNCH_CHECK();
  return NAT_OK;
}

nat_status logp_bf16_run(const LogpArgs& a) {
  int cap = recommended_cap(a.N_k, a.H, false);
  while (cap > kBN && make_fwd_plan(a.H, a.V, cap).total > a.ws_bytes) cap -= kBN;
  const FwdPlan p = make_fwd_plan(a.H, a.V, cap);
  if (p.total > a.ws_bytes) return NAT_WORKSPACE_TOO_SMALL;
  hipStream_t s = a.stream;
  char* ws = (char*)a.ws;
  uint16_t* Wb = (uint16_t*)(ws + p.off_Wb);
  uint16_t* Hb = (uint16_t*)(ws + p.off_Hb);
  float* s_part = (float*)(ws + p.off_s);
  float* t_part = a.entropy ? (float*)(ws + p.off_t) : nullptr;
  float* zt = (float*)(ws + p.off_zt);
  float* ref = (float*)(ws + p.off_ref);
  const uint16_t* W = (const uint16_t*)a.W;
  const uint16_t* hidden = (const uint16_t*)a.hidden;
  const int H = a.H, V = a.V, Vp = (int)p.Vp;
  const bool direct = a.N_k <= direct_tokens_forward(H);
  if (!direct) {
    ProfScope prof(PC_TRANSPOSE, s);
    pack_blocked_kernel<<<dim3(Vp / 64, H / 64), 256, 0, s>>>(W, H, V, H, Vp, H, Wb, nullptr, 0, nullptr);
    NAT_LAUNCH_CHECK();
  }
  for (int c0 = 0; c0 < a.N_k; c0 += cap) {
    const int nv = a.N_k - c0 < cap ? a.N_k - c0 : cap;
    const int np = (int)round_up(nv, kBN);
    const uint16_t* hid_c = hidden + (int64_t)c0 * H;
    {
      ProfScope prof(PC_TRANSPOSE, s);
      const int pack_blocks = np / 64 * (H / 64);
      hidden_prep_kernel<<<pack_blocks + (nv + 3) / 4, 256, 0, s>>>(hid_c, W, a.ids + c0, nv, H, V, Hb, ref, pack_blocks);
      NAT_LAUNCH_CHECK();
    }
    {
      nat_status st;
      if (t_part) {
        LogitsEpilogue<true, false> e{V, nv, cap, 0, nullptr, s_part, t_part, zt, a.ids + c0, ref};
        st = launch_logits(W, direct ? nullptr : Wb, Hb, V, H, Vp, np / kBN, e, s);
      } else {
        LogitsEpilogue<false, false> e{V, nv, cap, 0, nullptr, s_part, nullptr, zt, a.ids + c0, ref};
        st = launch_logits(W, direct ? nullptr : Wb, Hb, V, H, Vp, np / kBN, e, s);
      }
      if (st != NAT_OK) return st;
    }
    {
      ProfScope prof(PC_TOKEN_STATS, s);
      logp_stats_kernel<<<(nv + kStatTokens - 1) / kStatTokens, kStatTokens * kStatParts, 0, s>>>(s_part, t_part, p.n_granules, cap, ref, zt, nv, c0, a.ids + c0, V,
                                                      a.logp, a.entropy, a.diag);
      NAT_LAUNCH_CHECK();
    }
  }
  return NAT_OK;
}

}  // namespace nat
