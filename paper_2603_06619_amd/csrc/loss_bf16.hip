// bf16 path of nat_loss_fwd_bwd / nat_loss_fwd_bwd_kl / nat_logp_fwd for gfx950: LM-head
// projection, full-vocabulary log-softmax, clipped GRPO surrogate with Horvitz-Thompson
// weights (Eq. 1, 3, 5, 6/9), optional KL term (Eq. 4) and entropy, and the gradients dH, dW
// (App. A) on the kept tokens.  The forward pass alone runs the first two steps below and
// keeps only the sums.
//
// Tokens are processed in chunks of at most `cap` rows (16384 or 32768 with the recommended workspace); the
// forward sweep and the dH contraction of a chunk run in sub-chunks of 8192 rows.  Per chunk:
//   reference     ref_k = h_k . W[ids_k]: the target logit, used only as the exponent shift;
//   logits GEMM   Z^T = W . H_chunk^T on bf16 MFMA with fp32 accumulators; the epilogue never
//                 stores Z: it stores E = exp(z - ref_k) as bf16, ONCE, rows = token (soft-max
//                 numerators: bf16 keeps their relative precision), per (token, 128-row vocabulary
//                 granule) partial sums of E, and the exact target logit;
//   token stats   S_k = sum of the partials (fixed order), lse = ref + log S, log-prob, ratio,
//                 clipped surrogate, c_k = dLoss/dlogp_k, beta_k = -c_k / S_k;
//                 dz_kv = beta_k E_kv, except the target entry c_k (1 - p_target), which is
//                 patched into E as -S_k (1 - p_target), computed in fp32 before rounding;
//   dH GEMM       dH = diag(beta) (E . W)            (contraction over the vocabulary);
//   dW GEMM       dW (+)= E^T . (diag(beta) H_chunk) (contraction over the chunk's tokens, fp32,
//                 one owner per output tile, chunks in order: deterministic).  Its operand E^T is
//                 the same copy of E, which is stored along this contraction's k axis: the tile
//                 is gathered in 2 KiB pieces and fragments are formed by the transposing LDS
//                 read (ds_read_b64_tr_b16).
// The shift by the target logit needs log(p_max / p_target) < 70 for every kept token (E is
// clamped there; the token statistics count the tokens this may have touched); a token the current
// policy gives less than e^-70 of its mode's probability does not occur for rollouts drawn from a
// behaviour policy inside the clip range.
// All three contractions run through one "NT" kernel (both operands contiguous along the
// contraction axis; the k-major operand of dW is the one exception described above).  Every
// operand is kept in a blocked layout in the workspace: blocks of 256 rows x 32 k-elements (16 KiB,
// contiguous), ordered k-fastest inside a 256-row tile, so a workgroup streams one contiguous
// region per operand instead of 256 strided rows.  W and H_chunk are repacked (plain and
// transposed); the soft-max numerators are produced directly in that layout.  Short batches do not
// repack W (direct_tokens): the logits contraction reads its rows, the dH contraction reads them as a
// k-major operand.
#include "nat_internal.h"
#include "grpo_scalar.hip.h"
#include "row_stage.hip.h"
#include "walk.hip.h"

#include <type_traits>

namespace nat {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
// The soft-max numerators are written once and read back only by the two backward contractions,
// long after they have left the L2: non-temporal stores (logits of 8192 tokens
// at H = 4096 6990 -> 6929 us, of 16384 at H = 1024 4200 -> 4084).
#define NAT_E_STORE(ptr, val) __builtin_nontemporal_store((val), (ptr))

constexpr int kBM = 256, kBK = 32;                // block tile kBM x kBN: 4 wavefronts of 128 x 128, one per SIMD
constexpr int kGranule = 128;                     // vocabulary rows per soft-max partial
constexpr int kTileBytes = kBM * kBK * 2;         // 16 KiB per operand per stage
// LDS ring of k-slices: both operands' tiles, nb 32-row blocks of the second one; four of 32 KiB, or six where the second one's are narrow
constexpr int stage_bytes(int nb) { return kTileBytes + nb * 32 * kBK * 2; }
constexpr int ring_stages(int nb) { return nb <= 5 ? 6 : 4; }
// Tile rows per group of the block -> tile map, per contraction (whole step at the 8B head: logits in groups of 4 equal,
// of 16 3.4 % slower; dH and dW in groups of 8 1.5 % slower).
#ifndef NAT_GROUP_LOGITS
#define NAT_GROUP_LOGITS 8
#endif
#ifndef NAT_GROUP_DHIDDEN
#define NAT_GROUP_DHIDDEN 4
#endif
#ifndef NAT_GROUP_DWEIGHT
#define NAT_GROUP_DWEIGHT 4
#endif
constexpr int kMaxChunk = 32768;                  // most token rows per chunk (see recommended_cap)
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

// The 16-byte chunks of a 64-byte row (32 k) are stored permuted: chunk c at position c ^ chunk_xor(row / 4).  A wavefront
// reads a fragment of 16 rows with ds_read_b128, lane l chunk l / 16 of row l % 16; the LDS serves 16 lanes at a time over
// its 64 banks, lanes 0-3, 12-15, 20-27 together, then 4-11, 16-19, 28-31, and the same of the upper half.  Four rows
// apart the bank is the same, so the chunks of lanes 0-3, 12-15 (c ^ f(0), c ^ f(3)) and 20-23, 24-27 ((c + 1) ^ f(1), (c + 1)
// ^ f(2)) have to differ: f = 0, 2, 3, 1 does it (f = row / 4 itself: half of the LDS cycles were conflicts).
__host__ __device__ __forceinline__ constexpr int chunk_xor(int row4) { return (((row4 ^ (row4 >> 1)) & 1) << 1) | ((row4 >> 1) & 1); }

// element (row, k) of an operand with kb = K/32 k-slices.  With the chunks of a row permuted a block is
// a byte-for-byte image of the bank-conflict-free LDS tile, and the direct-to-LDS copy reads it
// linearly, 16 bytes per lane.
__host__ __device__ __forceinline__ int64_t blk_off(int row, int k, int kb) {
  return ((int64_t)(row >> 8) * kb + (k >> 5)) * kBlkElems + ((row & 255) << 5) +
         ((((k & 31) >> 3) ^ chunk_xor(row >> 2)) << 3) + (k & 7);
}

// element (row, k) of an operand in the blocked layout whose rows are read interleaved (16 lanes read rows 8 a + 4 p + b,
// a, b = 0..3): as blk_off, with the permutation by row / 8
__host__ __device__ __forceinline__ int64_t blk_off_interleaved(int row, int k, int kb) {
  return ((int64_t)(row >> 8) * kb + (k >> 5)) * kBlkElems + ((row & 255) << 5) +
         ((((k & 31) >> 3) ^ chunk_xor(row >> 3)) << 3) + (k & 7);
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
                    const float* __restrict__ row_scale) {     // row_scale: the chunk's rows, in order; none: W, interleaved
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
    if (out_rk && c < C) *reinterpret_cast<uint4*>(out_rk + blk_off_interleaved(r, c, C >> 5)) = x.q;
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
    const int64_t at = row_scale ? blk_off(c0 + cj, r0 + rbase, kb_cr) : blk_off_interleaved(c0 + cj, r0 + rbase, kb_cr);
    *reinterpret_cast<uint4*>(out_cr + at) = y.q;
  }
}

// ------------------------------------------------------------------- GEMM ----
struct GemmArgs {
  const uint16_t* A;          // [tiles_m * 256, K], stored as the kernel's Src says
  const uint16_t* B;          // [tiles_n * 256, K] in the blocked layout
  int K;                      // multiple of 2 * kBK
  int tiles_m, tiles_n;
  int group_m;                // tile rows walked together (see tile_of_block)
  int kb_a_src;               // k-major A only (see TileLoaderKMajor): k-slices of the source operand
  int kb_b;                   // k-slices of the B operand as it is stored (>= K / kBK)
  // k_splits > 1: the contraction axis of the last tail_tiles tiles in launch order (all of them when there are fewer
  // than compute units) is cut into k_splits ranges of kt_per_split k-slices, one workgroup per (tile, range); the
  // epilogue is told which slab its raw sums go to (position among the cut tiles * k_splits + range)
  int k_splits, kt_per_split, tail_tiles;
  int src_rows, src_cols;     // A read from a row-major matrix (TileLoaderRows, TileLoaderKMajorRows): its extent
  int walk;                   // kMany: most units per workgroup (walk_of)
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

// Global -> LDS copy of one [256][32] bf16 operand block (16 KiB, contiguous in memory)
// without staging registers: the 4 wavefronts issue 16 direct-to-LDS loads of 16 bytes per
// lane between them.  One instruction copies 1 KiB (16 tile rows) linearly: the hardware
// places lane l at byte 16*l of that KiB, and the block in memory already has the LDS tile's
// chunk order.
struct TileLoader {
  static constexpr int kLoads = kTileBytes / 1024 / 4;      // per wavefront
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
};

// kBlocks * 32 rows of a blocked operand from row `row0` on, a multiple of 16 (16 rows are one KiB of a block, and their chunk
// order repeats from one to the next): 2 * kBlocks KiB per slice, dealt to the 4 wavefronts; where that does not come out even the last
// one loads its last KiB again.
template <int kBlocks>
struct PartTileLoader {
  static constexpr int kPieces = 2 * kBlocks, kLoads = (kPieces + 3) / 4;
  const uint16_t* src[kLoads];
  static __device__ __forceinline__ int piece(int wave, int i) { const int q = wave * kLoads + i; return q < kPieces ? q : kPieces - 1; }
  __device__ __forceinline__ void init(const uint16_t* base, int row0, int kb, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int q = row0 / 16 + piece(wave, i);
      src[i] = base + (int64_t)(q >> 4) * kb * kBlkElems + (q & 15) * 512 + lane * 8;
    }
  }
  __device__ __forceinline__ void start_at(int kt0) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) src[i] += (int64_t)kt0 * kBlkElems;
  }
  template <int kIdx>
  __device__ __forceinline__ void issue_one(char* lds_tile, int kt, int wave) const {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[kIdx] + (int64_t)kt * kBlkElems),
                                     (__attribute__((address_space(3))) void*)(lds_tile + piece(wave, kIdx) * 1024), 16, 0, 0);
  }
};

// The same copy for an operand that is only stored with its rows along THIS contraction's k axis
// (the soft-max numerators: rows = token, k = vocabulary, read by the dW contraction whose k axis is
// the token).  A [256 rows][32 k] tile of the contraction is then eight pieces of the source, one per
// 32-row block of the tile: rows (kt % 8) * 32 .. + 31 of the source block (token tile kt / 8, k-slice
// 8 * tile + piece), 2 KiB contiguous each.  The LDS tile holds the pieces one after another, i.e.
// [row block][k][row within block], and fragments come out of it through the transposing LDS read.
struct TileLoaderKMajor {
  static constexpr int kLoads = kTileBytes / 1024 / 4;      // per wavefront
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
// p of a tile row holds chunk p ^ chunk_xor).  Rows past the end read the last row: as vocabulary rows
// of the logits tile they are masked by the epilogue, as k of the dH contraction they meet numerators that are 0.
struct TileLoaderRows {          // [256 rows][32 k]: rows of the matrix, k its columns
  static constexpr int kLoads = kTileBytes / 1024 / 4;
  const uint16_t* src[kLoads];   // this lane's chunk in k-slice 0 of each load
  __device__ __forceinline__ void init(const uint16_t* W, int tile, int rows, int ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int r = (wave * kLoads + i) * 16 + (lane >> 2), row = tile * kBM + r;
      src[i] = W + (int64_t)(row < rows ? row : rows - 1) * ld + (((lane & 3) ^ chunk_xor(r >> 3)) << 3);
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
};

struct TileLoaderKMajorRows {    // [256 rows][32 k] with k the rows of the matrix: pieces of 32 k x 32 rows, as TileLoaderKMajor
  static constexpr int kLoads = kTileBytes / 1024 / 4;
  const uint16_t* src;           // this lane's chunk of row 0 of the wavefront's first piece
  int piece_step;                // elements from the wavefront's first piece to its second
  int k_rows, ld, k_lane, kt_first;
  __device__ __forceinline__ void init(const uint16_t* W, int tile, int rows, int cols, int wave, int lane) {
    const int c0 = tile * kBM + 64 * wave, c1 = c0 + 32;         // columns past the end (a multiple of 64 is valid): any valid ones
    const int s0 = c0 < cols ? c0 : cols - 32, s1 = c1 < cols ? c1 : cols - 32;
    k_lane = lane >> 2;
    src = W + s0 + (((lane & 3) ^ chunk_xor(lane >> 4)) << 3);
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

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

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

// Four 16-byte reads, waited for: as inline assembly for the same reason.  (Accesses of one wavefront to LDS are in order: what it wrote before is read.)
__device__ __forceinline__ void lds_read_rows(const uint32_t (&addr)[4], f32x4 (&x)[4]) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]) : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]) : "memory");
}

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }

// one LDS object (with a second one the compiler's wait-count pass orders every fragment read behind all
// direct-to-LDS loads in flight): the ring, and behind it the words of the epilogue (parked across the k-loop, or staged)
template <int kWords, int kNB = 8>
struct GemmShared {
  char ring[ring_stages(kNB)][stage_bytes(kNB)];
  int words[4][kWords];          // per wavefront
};

// ---------------------------------------------------------------- GEMM core ----
// One workgroup computes a 256 x 256 tile of C = P . Q^T (P: rows of the result, Q: its columns, both along the
// contraction axis) with 4 wavefronts of 128 x 128 in 8 x 8 blocks of v_mfma_f32_16x16x32_bf16:
// acc[i][j] element r of lane l is C[p0 + row(i, l, r)][q0 + 16 j + l % 16], row = 16 i + 4 (l / 16) + r for an operand whose
// rows are in their order and 32 (i / 2) + 8 (l / 16) + 4 (i % 2) + r for one that is read with its rows interleaved
// (is_interleaved), so that a lane holds eight consecutive rows: a 16-byte store of bf16.
// Why 16 x 16 x 32: the three contractions run at the package's power limit, and this instruction needs less of it than
// 32 x 32 x 16 at the same peak (an accumulator is read and written once per 32 k instead of once per 16): operands in
// registers, nothing else going on, 1990 against 1755 TFLOP/s on normally distributed values, 1960 against 1710 with
// exponentials on one side, equal (2450) on zeros.

template <int kN, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (kN > 0) {
    static_for<kN - 1>(f);
    f(std::integral_constant<int, kN - 1>{});
  }
}

// how many of `count` things spread evenly over slots 0 .. span - 1 come before slot m
constexpr int spread(int m, int count, int span) { return m <= 0 ? 0 : m >= span ? count : (m * count + span - 1) / span; }

// How an operand is stored: blocked layout (rows in order or interleaved), rows of a row-major matrix (interleaved, read as
// it is), or either of them along the contraction's own axis (fragments through the transposing read).
enum class Src { kBlocked, kBlockedInterleaved, kRows, kKMajorBlocked, kKMajorRows };

constexpr bool is_kmajor(Src s) { return s == Src::kKMajorBlocked || s == Src::kKMajorRows; }
constexpr bool is_interleaved(Src s) { return s == Src::kBlockedInterleaved || s == Src::kRows; }

// Fragments of a wavefront's 16-row blocks out of an LDS tile: lane l gets row l % 16 of the block, k = 8 (l / 16) .. + 7.
template <Src kS>
struct FragReader {
  static constexpr int kReads = is_kmajor(kS) ? 2 : 1;          // LDS reads per fragment
  uint32_t off[is_kmajor(kS) ? 4 : 1];
  __device__ __forceinline__ void init(int row0, int lane) {    // row0: the wavefront's first row, a multiple of 16 (k-major: of 64)
    const int i = lane & 15, g = lane >> 4;
    if constexpr (is_kmajor(kS)) {
      // tile: [32-row piece][k = 32][32 rows], 16-byte chunks of a k-row XOR chunk_xor(k / 4).  Read q = 0, 1 of the block
      // with rows 16 h .. of its piece: the transposing read works on groups of 16 lanes, lane i of a group supplies the address
      // of 4 consecutive elements and receives element i % 4 of the lanes i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12.  With lane i pointing at
      // k = 8 g + 4 q + i / 4 and rows 16 h + 4 (i % 4) .. + 3 it gets row 16 h + i, k = 8 g + 4 q .. + 3.  The 32 lanes of a
      // half-wavefront cover all 64 banks once
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          off[2 * h + q] = row0 * 64 + (8 * g + 4 * q + (i >> 2)) * 64 + (((2 * h + ((i & 3) >> 1)) ^ chunk_xor(2 * g + q)) << 4) + (i & 1) * 8;
    } else if constexpr (is_interleaved(kS)) {
      off[0] = (row0 + 8 * (i >> 2) + (i & 3)) * 64 + ((g ^ chunk_xor(i >> 2)) << 4);
    } else {
      off[0] = (row0 + i) * 64 + ((g ^ chunk_xor(i >> 2)) << 4);
    }
  }
};

// c += a . b, the accumulator in the accumulation registers.  As inline assembly, because the allocator moves accumulators
// about between the two register files in the loop when it is given 64 of them through the builtin (several hundred
// moves per slice).  The compiler then does not know the instruction's wait states: a and b come from LDS reads that have
// been waited for, c is next touched by another product of the same kind, and the epilogues read it through AccReader,
// behind the wait states that a reader of the results needs.
template <bool kFirst>             // kFirst: c = a . b
__device__ __forceinline__ void mfma16(f32x4& c, const bf16x8& a, const bf16x8& b) {
  if constexpr (kFirst) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// Reads accumulators after the k-loop: the reads depend on `settled`, which the wait states produce, and take their operand
// from the accumulation registers as it is (copied out by the compiler all 256 would be wanted at once: spills).
struct AccReader {
  int settled;
  __device__ __forceinline__ AccReader() { asm volatile("s_nop 15\n\ts_nop 7\n\ts_mov_b32 %0, 0" : "=s"(settled)); }
  __device__ __forceinline__ float operator()(const f32x4& c, int r) const {
    float x;
    asm("v_accvgpr_read_b32 %0, %1 ; %2" : "=v"(x) : "a"(c[r]), "s"(settled));
    return x;
  }
  __device__ __forceinline__ f32x4 operator()(const f32x4& c) const {
    return f32x4{(*this)(c, 0), (*this)(c, 1), (*this)(c, 2), (*this)(c, 3)};
  }
  // c to LDS as it is
  __device__ __forceinline__ void stage(uint32_t addr, const f32x4& c) const {
    asm volatile("ds_write_b128 %0, %1 ; %2" : : "v"(addr), "a"(c), "s"(settled) : "memory");
  }
};

// The fragments of kN 16-row blocks.  Read r of the set is r-th in block order (two reads make a fragment of a k-major tile).
template <Src kS, int kN>
struct FragSet {
  static constexpr int kReads = kN * FragReader<kS>::kReads;
  typename std::conditional<is_kmajor(kS), s16x4, bf16x8>::type v[kReads];
  template <int kR>
  __device__ __forceinline__ void read(const FragReader<kS>& rd, const char* tile) {
    if constexpr (is_kmajor(kS)) v[kR] = lds_read_tr16_b64(lds_addr(tile) + rd.off[kR & 3], (kR >> 2) * 2048);
    else if constexpr (is_interleaved(kS)) v[kR] = *(const bf16x8*)(tile + rd.off[0] + (kR >> 1) * 2048 + (kR & 1) * 256);
    else v[kR] = *(const bf16x8*)(tile + rd.off[0] + kR * 1024);
  }
  template <int kB>
  __device__ __forceinline__ bf16x8 get() const {
    if constexpr (is_kmajor(kS)) {
      const s16x4 a = v[2 * kB], b = v[2 * kB + 1];
      const s16x8 both = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
      return __builtin_bit_cast(bf16x8, both);
    } else {
      return v[kB];
    }
  }
};

template <Src kS>
using LoaderOf = typename std::conditional<kS == Src::kRows, TileLoaderRows,
                 typename std::conditional<kS == Src::kKMajorBlocked, TileLoaderKMajor,
                 typename std::conditional<kS == Src::kKMajorRows, TileLoaderKMajorRows, TileLoader>::type>::type>::type;

// What one workgroup computes at a time: a tile (tm, tn), over slices kt0 .. kt0 + kt_n - 1 of the contraction axis; slab: where
// its raw sums go if that is one range of the axis (-1: the whole axis).
struct Unit { int tm, tn, kt0, kt_n, slab; };
__device__ __forceinline__ Unit unit_of(const GemmArgs& g, int id) {
  Unit u{0, 0, 0, g.K / kBK, -1};
  const int whole = g.tiles_m * g.tiles_n - g.tail_tiles;
  if (g.k_splits > 1 && id >= whole) {
    // ids congruent mod 8 share an L2, as in tile_of_block (whole is a multiple of 256): an XCD gets consecutive ranges, and of a range consecutive tiles,
    // so that the tiles of one range, which read the same slices of both operands, fetch them once.  dH, us, tile by tile over the XCDs / so: H =
    // 4096 150 tokens 290 / 233, 300 455 / 390, 560 663 / 627, H = 1024 300 155 / 115, 600 222 / 177.  dW, whose ranges read less in common, takes the same
    // time either way (H = 1024 to 5120, V = 9000 to 151936, 600 to 8192 tokens: 0 +/- 1.5 %)
    const int n = g.tail_tiles * g.k_splits, per = n / 8, r = id - whole;
    const int v = r < per * 8 ? (r & 7) * per + (r >> 3) : r, range = v / g.tail_tiles;
    int pos = v - range * g.tail_tiles;
    if (g.tail_tiles % 8 == 0) pos = pos % (g.tail_tiles / 8) * 8 + pos / (g.tail_tiles / 8);
    u.kt0 = range * g.kt_per_split;                            // with a blocked k-major A a multiple of 8 (TileLoaderKMajor::start_at)
    if (u.kt_n - u.kt0 > g.kt_per_split) u.kt_n = g.kt_per_split;
    else u.kt_n -= u.kt0;
    u.slab = pos * g.k_splits + range;
    id = whole + pos;
  }
  tile_of_block(g, id, u.tm, u.tn);
  return u;
}

// Units first, first + kNumCU, ... below end.  A is the operand of the tile grid's rows, B that of its columns.  kPIsB: the
// result's rows P are B's.  NB: 16-row blocks of B per wavefront, 8, or fewer for tiles with fewer columns: of a grid of columns that
// are kColumns wide, all of them or the first NB * 32 of 256.  kRing: the NB that the ring in LDS is laid out for.
//
// Software pipeline over k-slices of 32.  The n-th slice lives in ring buffer n % kS, kS = 4 or 6; its fragments are read into registers while
// slice n - 1 is multiplied.  At the barrier in front of slice n's products every wavefront has the fragments of slice
// n, so its buffer is refilled with slice n + kS under them, and slice n + 1 has landed: loads complete in issue order,
// hence a vmcnt that leaves slices n + 2 to n + kS - 1 outstanding (the epilogue's stores and loads count too: then it waits for
// more than that, never for less).  The number of slices of a unit is even (H is a multiple of 64, the vocabulary and the
// tokens are padded, ranges start and end at even slices): two per turn of the loop.  The slices of a workgroup's
// units follow one another: while the last ones of a unit are multiplied and its epilogue runs, the first ones of the next are
// loaded (kMany; without it there is one unit, and neither the bookkeeping nor a first pair of slices of its own that starts
// from zero: 1 % on dH's thousands of slices, 0.7 % on logits of 112 to 160; dW of 512 slices took 14523 us without and 14489 with
// it).  Past the last unit the last two slices are loaded again (into buffers nobody reads), so that the body is free of
// branches and the count fixed.  The 8 x NB products of a slice are written slot by slot (the compiler may not move anything
// across a slot's end): fragment reads behind the products of the first half, one every second of them, loads of the refill
// evenly spaced behind the second half.
template <class Epilogue, Src kA, Src kB, bool kPIsB, bool kMany, int NB, int kColumns = kBN, int kRing = 8>
__device__ __forceinline__ void mfma_units(const GemmArgs& g, const Epilogue& epi, GemmShared<Epilogue::kWords, kRing>& sm, int first, int end) {
  constexpr int NP = kPIsB ? NB : 8, NQ = kPIsB ? 8 : NB;
  static_assert(kColumns == kBN || !kPIsB, "narrow columns of the tile grid are the result's");
  using LoadA = LoaderOf<kA>;
  using LoadB = typename std::conditional<NB < 8, PartTileLoader<NB>, LoaderOf<kB>>::type;
  constexpr int kLoadsA = LoadA::kLoads, kLoadsB = LoadB::kLoads, kLoads = kLoadsA + kLoadsB;    // per wavefront and slice
  using std::integral_constant;
  constexpr integral_constant<int, 0> zero{};
  constexpr integral_constant<int, 1> one{};
  constexpr int kS = ring_stages(kRing), kAhead = kS / 2 - 1;  // ring buffers; pairs of slices that stay in flight
  auto a_buf = [&](int st) { return &sm.ring[st][0]; };
  auto b_buf = [&](int st) { return &sm.ring[st][kTileBytes]; };
  auto pair_after = [](int st) { return kS == 4 ? st ^ 2 : st + 2 == kS ? 0 : st + 2; };
  auto pair_before = [](int st) { return kS == 4 ? st ^ 2 : st == 0 ? kS - 2 : st - 2; };
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int a_row0 = (wave >> 1) * 128, b_row0 = (wave & 1) * (NB * 16);

  // the loading side: slice `slice` and the one behind it of a unit of `slices` are loaded next
  LoadA la;
  LoadB lb;
  int load_id = first, slice = 0, slices;
  LoadB lb_last;                                               // kPaired: B of the slice loaded last comes with the next even one
  int slice_last;
  auto open = [&] {
    const Unit u = unit_of(g, load_id);
    if constexpr (kA == Src::kRows || kA == Src::kKMajorRows) la.init(g.A, u.tm, g.src_rows, g.src_cols, wave, lane);
    else la.init(g.A, u.tm, kA == Src::kKMajorBlocked ? g.kb_a_src : g.K / kBK, wave, lane);
    lb.init(g.B, NB < 8 ? u.tn * kColumns : u.tn, g.kb_b, wave, lane);
    la.start_at(u.kt0);
    lb.start_at(u.kt0);
    slice = 0;
    slices = u.kt_n;
  };
  auto advance = [&] {
    lb_last = lb;
    slice_last = slice + 1;
    slice += 2;
    if constexpr (kMany) {
      if (slice < slices) return;
      slice = slices - 2;
      if (load_id + kNumCU >= end) return;
      load_id += kNumCU;
      open();
    } else {
      slice = slice < slices ? slice : slices - 2;
    }
  };
  auto load_a = [&](auto idx, int st, int k) { la.template issue_one<decltype(idx)::value>(a_buf(st), k, wave); };
  auto load_b = [&](auto idx, int st, int k) { lb.template issue_one<decltype(idx)::value>(b_buf(st), k, wave); };
  // Load n of the next two slices into buffers st and st + 1: first kEven with the even one, then kOdd.  A slice of an A read
  // from rows is 64 bytes of a row, half a cache line; fetched a slice apart, the halves cost the line twice on the way from
  // the L2 (log-probs of 12288 tokens at H = 4096 10454 us, 10163 together; 2048 1824 / 1766, at H = 1024 519 / 504): both slices'
  // A tiles go with the odd one, half after half, and B's odd tile with the next even one, 8 loads each.
  constexpr bool kPaired = kA == Src::kRows;
  constexpr int kEven = kPaired ? 2 * kLoadsB : kLoads, kOdd = kPaired ? 2 * kLoadsA : kLoads;
  auto load_even = [&](auto n, int st) {
    constexpr int i = decltype(n)::value;
    if constexpr (kPaired && i < kLoadsB) lb_last.template issue_one<i>(b_buf(pair_before(st) + 1), slice_last, wave);
    else if constexpr (kPaired) load_b(integral_constant<int, i - kLoadsB>{}, st, slice);
    else if constexpr (i < kLoadsA) load_a(n, st, slice);
    else load_b(integral_constant<int, i - kLoadsA>{}, st, slice);
  };
  auto load_odd = [&](auto n, int st) {
    constexpr int i = decltype(n)::value;
    if constexpr (kPaired) load_a(integral_constant<int, i / 2>{}, st + (i & 1), slice + (i & 1));
    else if constexpr (i < kLoadsA) load_a(n, st + 1, slice + 1);
    else load_b(integral_constant<int, i - kLoadsA>{}, st + 1, slice + 1);
  };
  // loads younger than the slice that has to have landed in front of an even and an odd slice's products
  constexpr int kYoungEven = kPaired ? 2 * kAhead * kLoadsA + (2 * kAhead - 1) * kLoadsB : 2 * kAhead * kLoads;
  constexpr int kYoungOdd = kPaired ? 2 * (kAhead - 1) * kLoadsA + 2 * kAhead * kLoadsB : 2 * kAhead * kLoads;

  FragReader<kA> ra;
  FragReader<kB> rb;
  ra.init(a_row0, lane);
  rb.init(b_row0, lane);
  FragSet<kA, 8> fa[2];
  FragSet<kB, NB> fb[2];
  constexpr int kReadsA = FragSet<kA, 8>::kReads, kReads = kReadsA + FragSet<kB, NB>::kReads;
  f32x4 acc[NP][NQ];

  // products of the slice whose fragments are in set kCur; between them the fragments of the next one from ring buffer
  // `next` into the other set and load(n), n = 0 .. kN - 1
  auto products = [&](auto is_first, auto cur, int next, auto count, auto load) {
    constexpr bool kFirst = decltype(is_first)::value;
    constexpr int kCur = decltype(cur)::value, kN = decltype(count)::value, kSlots = 8 * NB, kReadSpan = kSlots / 2;
    const char *a_tile = a_buf(next), *b_tile = b_buf(next);
    static_for<kSlots>([&](auto slot) {
      constexpr int m = decltype(slot)::value, i = m / NB, j = (i & 1) ? NB - 1 - m % NB : m % NB;
      if constexpr (kPIsB) mfma16<kFirst>(acc[j][i], fb[kCur].template get<j>(), fa[kCur].template get<i>());
      else mfma16<kFirst>(acc[i][j], fa[kCur].template get<i>(), fb[kCur].template get<j>());
      constexpr int r0 = spread(m, kReads, kReadSpan), r1 = spread(m + 1, kReads, kReadSpan);
      static_for<r1 - r0>([&](auto read) {
        constexpr int r = r0 + decltype(read)::value;
        if constexpr (r < kReadsA) fa[1 - kCur].template read<r>(ra, a_tile);
        else fb[1 - kCur].template read<r - kReadsA>(rb, b_tile);
      });
      constexpr int n0 = spread(m - kReadSpan, kN, kSlots - kReadSpan), n1 = spread(m + 1 - kReadSpan, kN, kSlots - kReadSpan);
      static_for<n1 - n0>([&](auto n) { load(std::integral_constant<int, n0 + decltype(n)::value>{}); });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // between two slices: this wavefront's fragments are in its registers and its share of all but the `young` youngest
  // loads has landed; the barrier covers the others' shares
  auto turn = [&](auto young) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(decltype(young)::value) & 0xf0ff);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  // what the epilogue needs per column (token id, exponent shift): fetched into LDS ahead of the operands, read after the
  // k-loop
  Unit u = unit_of(g, first);
  auto prefetch = [&] { epi.template prefetch<NQ>(sm.words[wave], kPIsB ? u.tm * kBM + a_row0 : u.tn * kColumns + b_row0, lane); };
  prefetch();
  open();
  if constexpr (kPaired) {
#pragma unroll
    for (int st = 0; st < kS; st += 2) {
      static_for<kOdd>([&](auto n) { load_odd(n, st); });
      static_for<kLoadsB>([&](auto n) { load_b(n, st, slice); });
      if (st + 2 < kS) static_for<kLoadsB>([&](auto n) { load_b(n, st + 1, slice + 1); });
      advance();
    }
    turn(integral_constant<int, 2 * kAhead * (kLoadsA + kLoadsB)>{});
  } else {
#pragma unroll
    for (int st = 0; st < kS; st += 2) {
      static_for<kEven>([&](auto n) { load_even(n, st); });
      static_for<kOdd>([&](auto n) { load_odd(n, st); });
      advance();
    }
    turn(integral_constant<int, (kS - 1) * kLoads>{});
  }
  static_for<kReadsA>([&](auto r) { fa[0].template read<decltype(r)::value>(ra, a_buf(0)); });
  static_for<kReads - kReadsA>([&](auto r) { fb[0].template read<decltype(r)::value>(rb, b_buf(0)); });
  turn(integral_constant<int, kYoungEven>{});
  int st = 0;                                                  // ring buffer of the slice that is multiplied next
  for (int id = first;;) {
    __builtin_amdgcn_s_waitcnt(0xc07f);                        // lgkmcnt(0): else the compiler waits for scalar loads inside the loop
    auto two_slices = [&](auto is_first) {
      products(is_first, zero, st + 1, integral_constant<int, kEven>{}, [&](auto n) { load_even(n, st); });
      turn(integral_constant<int, kYoungOdd>{});
      products(std::false_type{}, one, pair_after(st), integral_constant<int, kOdd>{}, [&](auto n) { load_odd(n, st); });
      turn(integral_constant<int, kYoungEven>{});
      st = pair_after(st);
      advance();
    };
    if constexpr (kMany) {
      two_slices(std::true_type{});
      for (int kt = 2; kt < u.kt_n; kt += 2) two_slices(std::false_type{});
    } else {
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int j = 0; j < NQ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int kt = 0; kt < u.kt_n; kt += 2) two_slices(std::false_type{});
    }
    // with more slices in flight than a unit of two has, what its prefetch() fetched may be among them
    if constexpr (kMany && kAhead > 1)
      if (u.kt_n == 2) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kLoads));
    const AccReader rd;
    epi(acc, rd, kPIsB ? u.tn * kBN + b_row0 : u.tm * kBM + a_row0, kPIsB ? u.tm * kBM + a_row0 : u.tn * kColumns + b_row0, lane, sm.words[wave], u.slab);
    id += kNumCU;
    if (!kMany || id >= end) break;
    u = unit_of(g, id);
    prefetch();
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // no direct-to-LDS load may outlive this
  __syncthreads();
}

template <class Epilogue, Src kA, Src kB, bool kPIsB, bool kMany, int NB = 8>
__global__ void __launch_bounds__(256, 1)
mfma_nt_kernel(GemmArgs g, Epilogue epi) {
  __shared__ __attribute__((aligned(1024))) GemmShared<Epilogue::kWords, NB> sm;
  if constexpr (kMany) {
    const Walk w = walk_of((int)blockIdx.x, g.walk, g.tiles_m * g.tiles_n + (g.k_splits - 1) * g.tail_tiles);
    mfma_units<Epilogue, kA, kB, kPIsB, true, NB, NB * 32, NB>(g, epi, sm, w.first, w.end);
  } else if constexpr (NB < 8) {
    mfma_units<Epilogue, kA, kB, kPIsB, false, NB, NB * 32, NB>(g, epi, sm, (int)blockIdx.x, (int)blockIdx.x + 1);
  } else {
    const int id = (int)blockIdx.x;
    // Where W is read as it is the batch is short and the columns are its tokens: a last tile with at most 128 or 64 of them
    // computes only those (where the columns are not all narrower, logits_columns_pay and dh_columns_pay.  Loss at the 8B head, 1100 tokens, with 256 /
    // 128 columns 3557 / 3479 us).
    if constexpr (kA == Src::kRows || kA == Src::kKMajorRows) {
      const int blocks = last_blocks(epi.n_valid, g.tiles_n);
      if (blocks < 8 && unit_of(g, id).tn == g.tiles_n - 1) {
        if (blocks == 2) mfma_units<Epilogue, kA, kB, kPIsB, false, 2>(g, epi, sm, id, id + 1);
        else mfma_units<Epilogue, kA, kB, kPIsB, false, 4>(g, epi, sm, id, id + 1);
        return;
      }
    }
    mfma_units<Epilogue, kA, kB, kPIsB, false, 8>(g, epi, sm, id, id + 1);
  }
}

// ------------------------------------------------------------- epilogues ----

// sum of a value over the lanes l % 16 + 16 q, q = 0..3
__device__ __forceinline__ float sum_quarters(float x) {
  uint32_t a = __builtin_bit_cast(uint32_t, x);
  const auto q = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  a = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, (uint32_t)q[0]) + __builtin_bit_cast(float, (uint32_t)q[1]));
  const auto h = __builtin_amdgcn_permlane32_swap(a, a, false, false);
  return __builtin_bit_cast(float, (uint32_t)h[0]) + __builtin_bit_cast(float, (uint32_t)h[1]);
}

// Logits tile: rows = vocabulary (A = W), columns = tokens of the chunk (B = H_chunk).
template <bool kEntropy, bool kStoreE = true>
struct LogitsEpilogue {
  int V, n_valid;                  // vocabulary size, valid tokens in the chunk
  int64_t ld_part;                 // leading dimension (tokens) of the partial sums
  int kb_z;                        // k-slices of Eb (Vp / 32)
  uint16_t* Eb;                    // blocked, rows = token, k = vocabulary: E = exp(z - ref), stored once
  static constexpr int kWords = 256;
  float* s_part;                   // [Vp/128, ld_part] partial sums of E
  float* t_part;                   // [Vp/128, ld_part] partial sums of E (z - ref) (entropy), kEntropy only
  float* z_target;                 // [ld_part] exact target logits
  const int32_t* ids;              // target ids of the chunk's tokens
  const float* ref;                // [ld_part] exponent shift per token

  // The per-column scalars the epilogue needs (token id, exponent shift) are fetched before the k-loop
  // straight into LDS (direct-to-LDS loads of 4 bytes per lane, from a clamped index; n_valid >= 1 in
  // every launch) and read back after it: they wait for nothing, hold no registers across the loop, and
  // are older than every operand load, so the loop's load counting is unchanged.  words: this wavefront's, ids in the first
  // 128, shifts in the others.
  template <int NQ>
  __device__ __forceinline__ void prefetch(int* words, int k0, int lane) const {
#pragma unroll
    for (int i = 0; i < (NQ + 3) / 4; ++i) {
      const int kk = k0 + i * 64 + lane;
      const int kc = kk < n_valid ? kk : n_valid - 1;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(ids + kc),
                                       (__attribute__((address_space(3))) void*)(words + i * 64), 4, 0, 0);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(ref + kc),
                                       (__attribute__((address_space(3))) void*)(words + 128 + i * 64), 4, 0, 0);
    }
  }

  // acc: rows = vocabulary, interleaved: element r of acc[2 j + p][nb] in lane l is entry v0 + 32 j + 8 (l / 16) + 4 p + r of
  // token k0 + 16 nb + l % 16
  template <int NQ>
  __device__ __forceinline__ void operator()(const f32x4 (&acc)[8][NQ], const AccReader& rd, int v0, int k0, int lane, const int* words, int) const {
    const int l15 = lane & 15, g = lane >> 4;
    const int granule = v0 / kGranule;
    const bool all_rows_valid = v0 + kGranule <= V;
    constexpr float kLog2e = 1.44269504088896340736f, kLn2 = 0.69314718055994530942f;

    int y_of[NQ];                  // target id of this lane's token per column block; -1: padding column, or
    float shift_of[NQ];            // an id outside the vocabulary (matches no row)
#pragma unroll
    for (int nb = 0; nb < NQ; ++nb) {
      const bool tok_valid = k0 + nb * 16 + l15 < n_valid;
      const int y = words[nb * 16 + l15];
      y_of[nb] = (tok_valid && y >= 0 && y < V) ? y : -1;
      shift_of[nb] = tok_valid ? __builtin_bit_cast(float, words[128 + nb * 16 + l15]) : 0.f;
    }

    // exact target logit, if the target row lies in this granule and in this lane's quarter
#pragma unroll
    for (int nb = 0; nb < NQ; ++nb) {
      const int yrel = y_of[nb] - v0;
      if (__any(yrel >= 0 && yrel < kGranule)) {
        if (yrel >= 0 && yrel < kGranule && ((yrel >> 3) & 3) == g) {
          float zt = 0.f;
#pragma unroll
          for (int mb = 0; mb < 8; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float z = rd(acc[mb][nb], r);
              zt = yrel == (mb >> 1) * 32 + 8 * g + 4 * (mb & 1) + r ? z : zt;
            }
          z_target[k0 + nb * 16 + l15] = zt;
        }
      }
    }

    // One pass over the accumulators, 16 token columns (all 128 vocabulary rows of the wavefront) at a
    // time: E = exp(min(z - shift, 70)) as 2^(z * log2(e) - shift * log2(e)) (one fma and the hardware exponential per
    // logit, eight at a time with independent temporaries), its running sums, and at once the store.  The bound of 70 acts
    // on hardly any tile: where the sums show that it would (an exponential at or above e^70, an infinity or NaN among them
    // makes them that large), the wavefront makes the pass again with it.  (One minimum less per logit: logits of 16384 tokens at H = 1024 4040
    // -> 3966 us, log-probs of 8192 there 1886 -> 1845, of 4000 at H = 256 389 -> 369.  Where one token in 128 or all are beyond the bound, every
    // pass is made twice: 4000 tokens at H = 256 485, 8192 at H = 1024 2067, at H = 4096 6956 against 6775 with the minimum.)  E is stored once, rows = token, k = vocabulary (the
    // dH contraction reads it as it is, the dW contraction through the transposing LDS read): the rows of W are read
    // interleaved, so a lane holds 8 consecutive vocabulary entries of its token, one 16-byte chunk of the blocked layout,
    // and an instruction stores 1 KiB (16 token rows of one 32-wide vocabulary slice) contiguous.
    float total = 0.f;
    auto sweep = [&](auto clamped) {
      constexpr bool kClamp = decltype(clamped)::value;
#pragma unroll
      for (int nb = 0; nb < NQ; ++nb) {
        const float nshift2 = -shift_of[nb] * kLog2e;
        uint16_t* e_row = kStoreE ? Eb + blk_off(k0 + nb * 16 + l15, v0 + 8 * g, kb_z) : nullptr;
        float s2[2] = {0.f, 0.f}, t2[2] = {0.f, 0.f};      // two independent chains per sum
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float x2[8], e[8];
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            x2[r] = fmaf(rd(acc[2 * j + (r >> 2)][nb], r & 3), kLog2e, nshift2);
            if (kClamp) x2[r] = fminf(x2[r], 70.f * kLog2e);
          }
#pragma unroll
          for (int r = 0; r < 8; ++r) e[r] = __builtin_amdgcn_exp2f(x2[r]);
          if (!all_rows_valid) {                           // only the last vocabulary tile pays for the row check
#pragma unroll
            for (int r = 0; r < 8; ++r)
              if (v0 + j * 32 + 8 * g + r >= V) e[r] = x2[r] = 0.f;    // x2 too: it may be infinite or NaN, and no sum would tell
          }
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            s2[r & 1] += e[r];
            if (kEntropy) t2[r & 1] = fmaf(e[r], x2[r], t2[r & 1]);
          }
          if (kStoreE) {
            u32x4v w;
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = pack_bf16x2(e[2 * r], e[2 * r + 1]);
            NAT_E_STORE((u32x4v*)(e_row + j * kBlkElems), w);
          }
        }
        const int kk = k0 + nb * 16 + l15;                 // token column (always inside the padded chunk)
        if (!kClamp) total += s2[0] + s2[1];
        const float sum = sum_quarters(s2[0] + s2[1]);
        if (g == 0) s_part[(int64_t)granule * ld_part + kk] = sum;
        if (kEntropy) {
          const float t = sum_quarters((t2[0] + t2[1]) * kLn2);  // back to natural-log units
          if (g == 0) t_part[(int64_t)granule * ld_part + kk] = t;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    sweep(std::false_type{});
    constexpr float kBelowClamp = 1e30f;                   // < e^70: no exponential of a smaller sum was above the bound
    if (__builtin_expect(__any(!(total < kBelowClamp)), 0)) sweep(std::true_type{});
  }
};

// dH tile: rows = hidden units (W^T, either interleaved or, when W is read as it is, k-major in order), columns = tokens of
// the chunk (E); columns scaled by beta.  A lane holds its token's hidden units h0 + 32 j + 8 (l / 16) .. + 7 in acc[2 j], acc[2 j + 1]
// (interleaved: one 16-byte store, 64 bytes of 16 token rows per instruction) or h0 + 16 i + 4 (l / 16) .. + 3 in acc[i].
template <bool kInterleaved>
struct DHiddenEpilogue {
  static constexpr int kWords = 1;
  int n_valid, H;
  uint16_t* dH;                    // rows of this chunk, [n_valid, H] bf16
  const float* beta;               // [n_valid]
  float* partial;                  // tiles whose contraction is cut into ranges: [slab][256 tokens][256 hidden] fp32 raw sums

  template <int NQ> __device__ __forceinline__ void prefetch(int*, int, int) const {}
  template <int NQ>
  __device__ __forceinline__ void operator()(const f32x4 (&acc)[8][NQ], const AccReader& rd, int h0, int k0, int lane, const int*, int slab_id) const {
    const int l15 = lane & 15, g = lane >> 4;
    if (slab_id >= 0) {            // this workgroup's range of the vocabulary: the raw sums go to its slab
      float* slab = partial + (int64_t)slab_id * (kBM * kBN) + (h0 & (kBM - 1));
#pragma unroll
      for (int nb = 0; nb < NQ; ++nb) {
        const int k = k0 + nb * 16 + l15;
        if (k >= n_valid) continue;                            // padding rows of a short batch are not read back
#pragma unroll
        for (int i = 0; i < 8; ++i)
          *(f32x4*)(slab + (k & (kBN - 1)) * kBM + (kInterleaved ? (i >> 1) * 32 + 8 * g + 4 * (i & 1) : i * 16 + 4 * g)) = rd(acc[i][nb]);
      }
      return;
    }
    float betas[NQ];               // all at once: block by block each waits for memory (8 tiles of 32 slices 27.3 us, 25.3 so)
#pragma unroll
    for (int nb = 0; nb < NQ; ++nb) betas[nb] = k0 + nb * 16 + l15 < n_valid ? beta[k0 + nb * 16 + l15] : 0.f;
#pragma unroll
    for (int nb = 0; nb < NQ; ++nb) {
      const int k = k0 + nb * 16 + l15;
      const bool ok = k < n_valid;
      const float b = betas[nb];
      uint16_t* row = dH + (int64_t)k * H + h0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 lo = rd(acc[2 * j][nb]), hi = rd(acc[2 * j + 1][nb]);
        const uint2 wl = make_uint2(pack_bf16x2(b * lo[0], b * lo[1]), pack_bf16x2(b * lo[2], b * lo[3]));
        const uint2 wh = make_uint2(pack_bf16x2(b * hi[0], b * hi[1]), pack_bf16x2(b * hi[2], b * hi[3]));
        if (!ok || h0 + 32 * j >= H) continue;                 // H is a multiple of 64: 32 units are in or out
        if (kInterleaved) {
          *(uint4*)(row + 32 * j + 8 * g) = make_uint4(wl.x, wl.y, wh.x, wh.y);
        } else {
          *(uint2*)(row + 32 * j + 4 * g) = wl;
          *(uint2*)(row + 32 * j + 16 + 4 * g) = wh;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// dW tile: rows = hidden units ((diag(beta) H_chunk)^T), columns = vocabulary (E^T): a lane holds hidden units h0 + 16 i + 4 (l / 16)
// .. + 3 of its vocabulary entry.  Stored from there an instruction writes half a cache line of 16 rows, and a tile's 256 KiB leave its compute unit at
// 16 bytes a cycle (16 k cycles, 27 k when accumulating, beside 1090 per k-slice): a wavefront's results go through LDS, 16 vocabulary entries x 64 hidden
// units at a time, and leave as 256 bytes of four rows per instruction.  From registers / so, us: 8 tiles of 8 slices 14.7 / 11.0; 200 tokens at H = 1024, V =
// 160000 184 / 159; H = 4096, V = 151936: 300 632 / 608, 1237 accumulating 1773 / 1611, 16384 accumulating 14931 / 14966.
// A dW beyond the Infinity Cache (kDWeightStreamBytes) is read and written past the caches: nothing of it is there when it is next wanted, and
// what it would push out is W, and the numerators of this launch.  Cached / past, whole call at H = 4096, V = 151936, us: 300 tokens 1537 / 1466, 1237 3663 /
// 3636, twice 1237 (the second accumulating) 7580 / 7502, twice 60 2452 / 2303, 32768 82170 / 82054.  Where the line lies: whole calls of 40 / 600 tokens past the
// caches against cached, per cent, overwriting and accumulating: H = 1024, 41 MB -5 / -1, +6 / +5; 82 MB +3 / +2, +12 / +7; 131 MB +4 / 0, +7 / -3; 184 MB 0 / -6, -2 / -5; 246 MB
// -7 / -9, -13 / -5; 307 MB -15 / -6, -15 / -3; H = 4096, 164 MB -2 / -7, -10 / -6; 246 MB -17 / -10, -16 / -8; 328 MB -21 / -7, -10 / -5.  Above 256 MiB past the caches was never
// slower; between 180 MB and the line it would be faster too.
constexpr int64_t kDWeightStreamBytes = int64_t(256) << 20;
template <bool kAccumulate>
struct DWeightEpilogue {
  static constexpr int kWords = kStageFloats;
  int V, H;
  bool stream;                     // dW past the caches
  float* dW;                       // [V, H] fp32
  float* partial;                  // tiles whose contraction is cut into ranges: [slab][256][256] fp32 raw sums

  template <int NQ> __device__ __forceinline__ void prefetch(int*, int, int) const {}
  __device__ __forceinline__ void operator()(const f32x4 (&acc)[8][8], const AccReader& rd, int h0, int v0, int lane, const int* words, int slab_id) const {
    asm volatile("" : "+v"(lane)); // else all that is formed from it is kept across the walk, and spilled
    uint32_t write[4], read[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      write[i] = lds_addr(words) + 4 * stage_write_at(lane, i);
      read[i] = lds_addr(words) + 4 * stage_read_at(lane, i);
    }
    // to dst: this wavefront's [128 vocabulary entries][128 hidden units], a row `ld` elements, rows x cols of them valid (cols a multiple of 64).  One owner
    // per element and launch, launches in stream order: one fp32 addition old + sum per element.  Old values are loaded a step ahead.
    auto sweep = [&](auto all_valid, auto add, auto past_caches, float* dst, int ld, int rows, int cols) {
      constexpr bool kAll = decltype(all_valid)::value, kAdd = decltype(add)::value, kStream = decltype(past_caches)::value;
      auto ok = [&](int step, int j) { return kAll || ((step & 7) * 16 + stage_read_row(lane, j) < rows && (step >> 3) * 64 < cols); };
      const uint32_t lane_bytes = 4u * (uint32_t)(stage_read_row(lane, 0) * ld + stage_read_column(lane));     // the rest of an address is the wavefront's
      auto at = [&](int step, int j) {
        return (f32x4*)((char*)(dst + (int64_t)((step & 7) * 16 + stage_read_row(0, j)) * ld + (step >> 3) * 64) + lane_bytes);
      };
      f32x4 old[2][4];
      auto fetch = [&](int step) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (ok(step, j)) old[step & 1][j] = kStream ? __builtin_nontemporal_load(at(step, j)) : *at(step, j);
          else old[step & 1][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      };
      if (kAdd) fetch(0);
#pragma unroll
      for (int step = 0; step < 16; ++step) {
        if (!kAll && (step >> 3) * 64 >= cols) break;
        if (kAdd && step < 15) fetch(step + 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) rd.stage(write[i], acc[(step >> 3) * 4 + i][step & 7]);
        f32x4 x[4];
        lds_read_rows(read, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (kAdd) x[j] = old[step & 1][j] + x[j];
          if (!ok(step, j)) continue;
          if (kStream) __builtin_nontemporal_store(x[j], at(step, j));
          else *at(step, j) = x[j];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (slab_id >= 0) {            // one range of this tile's tokens: raw sums to the slab, added up by dw_tail_reduce_kernel
      sweep(std::true_type{}, std::false_type{}, std::false_type{}, partial + (int64_t)slab_id * (kBM * kBN) + (v0 & (kBM - 1)) * kBN + (h0 & (kBN - 1)), kBN, 128, 128);
      return;
    }
    if (v0 >= V) return;
    float* dst = dW + (int64_t)v0 * H + h0;
    constexpr std::bool_constant<kAccumulate> add{};
    if (V - v0 < 128 || h0 + 128 > H) sweep(std::false_type{}, add, std::false_type{}, dst, H, V - v0, H - h0);
    else if (stream) sweep(std::true_type{}, add, std::true_type{}, dst, H, 128, 128);
    else sweep(std::true_type{}, add, std::false_type{}, dst, H, 128, 128);
  }
};

// dH tiles of a launch whose last tail_tiles tiles (in launch order) were cut into k_splits ranges of the vocabulary:
// dH[k][h] = beta_k * (slab 0 + slab 1 + ...) of the tile, in range order.  One block per 1024 elements of a tile.
__global__ void __launch_bounds__(256)
dh_tail_reduce_kernel(const float* __restrict__ partial, GemmArgs g, bool transposed, int columns /*tokens of a tile*/, const float* __restrict__ beta,
                      int n_valid, int H, uint16_t* __restrict__ dH) {
  const int pos = blockIdx.y;
  int tm, tn;                                                          // tile of tokens, of hidden units
  if (transposed) tile_of_block(g, g.tiles_m * g.tiles_n - g.tail_tiles + pos, tn, tm);
  else tile_of_block(g, g.tiles_m * g.tiles_n - g.tail_tiles + pos, tm, tn);
  const int e = (blockIdx.x * 256 + threadIdx.x) * 4;                  // four hidden units of a token
  const int row = e / kBN, k = tm * columns + row, h = tn * kBN + e % kBN;
  if (row >= columns || k >= n_valid || h >= H) return;                // H is a multiple of 64
  const float* slab = partial + (int64_t)pos * g.k_splits * (kBM * kBN) + (k & (kBM - 1)) * kBN + e % kBN;
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
// does not depend on timing.  Bound by the latency of the walk (75 granules per group at V = 151936) in a short batch: 32
// loads in flight (3000 tokens in 8 groups 14 us, 19 with 8 loads), and 16 groups (8 / 16 / 32: 40 tokens with the entropy at V = 160000 18.1 / 12.6 /
// 12.5 us, 1237 tokens 13.9 / 12.1 / 12.1, 16384 21.6 / 21.8 / 24.8).  Returns to the first kStatTokens threads only.
constexpr int kStatTokens = 32, kStatParts = 16, kStatBatch = 32;
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
  auto tree = [&](const float (&x)[kStatParts][kStatTokens]) {
    float v[kStatParts];
#pragma unroll
    for (int q = 0; q < kStatParts; ++q) v[q] = x[q][t];
#pragma unroll
    for (int n = kStatParts / 2; n > 0; n /= 2)
#pragma unroll
      for (int q = 0; q < n; ++q) v[q] = v[2 * q] + v[2 * q + 1];
    return v[0];
  };
  out.S = tree(sh.s);
  out.TZ = tree(sh.t);
  float m = sh.m[0][t];
  for (int q = 1; q < kStatParts; ++q) m = fmaxf(m, sh.m[q][t]);
  out.in_shift_range = m >= kShiftRangeLimit;
  return out;
}

__global__ void __launch_bounds__(kStatTokens * kStatParts)
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
    // the scalar part of a token in fp64: a log-prob of 12 formed from fp32 numbers is rounded three times by up to 5e-7,
    // and that is what a loss whose terms cancel was off by
    const double log_S = log((double)S);
    if (entropy_out) entropy_out[k] = (float)(log_S - (double)sums.TZ / (double)S);   // -sum_v p_v log p_v, p_v = E_v / S
    if (bad_id) {                                        // left out: no loss term, zero gradient
      beta_out[kk] = 0.f;
      if (logp_out) logp_out[k] = __builtin_nanf("");
      if (kl_out) kl_out[k] = __builtin_nanf("");
      term[k] = 0.f;
    } else {
      const double logp = (double)z_target[kk] - ((double)ref[kk] + log_S);
      const float w = kept_w[k];
      const float A = adv[kept_seq[k]];
      const TokenScalars ts = grpo_token_scalars(logp, old_logp[k], A, w, eps_lo, eps_hi, grad_scale,
                                                 klp.beta, klp.kind, klp.beta != 0.f ? klp.ref_logp[k] : 0.f);
      clipped = ts.clipped;
      nonzero_adv = A != 0.f;
      beta_out[kk] = -ts.c / S;                          // dz_kv = beta_k E_kv off the target
      // the target entry of E is replaced by E' with beta_k E' = c_k (1 - p_target): the two backward
      // contractions then need no separate one-hot term
      Eb[blk_off(kk, y, kb_z)] = f32_to_bf16_bits(-S * (1.f - __expf((float)logp)));
      if (logp_out) logp_out[k] = (float)logp;
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
__global__ void __launch_bounds__(kStatTokens * kStatParts)
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
    const double log_S = log((double)sums.S);          // in fp64, as in token_stats_kernel
    logp_out[k] = bad_id ? __builtin_nanf("") : (float)((double)z_target[kk] - ((double)ref[kk] + log_S));
    if (entropy_out) entropy_out[k] = (float)(log_S - (double)sums.TZ / (double)sums.S);
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
// contraction axis is the chunk, gains nothing beyond 16384 (whole step at the 8B head 355.5 ms, 355.3 at 24576 and
// 355.6 at 32768 with 34 and 68 % more workspace; 8192: 0.8 % slower): the smallest of 16384 / 24576 / 32768 rows
// whose dH launch fills whole rounds of workgroups to 97 %.
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
// what that rounding leaves (1256 slices: 36 ranges of 34 and one of 32).
// 5003 tokens at the 7B head: 280 dH tiles took a second round for 24 of them, 6.52 ms; cut into ten ranges, 3.87 ms.  1237 at the 8B
// head 2.82 / 1.13; dW of 16384 tokens there 14.14 / 13.93.
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
// batch; what reading rows costs the logits contraction and the dH contraction, with its transposing reads, grows with it.  Repacked /
// direct in alternating runs, whole call, ms at V = 151936 unless stated.  H a multiple of the 256-wide dH tile: 1500 tokens
// 5.06 / 4.49 (H = 4096), 1.44 / 1.30 (1024); 5000: 13.55 / 13.02, 3.74 / 3.65; 7168: 18.87 / 18.62 (4096), 5.15 / 5.08 (1024), 23.74 / 23.63
// (5120), but 17.41 / 17.56 (3584, V = 152064); 8192: 20.99 / 20.63 (4096), 26.44 / 26.73 (5120).  Other H, whose dH tiles are padded (the work
// grows with the tiles, the repack with H): 1500: 1.00 / 0.91 (576), 0.73 / 0.64 (320); 5000: 2.61 / 2.58, 1.85 / 1.81; 6144: 3.14 / 3.13, 2.16 / 2.15; 7168:
// 3.54 / 3.55, 2.49 / 2.54; 8192 at V = 50000: 0.98 / 0.99 (320).  Forward pass alone: 2000 tokens 2.16 / 1.76 (4096), 0.59 / 0.50 (1024); 12288: 10.62 / 10.13,
// 2.92 / 2.83; 24576: 21.2 / 20.4, 5.75 / 5.71, 26.4 / 26.3 (5120); 49152: 41.8 / 40.8, 11.3 / 11.4, 52.0 / 52.3; with contractions of a few
// slices 5000: 0.328 / 0.322 (H = 64, V = 160000), 8192: 0.510 / 0.506, 16384: 0.992 / 0.991.
static int direct_tokens(int H) { return H % kBN == 0 ? 7168 : 6144; }
static int direct_tokens_forward(int H) { return H >= kBN ? 24576 : 8192; }

// launch(integral_constant) with the number of blocks that is built for so many: 2, 4, 5, 6 or 7
template <class F>
static void with_blocks(int blocks, F&& launch) {
  if (blocks <= 2) launch(std::integral_constant<int, 2>{});
  else if (blocks <= 4) launch(std::integral_constant<int, 4>{});
  else if (blocks == 5) launch(std::integral_constant<int, 5>{});
  else if (blocks == 6) launch(std::integral_constant<int, 6>{});
  else launch(std::integral_constant<int, 7>{});
}

// logits contraction: rows = vocabulary, columns = tokens (tiles_n tiles), contraction over the hidden size; W either
// repacked (Wb) or read as it is (Wb NULL)
template <class Epi>
static nat_status launch_logits(const uint16_t* W, const uint16_t* Wb, const uint16_t* Hb, int V, int H, int Vp, int tiles_n,
                                const Epi& epi, hipStream_t s) {
  ProfScope prof(PC_LOGITS, s);
  GemmArgs g{Wb ? Wb : W, Hb, H, Vp / kBM, tiles_n, NAT_GROUP_LOGITS, 0, H / kBK, 1, 0, 0, V, H, 1};
  const int units = g.tiles_m * g.tiles_n;
  const int blocks = Wb ? 8 : column_blocks(epi.n_valid, tiles_n);
  if (logits_columns_pay(blocks, tiles_n, g.tiles_m, H / kBK)) {
    g.walk = walk_length(units, H / kBK);                     // also beyond kLogitsWalkSlices (one or two columns there: within 1 % of one tile each)
    with_blocks(blocks, [&](auto nb) {
      mfma_nt_kernel<Epi, Src::kRows, Src::kBlocked, false, true, decltype(nb)::value><<<walk_grid(units, g.walk), 256, 0, s>>>(g, epi);
    });
    NAT_LAUNCH_CHECK();
    return NAT_OK;
  }
  g.walk = logits_walk(units, H / kBK, Wb ? 8 : last_blocks(epi.n_valid, tiles_n), tiles_n);
  if (g.walk > 1) {
    if (Wb) mfma_nt_kernel<Epi, Src::kBlockedInterleaved, Src::kBlocked, false, true><<<walk_grid(units, g.walk), 256, 0, s>>>(g, epi);
    else mfma_nt_kernel<Epi, Src::kRows, Src::kBlocked, false, true><<<walk_grid(units, g.walk), 256, 0, s>>>(g, epi);
  } else {
    if (Wb) mfma_nt_kernel<Epi, Src::kBlockedInterleaved, Src::kBlocked, false, false><<<units, 256, 0, s>>>(g, epi);
    else mfma_nt_kernel<Epi, Src::kRows, Src::kBlocked, false, false><<<units, 256, 0, s>>>(g, epi);
  }
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
    // (whole step at the 8B head: sub-chunks of 16384 instead of 8192 tokens 0.4 % slower), while the dW contraction below keeps
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
        const RangeCut cut = range_cut(tiles, Vp / kBK, 2);
        uint16_t* dH_s = (uint16_t*)a.dH + (int64_t)(c0 + s0) * H;
        ProfScope prof(PC_DHIDDEN, s);
        GemmArgs g{Eb_s, Wtb, Vp, snp / kBM, Hp / kBN, NAT_GROUP_DHIDDEN, 0, Vp / kBK, cut.splits, cut.kt_per, cut.tail, V, H, 1};
        int columns = kBN;
        if (direct) {            // dH^T = W^T E^T from W as it is
          g.A = W;
          g.B = Eb_s;
          g.tiles_m = Hp / kBM;
          g.tiles_n = snp / kBN;
          DHiddenEpilogue<false> e{snv, H, dH_s, beta + s0, dh_part};
          const int blocks = column_blocks(snv, g.tiles_n);
          if (dh_columns_pay(blocks, g.tiles_n, g.tiles_m, Vp / kBK)) {
            with_blocks(blocks, [&](auto nb) {
              constexpr int kNB = decltype(nb)::value;
              mfma_nt_kernel<DHiddenEpilogue<false>, Src::kKMajorRows, Src::kBlocked, false, false, kNB><<<cut.grid, 256, 0, s>>>(g, e);
              columns = kNB * 32;
            });
          } else {
            mfma_nt_kernel<DHiddenEpilogue<false>, Src::kKMajorRows, Src::kBlocked, false, false><<<cut.grid, 256, 0, s>>>(g, e);
          }
        } else {
          DHiddenEpilogue<true> e{snv, H, dH_s, beta + s0, dh_part};
          mfma_nt_kernel<DHiddenEpilogue<true>, Src::kBlocked, Src::kBlockedInterleaved, true, false><<<cut.grid, 256, 0, s>>>(g, e);
        }
        NAT_LAUNCH_CHECK();
        if (cut.splits > 1) {
          dh_tail_reduce_kernel<<<dim3(kBM * kBN / 1024, cut.tail), 256, 0, s>>>(dh_part, g, direct, columns, beta + s0, snv, H, dH_s);
          NAT_LAUNCH_CHECK();
        }
      }
    }
    {  // dW: rows = vocabulary, columns = hidden units, contraction over the chunk's (padded) tokens
      // A = E from its one copy (rows = token), i.e. stored along this contraction's k axis
      // The leftover tiles of the last round are cut into ranges of tokens (multiples of the 8 k-slices that the
      // k-major loader starts at): see range_cut.
      const int kt = (int)round_up((nv + kBK - 1) / kBK, 2);     // only the slices that hold tokens
      const RangeCut cut = range_cut((Vp / kBM) * (Hp / kBN), kt, 8);
      const int accumulate = (c0 > 0 || a.accumulate_dw) ? 1 : 0;
      GemmArgs g{Eb, Hktb, kt * kBK, Vp / kBM, Hp / kBN, NAT_GROUP_DWEIGHT, Vp / 32, np / kBK, cut.splits, cut.kt_per, cut.tail, 0, 0,
                 dw_walk(cut.grid, kt)};
      {
        ProfScope prof(PC_DWEIGHT, s);
        const int grid = walk_grid(cut.grid, g.walk);
        const bool stream = (int64_t)V * H * 4 > kDWeightStreamBytes;
        if (accumulate)
          mfma_nt_kernel<DWeightEpilogue<true>, Src::kKMajorBlocked, Src::kBlocked, true, true><<<grid, 256, 0, s>>>(g, DWeightEpilogue<true>{V, H, stream, a.dW, dh_part});
        else
          mfma_nt_kernel<DWeightEpilogue<false>, Src::kKMajorBlocked, Src::kBlocked, true, true><<<grid, 256, 0, s>>>(g, DWeightEpilogue<false>{V, H, stream, a.dW, dh_part});
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
