// nat_compact / nat_compact_pi: stable mask -> index compaction of the selected
// tokens with the Horvitz-Thompson weight of Eq. 6 / Eq. 9 folded with the
// 1/G * 1/|o_i| averaging of Eq. 5 (inclusion probability from the scheme's
// closed form, or read from a per-token array), plus an optional gather of the
// kept rows.
//
// Passes over the bit mask: per-tile population counts, (for large batches) an exclusive scan
// of the tile counts, and a scatter in which each wavefront ranks its 64 tokens with a
// bit-prefix so that consecutive lanes write consecutive outputs.  The scatter also gathers the
// per-token words (ids, behaviour log-probs) and writes the per-rollout offsets; the gather of
// hidden rows is a kernel of its own.
#include "nat_internal.h"

#include <mutex>

namespace nat {

constexpr int kTileTokens = 4096;                 // tokens per scatter block
constexpr int kTileWords = kTileTokens / 32;      // 128 mask words
// Up to this many tiles (4.2 million tokens) a scatter block adds up the counts of the tiles before
// its own instead of a scan launch between the two passes; up to kInlineCountTiles (half a million
// tokens, 64 KiB of mask) it counts the mask words themselves and there is no count launch either.
// Up to kInlineScanTiles the block also has sixteen wavefronts of 256 tokens, not four of 1024: with fewer
// blocks than the chip holds, the chain of loads of one wavefront is the kernel's time.
constexpr int kInlineScanTiles = 1024, kInlineCountTiles = 128;

__device__ __forceinline__ int wave_sum(int v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

__device__ __forceinline__ int wave_inclusive_scan(int v) {
  const int lane = threadIdx.x & 63;
  for (int off = 1; off < 64; off <<= 1) {
    const int up = __shfl_up(v, off);
    if (lane >= off) v += up;
  }
  return v;
}

// tile_count[b] = number of kept tokens among packed positions [b*4096, (b+1)*4096); one wavefront per tile
__global__ void __launch_bounds__(256)
compact_count_kernel(const uint32_t* __restrict__ mask_bits, int64_t n_words, int n_tiles,
                     int32_t* __restrict__ tile_count) {
  const int tile = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (tile >= n_tiles) return;
  const int64_t w = (int64_t)tile * kTileWords + 2 * lane;      // n_words is even
  const int c = wave_sum(w < n_words ? __popc(mask_bits[w]) + __popc(mask_bits[w + 1]) : 0);
  if (lane == 0) tile_count[tile] = c;
}

// tile_offset[0..n_tiles) = exclusive scan of tile_count.  One block, kScanPer consecutive tiles per thread.
constexpr int kScanPer = 8;
__global__ void __launch_bounds__(1024)
compact_scan_kernel(const int32_t* __restrict__ tile_count, int n_tiles, int32_t* __restrict__ tile_offset) {
  __shared__ int wave_tot[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int carry = 0;
  for (int base = 0; base < n_tiles; base += 1024 * kScanPer) {
    const int j0 = base + (int)threadIdx.x * kScanPer;
    int v[kScanPer], mine = 0;
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) {
      v[e] = j0 + e < n_tiles ? tile_count[j0 + e] : 0;
      mine += v[e];
    }
    const int incl = wave_inclusive_scan(mine);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int run = carry + incl - mine;
    for (int w = 0; w < 16; ++w) {
      if (w < wave) run += wave_tot[w];
      carry += wave_tot[w];
    }
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) {
      if (j0 + e < n_tiles) tile_offset[j0 + e] = run;
      run += v[e];
    }
    __syncthreads();
  }
}

// Horvitz-Thompson weight of kept token t (1-based) of a rollout of length T.
__device__ __forceinline__ float ht_weight(int scheme, int64_t T, int64_t t, double n_rollouts, double p, int64_t C) {
  double w;
  if (scheme == NAT_SCHEME_URS) {
    w = 1.0 / (n_rollouts * (double)T * p);
  } else {
    int64_t Ci = C < 1 ? 1 : C;
    if (Ci > T) Ci = T;
    if (scheme == NAT_SCHEME_RPC && t > Ci) {
      w = (double)(T - Ci + 1) / ((double)(T - t + 1) * (double)T * n_rollouts);
    } else {
      w = 1.0 / (n_rollouts * (double)T);
    }
  }
  return (float)w;
}

struct ScatterArgs {
  double n_rollouts; const double* pi;
  const uint32_t* mask_bits; int64_t n_words; int64_t n_tokens; int64_t kept_cap;
  const int64_t* cu; int B;
  const int32_t* tile_count; const int32_t* tile_offset;        // offsets; or NULL: the block adds up the counts; or both NULL:
                                                                // it counts the mask words
  int32_t* kept_idx; int32_t* kept_seq; float* kept_w; int32_t* cu_kept; int32_t* n_kept;
  const int32_t* ids; int32_t* ids_k; const float* old_logp; float* old_logp_k;
};

// One block per tile of 4096 positions, kWaves wavefronts, 64 positions at a time, four such groups in flight:
// the loads of a batch (ids, log-probs, probabilities) are issued before its first weight is computed.
// Bound by the bytes it moves and, for weights that differ from token to token, by their fp64 divisions; by latency
// at the size of a real batch.  The per-token words ride along here because the token is already in hand: a
// row-gather block per kept token for them took 8.66 ms of a 2^26-token batch (compaction as a whole 9.06 ->
// 0.39 ms), 190 us of a 1.3-million-token one (whole selection 225 -> 25 us; scatter 17 us with four wavefronts per
// block, 14.5 with sixteen).
template <int kWaves>
__global__ void __launch_bounds__(kWaves * 64)
compact_scatter_kernel(SelectArgs a, ScatterArgs c) {
  constexpr int kBatch = 4, kThreads = kWaves * 64, kGroups = 64 / kWaves;      // groups of 64 positions per wavefront
  __shared__ uint32_t words[kTileWords];
  __shared__ int prefix[kTileWords + 1];                        // kept tokens of the tile before word w
  __shared__ int wave_tot[2], wave_before[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = blockIdx.x, n_tiles = gridDim.x;
  const int64_t tile_first = (int64_t)tile * kTileTokens;

  uint32_t word = 0;
  if (tid < kTileWords) {
    const int64_t wi = (int64_t)tile * kTileWords + tid;
    word = wi < c.n_words ? c.mask_bits[wi] : 0u;
    words[tid] = word;
  }
  int before = 0;
  if (!c.tile_offset) {
    if (c.tile_count) for (int j = tid; j < tile; j += kThreads) before += c.tile_count[j];
    else for (int j = tid; j < tile * kTileWords; j += kThreads) before += __popc(c.mask_bits[j]);
  }
  // how many rollouts start before the tile, before its end; at or before this wavefront's first position, its last one
  const int64_t N = c.cu[c.B], span_first = tile_first + wave * (kGroups * 64), span_end = span_first + kGroups * 64;
  const int64_t span_last = span_end - 1 < N ? span_end - 1 : N - 1;
  const int64_t key[4] = {tile_first, tile_first + kTileTokens, span_first + 1, span_last + 1};
  int at[4];
  wave_lower_bounds<4>(c.cu, c.B + 1, key, at);
  const int cnt = __popc(word), incl = wave_inclusive_scan(cnt);
  if (tid < kTileWords && lane == 63) wave_tot[wave] = incl;
  before = wave_sum(before);
  if (lane == 0) wave_before[wave] = before;
  __syncthreads();
  if (tid < kTileWords) {
    const int excl = incl - cnt + (wave == 1 ? wave_tot[0] : 0);
    prefix[tid] = excl;
    if (tid == kTileWords - 1) prefix[kTileWords] = excl + cnt;
  }
  int tile_base = 0;
  if (c.tile_offset) tile_base = c.tile_offset[tile];
  else
    for (int w = 0; w < kWaves; ++w) tile_base += wave_before[w];
  __syncthreads();
  if (tile == n_tiles - 1 && tid == 0) *c.n_kept = tile_base + prefix[kTileWords];
  // Offsets of the rollouts that start in this tile (offsets outside [0, n_tokens] count as its ends), by the whole block
  // and four loads at a time: empty rollouts can put any number of them at one position.  Compaction of 100 rollouts of 1000
  // tokens and 4000 / 65000 / a million empty ones: 17.8 / 210 / 5300 us by the wavefront of their span, 8.7 / 22 / 311 by the block.
  const int r0 = tile == 0 ? 0 : at[0], r1 = tile == n_tiles - 1 ? c.B + 1 : at[1];
  for (int i0 = r0 + tid; i0 < r1; i0 += 4 * kThreads) {
    int64_t start[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) start[e] = r1 - i0 > e * kThreads ? c.cu[i0 + e * kThreads] : 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (r1 - i0 <= e * kThreads) break;
      const int64_t pos = start[e] < 0 ? 0 : start[e] > c.n_tokens ? c.n_tokens : start[e];
      const int64_t off = pos - tile_first;
      const int rel = off < 0 ? 0 : off > kTileTokens ? kTileTokens : (int)off, w = rel >> 5, rem = rel & 31;
      c.cu_kept[i0 + e * kThreads] = tile_base + prefix[w] + (rem ? __popc(words[w] & ((1u << rem) - 1u)) : 0);
    }
  }

  constexpr int kSpanWords = kGroups * 2;
  if (prefix[wave * kSpanWords] == prefix[(wave + 1) * kSpanWords]) return;      // nothing kept
  int i_lo = 0, i_hi = c.B;                                     // positions at or beyond N: any rollout (foreign mask)
  if (span_first < N) {                                         // the last rollout that starts at or before the first position
    i_lo = at[2] > 0 ? at[2] - 1 : 0;
    i_lo = i_lo < c.B ? i_lo : c.B - 1;                         // offsets that do not ascend must not lead past the array
    i_hi = at[3] < c.B ? at[3] : c.B;
    i_hi = i_hi <= i_lo ? i_lo + 1 : i_hi;
  }
  const bool one_rollout = i_hi - i_lo == 1;
  const int64_t one_start = c.cu[i_lo], one_T = c.cu[i_lo + 1] - one_start;
  const int one_scheme = a.scheme_per_rollout ? a.scheme_per_rollout[i_lo] : a.scheme;

  for (int g0 = 0; g0 < kGroups; g0 += kBatch) {
    bool keep[kBatch];
    int out[kBatch], id[kBatch], seq[kBatch];
    float lp[kBatch];
    double p[kBatch];
    int64_t n[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int w = wave * kSpanWords + 2 * (g0 + b);
      const uint64_t group = (uint64_t)words[w] | ((uint64_t)words[w + 1] << 32);
      n[b] = span_first + (g0 + b) * 64 + lane;
      out[b] = tile_base + prefix[w] + __popcll(group & ((1ull << lane) - 1ull));
      // entries beyond the outputs' capacity are counted but not written; a set bit at a position the
      // per-token arrays do not have (a foreign mask) is ranked but reads and writes nothing
      keep[b] = ((group >> lane) & 1ull) && out[b] < c.kept_cap && n[b] < c.n_tokens;
      id[b] = keep[b] && c.ids ? c.ids[n[b]] : 0;
      lp[b] = keep[b] && c.old_logp ? c.old_logp[n[b]] : 0.f;
      p[b] = keep[b] && c.pi ? c.pi[n[b]] : 1.0;
      seq[b] = i_lo;
    }
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      if (!keep[b]) continue;
      int64_t start = one_start, T = one_T;
      int scheme = one_scheme;
      if (!one_rollout) {
        seq[b] = rollout_of_pos(c.cu, i_lo, i_hi, n[b]);
        start = c.cu[seq[b]];
        T = c.cu[seq[b] + 1] - start;
        if (a.scheme_per_rollout) scheme = a.scheme_per_rollout[seq[b]];
      }
      const int o = out[b];
      c.kept_idx[o] = (int32_t)n[b];
      c.kept_seq[o] = seq[b];
      c.kept_w[o] = c.pi ? (float)(1.0 / ((c.n_rollouts * (double)T) * p[b]))
                         : ht_weight(scheme, T, n[b] - start + 1, c.n_rollouts, a.p, a.min_cut);
      if (c.ids) c.ids_k[o] = id[b];
      if (c.old_logp) c.old_logp_k[o] = lp[b];
    }
  }
}

// N = 0: nothing is kept, every rollout starts at 0.
__global__ void __launch_bounds__(256)
compact_empty_kernel(int B, int32_t* __restrict__ cu_kept, int32_t* __restrict__ n_kept) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i <= B) cu_kept[i] = 0;
  if (i == 0) *n_kept = 0;
}

// One block per kept row: copy row kept_idx[k] of `src` (row_bytes, multiple of 16) to row k.
__global__ void __launch_bounds__(256)
gather_rows_kernel(const int32_t* __restrict__ kept_idx, const int32_t* __restrict__ n_kept, int64_t rows_cap,
                   const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t row_vec16) {
  const int nk = *n_kept;
  for (int64_t k = blockIdx.x; k < nk && k < rows_cap; k += gridDim.x) {
    const int64_t n = kept_idx[k];
    const uint4* s = src + n * row_vec16;
    uint4* d = dst + k * row_vec16;
    for (int64_t j = threadIdx.x; j < row_vec16; j += blockDim.x) d[j] = s[j];
  }
}

constexpr int64_t n_tiles_of(int64_t N) { return (N + kTileTokens - 1) / kTileTokens; }

// tile_count[n_tiles] + tile_offset[n_tiles + 1], int32, rounded up to 256 bytes
constexpr size_t compact_ws_bytes(int64_t N) {
  return (((size_t)(2 * n_tiles_of(N) + 1) * sizeof(int32_t) + 255) / 256) * 256 + 256;
}

// Scratch of nat_compact_static: the tile counts and offsets of up to NAT_COMPACT_STATIC_MAX_TOKENS
// tokens (about 513 KiB), resident on every GPU the library runs on until the process ends.  In host
// code this name stands for the symbol, not for a device address: the address on each device comes
// from hipGetSymbolAddress (static_scratch below) and only that pointer is handed to kernels.
constexpr size_t kStaticScratchBytes = compact_ws_bytes(NAT_COMPACT_STATIC_MAX_TOKENS);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices];          // per device: each GPU has its own copy at its own address

// Address of `scratch` on the current device, looked up once per device.
static nat_status static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return NAT_HIP_ERROR;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return NAT_HIP_ERROR;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return NAT_OK;
}

}  // namespace nat

using namespace nat;

extern "C" size_t nat_compact_workspace_bytes(int64_t N) {
  if (N < 0) return 0;
  return compact_ws_bytes(N);
}

namespace nat {

nat_status compact_run(const SelectArgs& a, const CompactArgs& c) {
  if (!c.cu || !c.cu_kept || !c.n_kept || c.B <= 0 || c.N < 0 || c.N >= (int64_t(1) << 31) ||
      c.n_rollouts_global <= 0 || c.kept_cap < 0)
    return NAT_INVALID_ARG;
  if (c.N > 0 && !c.mask_bits) return NAT_INVALID_ARG;
  if (c.N > 0 && c.kept_cap > 0 && (!c.kept_idx || !c.kept_seq || !c.kept_w)) return NAT_INVALID_ARG;
  if ((c.hidden != nullptr) != (c.hidden_k != nullptr) || (c.ids != nullptr) != (c.ids_k != nullptr) ||
      (c.old_logp != nullptr) != (c.old_logp_k != nullptr))
    return NAT_INVALID_ARG;
  int64_t row_bytes = 0;
  if (c.hidden) {
    if (c.dtype != NAT_DTYPE_F32 && c.dtype != NAT_DTYPE_BF16) return NAT_UNSUPPORTED_DTYPE;
    if (c.H <= 0) return NAT_BAD_SHAPE;
    row_bytes = (int64_t)c.H * (c.dtype == NAT_DTYPE_F32 ? 4 : 2);
    if (row_bytes % 16 != 0) return NAT_BAD_SHAPE;
    if (((uintptr_t)c.hidden & 15) || ((uintptr_t)c.hidden_k & 15)) return NAT_INVALID_ARG;   // 16-byte row copies
  }
  if (!c.ws || c.ws_bytes < nat_compact_workspace_bytes(c.N)) return NAT_WORKSPACE_TOO_SMALL;

  hipStream_t s = c.stream;
  const int64_t n_tiles = n_tiles_of(c.N);
  const int64_t n_words = nat_mask_words(c.N);
  int32_t* tile_count = (int32_t*)c.ws;
  int32_t* tile_offset = tile_count + n_tiles;
  {
    ProfScope prof(PC_COMPACT, s, !c.no_timing);
    if (n_tiles > 0) {
      const bool count = n_tiles > kInlineCountTiles, scan = n_tiles > kInlineScanTiles;
      if (count) {
        compact_count_kernel<<<(unsigned)((n_tiles + 3) / 4), 256, 0, s>>>(c.mask_bits, n_words, (int)n_tiles, tile_count);
        NAT_LAUNCH_CHECK();
      }
      if (scan) {
        compact_scan_kernel<<<1, 1024, 0, s>>>(tile_count, (int)n_tiles, tile_offset);
        NAT_LAUNCH_CHECK();
      }
      const ScatterArgs sc{(double)c.n_rollouts_global, c.pi, c.mask_bits, n_words, c.N, c.kept_cap, c.cu, c.B,
                           count ? tile_count : nullptr, scan ? tile_offset : nullptr, c.kept_idx, c.kept_seq, c.kept_w,
                           c.cu_kept, c.n_kept, c.ids, c.ids_k, c.old_logp, c.old_logp_k};
      if (scan) compact_scatter_kernel<4><<<(unsigned)n_tiles, 256, 0, s>>>(a, sc);
      else compact_scatter_kernel<16><<<(unsigned)n_tiles, 1024, 0, s>>>(a, sc);
      NAT_LAUNCH_CHECK();
    } else {
      compact_empty_kernel<<<(c.B + 1 + 255) / 256, 256, 0, s>>>(c.B, c.cu_kept, c.n_kept);
      NAT_LAUNCH_CHECK();
    }
  }
  if (c.h_n_kept) NAT_HIP_TRY(hipMemcpyAsync(c.h_n_kept, c.n_kept, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  const int64_t gather_rows = c.N < c.kept_cap ? c.N : c.kept_cap;
  if (gather_rows > 0 && c.hidden) {
    ProfScope prof(PC_GATHER, s, !c.no_timing);
    const int64_t grid = gather_rows < 65536 * 4 ? gather_rows : 65536 * 4;
    gather_rows_kernel<<<(unsigned)grid, 256, 0, s>>>(c.kept_idx, c.n_kept, gather_rows, (const uint4*)c.hidden,
                                                     (uint4*)c.hidden_k, row_bytes / 16);
    NAT_LAUNCH_CHECK();
  }
  return NAT_OK;
}

}  // namespace nat

extern "C" nat_status nat_compact(const nat_select_params* params, int32_t n_rollouts_global,
                                  const uint32_t* d_mask_bits, const int64_t* d_cu_seqlens, int32_t B, int64_t N,
                                  int64_t kept_cap, int32_t* d_kept_idx, int32_t* d_kept_seq, float* d_kept_w, int32_t* d_cu_kept,
                                  int32_t* d_n_kept, int32_t* h_n_kept,
                                  const void* d_hidden, void* d_hidden_k, int32_t H, int32_t dtype,
                                  const int32_t* d_ids, int32_t* d_ids_k,
                                  const float* d_old_logp, float* d_old_logp_k,
                                  void* d_ws, size_t ws_bytes, void* stream) {
  SelectArgs a;
  nat_status st = validate_select(params, &a);
  if (st != NAT_OK) return st;
  return compact_run(a, CompactArgs{n_rollouts_global, d_mask_bits, nullptr, d_cu_seqlens, B, N, kept_cap, d_kept_idx,
                                    d_kept_seq, d_kept_w, d_cu_kept, d_n_kept, h_n_kept, d_hidden, d_hidden_k, H,
                                    dtype, d_ids, d_ids_k, d_old_logp, d_old_logp_k, d_ws, ws_bytes,
                                    (hipStream_t)stream, false});
}

extern "C" nat_status nat_compact_pi(int32_t n_rollouts_global, const uint32_t* d_mask_bits, const double* d_pi,
                                     const int64_t* d_cu_seqlens, int32_t B, int64_t N,
                                     int64_t kept_cap, int32_t* d_kept_idx, int32_t* d_kept_seq, float* d_kept_w, int32_t* d_cu_kept,
                                     int32_t* d_n_kept, int32_t* h_n_kept,
                                     const void* d_hidden, void* d_hidden_k, int32_t H, int32_t dtype,
                                     const int32_t* d_ids, int32_t* d_ids_k,
                                     const float* d_old_logp, float* d_old_logp_k,
                                     void* d_ws, size_t ws_bytes, void* stream) {
  if (N > 0 && !d_pi) return NAT_INVALID_ARG;
  SelectArgs a{};
  a.scheme = NAT_SCHEME_FULL;
  a.min_cut = 1;
  a.p = 1.0;
  return compact_run(a, CompactArgs{n_rollouts_global, d_mask_bits, d_pi, d_cu_seqlens, B, N, kept_cap, d_kept_idx,
                                    d_kept_seq, d_kept_w, d_cu_kept, d_n_kept, h_n_kept, d_hidden, d_hidden_k, H,
                                    dtype, d_ids, d_ids_k, d_old_logp, d_old_logp_k, d_ws, ws_bytes,
                                    (hipStream_t)stream, false});
}

extern "C" nat_status nat_compact_static(const nat_select_params* params, int32_t n_rollouts_global,
                                         const uint32_t* d_mask_bits, const int64_t* d_cu_seqlens, int32_t B,
                                         int64_t N, int64_t kept_cap, int32_t* d_kept_idx, int32_t* d_kept_seq,
                                         float* d_kept_w, int32_t* d_cu_kept, int32_t* d_n_kept, int32_t* h_n_kept,
                                         const void* d_hidden, void* d_hidden_k, int32_t H, int32_t dtype,
                                         const int32_t* d_ids, int32_t* d_ids_k,
                                         const float* d_old_logp, float* d_old_logp_k, void* stream) {
  SelectArgs a;
  nat_status st = validate_select(params, &a);
  if (st != NAT_OK) return st;
  if (N > NAT_COMPACT_STATIC_MAX_TOKENS) return NAT_BAD_SHAPE;      // beyond the resident scratch
  void* ws = nullptr;
  st = static_scratch(&ws);
  if (st != NAT_OK) return st;
  // every word of the scratch that the kernels read is written earlier in the same call (the tile
  // counts by the count pass, the offsets by the scan), so nothing has to be cleared between calls
  return compact_run(a, CompactArgs{n_rollouts_global, d_mask_bits, nullptr, d_cu_seqlens, B, N, kept_cap, d_kept_idx,
                                    d_kept_seq, d_kept_w, d_cu_kept, d_n_kept, h_n_kept, d_hidden, d_hidden_k, H,
                                    dtype, d_ids, d_ids_k, d_old_logp, d_old_logp_k, ws, kStaticScratchBytes,
                                    (hipStream_t)stream, true});
}
