// nat_compact / nat_compact_pi: stable mask -> index compaction of the selected
// tokens with the Horvitz-Thompson weight of Eq. 6 / Eq. 9 folded with the
// 1/G * 1/|o_i| averaging of Eq. 5 (inclusion probability from the scheme's
// closed form, or read from a per-token array), plus an optional gather of the
// kept rows.
//
// Passes over the bit mask: (for large batches) population counts of tiles and of groups of tiles,
// and a scatter in which each wavefront ranks its 64 tokens with a
// bit-prefix so that consecutive lanes write consecutive outputs.  The scatter also gathers the
// per-token words (ids, behaviour log-probs) and writes the per-rollout offsets; the gather of
// hidden rows is a kernel of its own.
#include "nat_internal.h"

#include <mutex>

namespace nat {

constexpr int kTileTokens = 4096;                 // tokens per scatter block
constexpr int kTileWords = kTileTokens / 32;      // 128 mask words
// Tiles whose counts are also added up, one block of the count pass: every tile adds up all groups before its own, so beyond kLongTiles (2^28 tokens)
// the groups are longer.  Compaction, us, a scan launch / groups of 16 / of 256: 2^29 tokens 1490 / 1488 / 1382, with ids and log-probs 2798 / 2433 / 2521; 2^30
// 3036 / 3278 / 2832, 6187 / 5335 / 5373; 2^31 6280 / 8335 / 6039, 11253 / 12509 / 10148, one token in a hundred kept 4262 / 6271 / 4012.
constexpr int kGroupTiles = 16, kLongGroupTiles = 256, kLongTiles = 65536;
constexpr int group_tiles_of(int64_t n_tiles) { return n_tiles > kLongTiles ? kLongGroupTiles : kGroupTiles; }
// Up to kInlineTiles (two million tokens, 256 KiB of mask) a scatter block counts the mask words before its own tile and
// there is no count launch; beyond, it adds up the counts of the groups before its own and of the tiles before it in its group.
// Up to there the block also has sixteen wavefronts of 256 tokens, not four of 1024: with few
// blocks the chain of loads of one wavefront is the kernel's time.  Whole selection with the line at 256 / 512 / 1024 tiles, us: 320 tiles 24.7 /
// 19.0 / 19.1; 450 tiles of 550-token rollouts 32.5 / 29.3 / 29.3; 980 tiles 35.4 / 35.6 / 43.9, Poisson 45.9 / 45.9 / 52.3.
constexpr int kInlineTiles = 512;
// With given probabilities, which take the registers, 1280 blocks of four wavefronts are resident at a time (waves_per_simd), and a launch of a few more
// takes twice as long: up to kEightTiles eight wavefronts of 512 tokens a block.  Compaction of rollouts of 20 / 400 / 16384 tokens with ids and log-probs,
// us, four / eight: 1300 tiles 63.6 / 53.0, 43.9 / 42.6, 33.8 / 33.5; 1536 71.3 / 57.0, 47.9 / 44.0, 36.7 / 37.1; 1792 76.1 / 63.2, 51.3 / 48.8, 40.9 / 41.6; 3500 144 / 136, 107 / 108, 91 /
// 93; 16384 608 / 581, 435 / 449, 382 / 391.
constexpr int kEightTilesFrom = 1280, kEightTiles = 1792;
// Wavefronts per SIMD that the registers of a kernel have to leave room for: a launch that is just over one round of the blocks that the chip holds takes
// twice as long.  Four wavefronts a block, rollouts of 20 / 400 / 16384 tokens, us, as the compiler likes it / so: 1700 tiles 70.5 / 57.7, 44.7 / 38.7, 33.6 / 31.2, with
// probabilities 1025 tiles 56.9 / 47.2, 39.6 / 33.0, 28.3 / 27.3; no slower anywhere from 700 to 16384 tiles.  (All eight: 16384 tiles of 1500 tokens 326 / 349; with
// probabilities seven, which spills: +15 %.)
constexpr int waves_per_simd(int waves, bool pi) { return waves == 4 ? pi ? 5 : 7 : waves == 8 ? 8 : 1; }

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

// tile_count[b] = number of kept tokens among packed positions [b*4096, (b+1)*4096), one wavefront per tile; group_count[g] = the sum of
// group_tiles of them, one block per group, 16 tiles at a time.  (A scan of the tile counts by one block, a launch of its own that every tile waited
// for, took 17 us at 2^26 tokens.)
__global__ void __launch_bounds__(kGroupTiles * 64)
compact_count_kernel(const uint32_t* __restrict__ mask_bits, int64_t n_words, int n_tiles, int group_tiles,
                     int32_t* __restrict__ tile_count, int32_t* __restrict__ group_count) {
  __shared__ int count[kGroupTiles];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int mine = 0;
  for (int t = wave; t < group_tiles; t += kGroupTiles) {
    const int tile = blockIdx.x * group_tiles + t;
    const int64_t w = (int64_t)tile * kTileWords + 2 * lane;    // n_words is even
    const int c = wave_sum(w < n_words ? __popc(mask_bits[w]) + __popc(mask_bits[w + 1]) : 0);
    if (lane == 0 && tile < n_tiles) tile_count[tile] = c;
    mine += c;
  }
  if (lane == 0) count[wave] = mine;
  __syncthreads();
  if (wave == 0) {
    const int sum = wave_sum(lane < kGroupTiles ? count[lane] : 0);
    if (lane == 0) group_count[blockIdx.x] = sum;
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
  const int32_t* tile_count; const int32_t* group_count;        // of the count pass; or NULL: the block counts the mask words
  int group_tiles;
  int mask_wide;                                                // mask_bits is 16-byte aligned
  int32_t* kept_idx; int32_t* kept_seq; float* kept_w; int32_t* cu_kept; int32_t* n_kept; int32_t* h_n_kept /*pinned, or NULL*/;
  const int32_t* ids; int32_t* ids_k; const float* old_logp; float* old_logp_k;
};

// One block per tile of 4096 positions, kWaves wavefronts, 64 positions at a time.
// Bound by the bytes it moves; by the chain of dependent loads at the size of a real batch.  A wavefront reads its own mask words and has all its
// per-token loads (probabilities, ids, log-probs) out before the tokens in front of the tile are counted and its rollouts are looked up: loads
// in flight are worth more than wavefronts (sixteen groups at once take 96 registers; 2^26 Poisson tokens, four groups at a time 362 us,
// eight 350, sixteen 337: 1.65 GB at 4.9 TB/s; 387 with the loads behind the search and a scan launch).  Tiles go from the last to the first: what
// the selection read and wrote last is still in the Infinity Cache (from the first: 20 us more).  1.3 million tokens in 128 rollouts: 20 -> 15 us.
// The per-token words ride along here because the token is already in hand: a row-gather block per kept token for them took
// 8.66 ms of a 2^26-token batch, 190 us of a 1.3-million-token one.
template <int kWaves, bool kPi>
__global__ void __launch_bounds__(kWaves * 64, waves_per_simd(kWaves, kPi))
compact_scatter_kernel(SelectArgs a, ScatterArgs c) {
  constexpr int kThreads = kWaves * 64, kGroups = 64 / kWaves, kSpanWords = kGroups * 2;      // groups of 64 positions per wavefront
  __shared__ uint32_t words[kTileWords];
  __shared__ int prefix[kTileWords];                            // kept tokens of the wavefront's span before word w
  __shared__ int wave_tot[kWaves], wave_before[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_tiles = gridDim.x, tile = n_tiles - 1 - (int)blockIdx.x;
  const int64_t tile_first = (int64_t)tile * kTileTokens;
  const int64_t span_first = tile_first + wave * (kGroups * 64), span_end = span_first + kGroups * 64;

  const int64_t wi = (int64_t)tile * kTileWords + wave * kSpanWords + lane;
  const uint32_t word = lane < kSpanWords && wi < c.n_words ? c.mask_bits[wi] : 0u;

  uint64_t group[kGroups];
  int id[kGroups];
  float lp[kGroups];
  double p[kGroups];
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    group[g] = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)word, 2 * g) |
               ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)word, 2 * g + 1) << 32);
    const int64_t n = span_first + g * 64 + lane;
    // a set bit at a position the per-token arrays do not have (a foreign mask) is ranked but reads and writes nothing
    const bool here = ((group[g] >> lane) & 1ull) && n < c.n_tokens;
    if (kPi) p[g] = here ? c.pi[n] : 1.0;                       // what the weight waits for first
    id[g] = here && c.ids ? c.ids[n] : 0;
    lp[g] = here && c.old_logp ? c.old_logp[n] : 0.f;
  }

  int before = 0;
  if (c.group_count) {
    const int group = tile / c.group_tiles, first = group * c.group_tiles;
    for (int j = tid; j < group; j += kThreads) before += c.group_count[j];
    for (int j = first + tid; j < tile; j += kThreads) before += c.tile_count[j];
  } else if (c.mask_wide) {
    const uint4* q = reinterpret_cast<const uint4*>(c.mask_bits);
#pragma unroll 4
    for (int j = tid; j < tile * (kTileWords / 4); j += kThreads) {
      const uint4 x = q[j];
      before += __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w);
    }
  } else {
#pragma unroll 4
    for (int j = tid; j < tile * kTileWords; j += kThreads) before += __popc(c.mask_bits[j]);
  }
  // how many rollouts start before the tile, before its end; at or before this wavefront's first position, its last one
  const int64_t N = c.cu[c.B];
  const int64_t span_last = span_end - 1 < N ? span_end - 1 : N - 1;
  const int64_t key[4] = {tile_first, tile_first + kTileTokens, span_first + 1, span_last + 1};
  int at[4];
  wave_lower_bounds<4>(c.cu, c.B + 1, key, at);
  int i_lo = 0, i_hi = c.B;                                     // positions at or beyond N: any rollout (foreign mask)
  if (span_first < N) {                                         // the last rollout that starts at or before the first position
    i_lo = at[2] > 0 ? at[2] - 1 : 0;
    i_lo = i_lo < c.B ? i_lo : c.B - 1;                         // offsets that do not ascend must not lead past the array
    i_hi = at[3] < c.B ? at[3] : c.B;
    i_hi = i_hi <= i_lo ? i_lo + 1 : i_hi;
  }
  const bool one_rollout = i_hi - i_lo == 1;
  const int64_t one_start = c.cu[i_lo], one_T = c.cu[i_lo + 1] - one_start;
  const int one_scheme = !kPi && a.scheme_per_rollout ? a.scheme_per_rollout[i_lo] : a.scheme;

  const int cnt = __popc(word), incl = wave_inclusive_scan(cnt);
  const int span_kept = __builtin_amdgcn_readlane(incl, 63);
  if (lane < kSpanWords) {
    words[wave * kSpanWords + lane] = word;
    prefix[wave * kSpanWords + lane] = incl - cnt;
  }
  before = wave_sum(before);
  if (lane == 0) {
    wave_tot[wave] = span_kept;
    wave_before[wave] = before;
  }
  __syncthreads();
  int tile_base = 0, span_base = 0, tile_kept = 0;              // kept tokens before the tile, in it before the span, in it
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    tile_base += wave_before[w];
    tile_kept += wave_tot[w];
    if (w < wave) span_base += wave_tot[w];
  }
  if (tile == n_tiles - 1 && tid == 0) {
    *c.n_kept = tile_base + tile_kept;
    if (c.h_n_kept) host_store(c.h_n_kept, tile_base + tile_kept);
  }
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
      int kept = tile_kept;
      if (w < kTileWords) {
        kept = prefix[w] + __popc(words[w] & ((1u << rem) - 1u));
        for (int v = 0; v < w / kSpanWords; ++v) kept += wave_tot[v];
      }
      c.cu_kept[i0 + e * kThreads] = tile_base + kept;
    }
  }
  if (span_kept == 0) return;

  int at_lane = lane;                                           // else all that was formed from it for the loads is kept: 131 and more registers
  asm volatile("" : "+v"(at_lane));
  int out0 = tile_base + span_base;                             // first output of the current group
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int64_t n = span_first + g * 64 + at_lane;
    const int o = out0 + __popcll(group[g] & ((1ull << at_lane) - 1ull));
    out0 += __popcll(group[g]);
    // entries beyond the outputs' capacity are counted but not written
    if (!((group[g] >> at_lane) & 1ull) || o >= c.kept_cap || n >= c.n_tokens) continue;
    int64_t start = one_start, T = one_T;
    int scheme = one_scheme, seq = i_lo;
    if (!one_rollout) {
      seq = rollout_of_pos(c.cu, i_lo, i_hi, n);
      start = c.cu[seq];
      T = c.cu[seq + 1] - start;
      if (!kPi && a.scheme_per_rollout) scheme = a.scheme_per_rollout[seq];
    }
    c.kept_idx[o] = (int32_t)n;
    c.kept_seq[o] = seq;
    c.kept_w[o] = kPi ? (float)(1.0 / ((c.n_rollouts * (double)T) * p[g]))
                      : ht_weight(scheme, T, n - start + 1, c.n_rollouts, a.p, a.min_cut);
    if (c.ids) c.ids_k[o] = id[g];
    if (c.old_logp) c.old_logp_k[o] = lp[g];
  }
}

// N = 0: nothing is kept, every rollout starts at 0.
__global__ void __launch_bounds__(256)
compact_empty_kernel(int B, int32_t* __restrict__ cu_kept, int32_t* __restrict__ n_kept, int32_t* __restrict__ h_n_kept) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i <= B) cu_kept[i] = 0;
  if (i == 0) {
    *n_kept = 0;
    if (h_n_kept) host_store(h_n_kept, 0);
  }
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

// tile_count[n_tiles] + group_count (at most n_tiles + 1), int32, rounded up to 256 bytes
constexpr size_t compact_ws_bytes(int64_t N) {
  return (((size_t)(2 * n_tiles_of(N) + 1) * sizeof(int32_t) + 255) / 256) * 256 + 256;
}

// Scratch of nat_compact_static: the counts of tiles and groups of up to NAT_COMPACT_STATIC_MAX_TOKENS
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
  int32_t* group_count = tile_count + n_tiles;
  int32_t* pinned = pinned_words(c.h_n_kept);
  {
    ProfScope prof(PC_COMPACT, s, !c.no_timing);
    if (n_tiles > 0) {
      const bool count = n_tiles > kInlineTiles;
      const int group_tiles = group_tiles_of(n_tiles);
      if (count) {
        compact_count_kernel<<<(unsigned)((n_tiles + group_tiles - 1) / group_tiles), kGroupTiles * 64, 0, s>>>(c.mask_bits, n_words, (int)n_tiles, group_tiles,
                                                                                                           tile_count, group_count);
        NAT_LAUNCH_CHECK();
      }
      const ScatterArgs sc{(double)c.n_rollouts_global, c.pi, c.mask_bits, n_words, c.N, c.kept_cap, c.cu, c.B,
                           count ? tile_count : nullptr, count ? group_count : nullptr, group_tiles, ((uintptr_t)c.mask_bits & 15) == 0,
                           c.kept_idx, c.kept_seq, c.kept_w, c.cu_kept, c.n_kept, pinned, c.ids, c.ids_k, c.old_logp, c.old_logp_k};
      if (count && c.pi && n_tiles > kEightTilesFrom && n_tiles <= kEightTiles) compact_scatter_kernel<8, true><<<(unsigned)n_tiles, 512, 0, s>>>(a, sc);
      else if (count && c.pi) compact_scatter_kernel<4, true><<<(unsigned)n_tiles, 256, 0, s>>>(a, sc);
      else if (count) compact_scatter_kernel<4, false><<<(unsigned)n_tiles, 256, 0, s>>>(a, sc);
      else if (c.pi) compact_scatter_kernel<16, true><<<(unsigned)n_tiles, 1024, 0, s>>>(a, sc);
      else compact_scatter_kernel<16, false><<<(unsigned)n_tiles, 1024, 0, s>>>(a, sc);
      NAT_LAUNCH_CHECK();
    } else {
      compact_empty_kernel<<<(c.B + 1 + 255) / 256, 256, 0, s>>>(c.B, c.cu_kept, c.n_kept, pinned);
      NAT_LAUNCH_CHECK();
    }
  }
  if (c.h_n_kept && !pinned) NAT_HIP_TRY(hipMemcpyAsync(c.h_n_kept, c.n_kept, sizeof(int32_t), hipMemcpyDeviceToHost, s));
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
  // every word of the scratch that the kernels read is written earlier in the same call (the counts of tiles and
  // groups by the count pass), so nothing has to be cleared between calls
  return compact_run(a, CompactArgs{n_rollouts_global, d_mask_bits, nullptr, d_cu_seqlens, B, N, kept_cap, d_kept_idx,
                                    d_kept_seq, d_kept_w, d_cu_kept, d_n_kept, h_n_kept, d_hidden, d_hidden_k, H,
                                    dtype, d_ids, d_ids_k, d_old_logp, d_old_logp_k, ws, kStaticScratchBytes,
                                    (hipStream_t)stream, true});
}
