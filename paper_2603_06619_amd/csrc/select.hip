// nat_advantage and nat_select: group-relative advantage (Eq. 2) and the token
// selection mask of Sec. 3.1 (URS) and Sec. 4 (RPC, Eq. 7; deterministic
// truncation), and the Poisson mask of schedule.hip's entry point.  Four packed token
// positions per lane; eight lanes combine their bits into a 32-bit mask word.
#include "nat_internal.h"
#include "philox.hip.h"

#include <type_traits>

namespace nat {

__global__ void advantage_kernel(const float* __restrict__ rewards, int P, int G, float eps_adv,
                                 float* __restrict__ adv) {
  // one wavefront per prompt; fixed-order lane-strided sums then a butterfly
  const int prompt = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (prompt >= P) return;
  const float* R = rewards + (size_t)prompt * G;
  float s = 0.f;
  for (int j = lane; j < G; j += 64) s += R[j];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  const float mu = s / (float)G;
  float q = 0.f;
  for (int j = lane; j < G; j += 64) { const float d = R[j] - mu; q += d * d; }
  for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off);
  const float sigma = sqrtf(q / (float)G);
  for (int j = lane; j < G; j += 64) adv[(size_t)prompt * G + j] = (R[j] - mu) / (sigma + eps_adv);
}

// L_i (RPC), K_i (DET), T_i (FULL, URS) of rollout i of length T; 0 for a dropped one
__device__ __forceinline__ int64_t rollout_cut(const SelectArgs& a, int scheme, int i, int64_t T) {
  int64_t cut = T;
  if (T > 0 && scheme == NAT_SCHEME_RPC) {
    int64_t Ci = a.min_cut < 1 ? 1 : a.min_cut;
    if (Ci > T) Ci = T;
    const uint64_t n = (uint64_t)(T - Ci + 1);
    const u32x4 r = philox4x32_10(u32x4{0u, (uint32_t)(a.rollout_id_base + i), 1u, a.step}, a.key0, a.key1);
    cut = Ci + (int64_t)(((uint64_t)r.x * n) >> 32);
  } else if (scheme == NAT_SCHEME_DET) {
    cut = (int64_t)floor(a.trunc_frac * (double)T);
  }
  if (a.drop_zero_adv && a.drop_zero_adv[i] == 0.f) cut = 0;
  return cut;
}

struct MaskArgs {
  const int64_t* cu; int B; int64_t N;
  const int32_t* cut_in;         // given cut lengths (a prefix mask whatever the scheme), or NULL: drawn here
  int32_t* cut_out;              // drawn cut lengths are also written here (blocks behind the mask blocks), or NULL
  const double* pi;              // Poisson sampling: inclusion probabilities (16-byte aligned when pi_wide)
  int pi_wide;
  unsigned mask_blocks;
  uint32_t* mask_bits;
};

constexpr int kStrip = 256;                       // packed positions of a wavefront's strip, four per lane

// keep iff word < floor(p 2^32); p <= 0 or NaN: never, p >= 1: always
__device__ __forceinline__ bool poisson_keep(uint32_t word, double p) {
  return p >= 1.0 || (p > 0.0 && word < (uint32_t)(p * 4294967296.0));
}

// Selection mask of every scheme.  Bound by the Philox rounds where tokens are drawn one by one (ten rounds of
// two quarter-rate wide multiplies per block of four tokens), by latency at the sizes of a real batch.  A wavefront
// owns kStrips strips of 256 positions (see strips_of) and finds their rollouts with two 64-wide searches.  If it is one
// rollout, that is uniform: lane l owns Philox block first + 64 j + l of strip j, and since a block's four words serve
// four consecutive tokens of the ROLLOUT, lanes whose four positions straddle two blocks take the second one's words from
// the next lane (the last lane: from the first lane of the next strip): 5 evaluations per 4 strips instead of 8.  Else
// each lane searches, strip after strip, and draws the cut of each rollout it meets anew (a Philox block, hidden by the
// other lanes' loads: RPC masks of 2^25 tokens in rollouts of 16 take 69 us, 144 us with a launch that draws the cuts and
// one that reads them).
// Poisson mask of 2^26 tokens: 289 us with a search and up to two evaluations per lane, 144 us now (reading the
// probabilities alone is 112 us); URS mask: 0.18 ms per 2^26 tokens before, 0.076 ms now.
template <bool kPoisson, int kStrips>
__global__ void __launch_bounds__(256)
select_mask_kernel(SelectArgs a, MaskArgs m) {
  constexpr int kSelPerWave = kStrips * kStrip;
  if (blockIdx.x >= m.mask_blocks) {               // the cut lengths themselves
    const int i = (int)(blockIdx.x - m.mask_blocks) * 256 + threadIdx.x;
    if (i >= m.B) return;
    const int scheme = a.scheme_per_rollout ? a.scheme_per_rollout[i] : a.scheme;
    m.cut_out[i] = (int32_t)rollout_cut(a, scheme, i, m.cu[i + 1] - m.cu[i]);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t w0 = ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kSelPerWave;
  if (w0 >= m.N) return;
  // positions at or beyond cu[B] belong to no rollout (the host-passed N may be larger): never kept
  const int64_t n_end = m.cu[m.B] < m.N ? m.cu[m.B] : m.N;
  int i_lo = 0, i_hi = 0;                          // rollouts of the span
  if (w0 < n_end) {
    const int64_t last = w0 + kSelPerWave - 1 < n_end ? w0 + kSelPerWave - 1 : n_end - 1;
    const int64_t key[2] = {w0 + 1, last + 1};
    int at[2];
    wave_lower_bounds<2>(m.cu, m.B, key, at);
    i_lo = at[0] > 0 ? at[0] - 1 : 0;
    i_hi = at[1] > i_lo ? at[1] : i_lo + 1;
  }
  uint32_t nibble[kStrips] = {};
  if (i_hi - i_lo == 1 && w0 + kSelPerWave <= n_end) {          // wavefront-uniform: one rollout
    const int64_t start = m.cu[i_lo], t_first = w0 - start;
    const int scheme = kPoisson ? NAT_SCHEME_URS : m.cut_in ? NAT_SCHEME_DET : a.scheme_per_rollout ? a.scheme_per_rollout[i_lo] : a.scheme;
    const bool dropped = a.drop_zero_adv && a.drop_zero_adv[i_lo] == 0.f;
    if (dropped) {
    } else if (scheme == NAT_SCHEME_URS) {
      const int shift = (int)(t_first & 3);
      const uint32_t first = (uint32_t)(t_first >> 2) + lane, id = (uint32_t)(a.rollout_id_base + i_lo);
      u32x4 r = philox4x32_10(u32x4{first, id, 0u, a.step}, a.key0, a.key1), r_next{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < kStrips; ++j) {
        double p[4];
        if (kPoisson) {
          const double* q = m.pi + w0 + kStrip * j + 4 * lane;
          if (m.pi_wide) {
            const double2 x = *reinterpret_cast<const double2*>(q), y = *reinterpret_cast<const double2*>(q + 2);
            p[0] = x.x; p[1] = x.y; p[2] = y.x; p[3] = y.y;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = q[e];
          }
        }
        if (j + 1 < kStrips || shift) r_next = philox4x32_10(u32x4{first + 64u * (j + 1), id, 0u, a.step}, a.key0, a.key1);
        uint32_t w[4] = {r.x, r.y, r.z, r.w};
        if (shift) {                               // words shift.. of this block, then the first ones of the next
          const uint32_t up[3] = {(uint32_t)__shfl_down((int)r.x, 1), (uint32_t)__shfl_down((int)r.y, 1), (uint32_t)__shfl_down((int)r.z, 1)};
          const uint32_t f0 = __builtin_amdgcn_readfirstlane(r_next.x), f1 = __builtin_amdgcn_readfirstlane(r_next.y),
                         f2 = __builtin_amdgcn_readfirstlane(r_next.z);
          const uint32_t n0 = lane == 63 ? f0 : up[0], n1 = lane == 63 ? f1 : up[1], n2 = lane == 63 ? f2 : up[2];
          if (shift == 1) { w[0] = r.y; w[1] = r.z; w[2] = r.w; w[3] = n0; }
          else if (shift == 2) { w[0] = r.z; w[1] = r.w; w[2] = n0; w[3] = n1; }
          else { w[0] = r.w; w[1] = n0; w[2] = n1; w[3] = n2; }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (kPoisson ? poisson_keep(w[e], p[e]) : (uint64_t)w[e] < a.urs_threshold) nibble[j] |= 1u << e;
        r = r_next;
      }
    } else {
      const int64_t cut = m.cut_in ? (int64_t)m.cut_in[i_lo] : rollout_cut(a, scheme, i_lo, m.cu[i_lo + 1] - start);
#pragma unroll
      for (int j = 0; j < kStrips; ++j) {
        const int64_t left = cut - (t_first + kStrip * j + 4 * lane);    // kept positions from this lane's first one on
        nibble[j] = left >= 4 ? 15u : left <= 0 ? 0u : (1u << left) - 1u;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < kStrips; ++j) {
      const int64_t n0 = w0 + kStrip * j + 4 * lane;
      if (n0 >= n_end) continue;
      int i = rollout_of_pos(m.cu, i_lo, i_hi, n0);
      int64_t start = 0, end = n0, cut = 0;        // of rollout i, set below
      int scheme = 0;
      bool dropped = false;
      u32x4 r{0u, 0u, 0u, 0u};
      int64_t have_block = -1;                     // index (t0 >> 2) of the block held in r, for rollout i
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t n = n0 + e;
        if (n >= n_end) break;
        if (n >= end) {                            // the first, or the next non-empty rollout (n < cu[B]: one exists below B)
          if (e > 0) do { ++i; } while (i < m.B - 1 && m.cu[i + 1] <= n);
          start = m.cu[i];
          end = m.cu[i + 1];
          scheme = kPoisson ? NAT_SCHEME_URS : m.cut_in ? NAT_SCHEME_DET : a.scheme_per_rollout ? a.scheme_per_rollout[i] : a.scheme;
          dropped = a.drop_zero_adv && a.drop_zero_adv[i] == 0.f;
          cut = scheme == NAT_SCHEME_URS ? 0 : m.cut_in ? (int64_t)m.cut_in[i] : rollout_cut(a, scheme, i, end - start);
          have_block = -1;
        }
        const int64_t t0 = n - start;
        bool keep;
        if (scheme == NAT_SCHEME_URS) {
          if ((t0 >> 2) != have_block) {
            have_block = t0 >> 2;
            r = philox4x32_10(u32x4{(uint32_t)have_block, (uint32_t)(a.rollout_id_base + i), 0u, a.step}, a.key0, a.key1);
          }
          const uint32_t word = (t0 & 3) == 0 ? r.x : (t0 & 3) == 1 ? r.y : (t0 & 3) == 2 ? r.z : r.w;
          keep = kPoisson ? poisson_keep(word, m.pi[n]) : (uint64_t)word < a.urs_threshold;
        } else {
          keep = t0 < cut;
        }
        if (keep && !dropped) nibble[j] |= 1u << e;
      }
    }
  }
  // the nibbles of eight lanes make a word; the mask has 2 ceil(N / 64) of them
#pragma unroll
  for (int j = 0; j < kStrips; ++j) {
    uint32_t v = nibble[j] << (4 * (lane & 7));
    v |= __shfl_xor((int)v, 1);
    v |= __shfl_xor((int)v, 2);
    v |= __shfl_xor((int)v, 4);
    const int64_t word = (w0 + kStrip * j) / 32 + (lane >> 3);
    if ((lane & 7) == 0 && (word >> 1) * 64 < m.N) m.mask_bits[word] = v;
  }
}

nat_status validate_select(const nat_select_params* p, SelectArgs* out) {
  if (!p) return NAT_INVALID_ARG;
  if (p->scheme < NAT_SCHEME_FULL || p->scheme > NAT_SCHEME_DET) return NAT_INVALID_ARG;
  if (!(p->p > 0.0 && p->p <= 1.0)) return NAT_INVALID_ARG;
  if (p->min_cut < 1) return NAT_INVALID_ARG;
  if (!(p->trunc_frac > 0.0 && p->trunc_frac <= 1.0)) return NAT_INVALID_ARG;
  out->scheme = p->scheme;
  out->min_cut = p->min_cut;
  out->p = p->p;
  out->trunc_frac = p->trunc_frac;
  out->urs_threshold = (uint64_t)floor(p->p * 4294967296.0);
  out->key0 = (uint32_t)(p->seed & 0xFFFFFFFFull);
  out->key1 = (uint32_t)(p->seed >> 32);
  out->step = p->step;
  out->rollout_id_base = p->rollout_id_base;
  out->scheme_per_rollout = p->d_scheme_per_rollout;
  out->drop_zero_adv = p->d_drop_zero_adv;
  return NAT_OK;
}

// Strips per wavefront.  Where rollouts are short a wavefront's strips are a chain of searches, so a batch that does not
// fill the chip is cut into more wavefronts; a large one shares the span's search and the straddling Philox blocks
// over more strips.  1 / 2 / 4 strips, us: Poisson, rollouts of 16: 2^18 positions 5.0 / 6.3 / 10.5, 2^20 6.7 / 7.4 / 10.7,
// 2^21 10.1 / 9.4 / 12.6, 2^23 37 / 30 / 36, 2^25 167 / 136 / 133; RPC, rollouts of 300: 2^20 5.0 / 5.0 / 6.8, 2^21 7.5 / 6.5 / 7.8,
// 2^22 11.6 / 10.0 / 9.6, 2^23 21.0 / 16.5 / 15.5.  The fp64 thresholds of a Poisson mask make two strips the better
// ones up to 2^23.
static int strips_of(int64_t N, bool poisson) {
  if (N <= (int64_t(1) << 20)) return 1;
  return N <= (int64_t(1) << (poisson ? 23 : 21)) ? 2 : 4;
}

// One launch of the mask kernel; further blocks draw the cut lengths where they are asked for.
template <bool kPoisson>
static nat_status launch_mask(const SelectArgs& a, MaskArgs m, hipStream_t s) {
  auto go = [&](auto strips) {
    constexpr int kStrips = decltype(strips)::value, kPerBlock = 4 * kStrips * kStrip;
    m.mask_blocks = (unsigned)((m.N + kPerBlock - 1) / kPerBlock);
    const unsigned cut_blocks = m.cut_out ? (unsigned)((m.B + 255) / 256) : 0;
    select_mask_kernel<kPoisson, kStrips><<<m.mask_blocks + cut_blocks, 256, 0, s>>>(a, m);
  };
  const int strips = strips_of(m.N, kPoisson);
  if (strips == 1) go(std::integral_constant<int, 1>{});
  else if (strips == 2) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 4>{});
  NAT_LAUNCH_CHECK();
  return NAT_OK;
}

nat_status launch_prefix_mask(const int64_t* d_cu, int32_t B, int64_t N, const int32_t* d_cut_len,
                              uint32_t* d_mask_bits, hipStream_t s) {
  if (N <= 0) return NAT_OK;
  return launch_mask<false>(SelectArgs{}, MaskArgs{d_cu, B, N, d_cut_len, nullptr, nullptr, 0, 0, d_mask_bits}, s);
}

nat_status launch_poisson_mask(const SelectArgs& a, const double* d_pi, const int64_t* d_cu, int32_t B, int64_t N,
                               uint32_t* d_mask_bits, hipStream_t s) {
  if (N <= 0) return NAT_OK;
  const int pi_wide = ((uintptr_t)d_pi & 15) == 0;
  return launch_mask<true>(a, MaskArgs{d_cu, B, N, nullptr, nullptr, d_pi, pi_wide, 0, d_mask_bits}, s);
}

}  // namespace nat

using namespace nat;

extern "C" nat_status nat_advantage(const float* d_rewards, int32_t P, int32_t G, float eps_adv,
                                    float* d_adv, void* stream) {
  if (!d_rewards || !d_adv || P <= 0 || G <= 0 || !(eps_adv >= 0.f)) return NAT_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  ProfScope prof(PC_ADVANTAGE, s);
  const int waves_per_block = 4;
  advantage_kernel<<<(P + waves_per_block - 1) / waves_per_block, 64 * waves_per_block, 0, s>>>(
      d_rewards, P, G, eps_adv, d_adv);
  NAT_LAUNCH_CHECK();
  return NAT_OK;
}

extern "C" int64_t nat_mask_words(int64_t N) { return N <= 0 ? 0 : 2 * ((N + 63) / 64); }

extern "C" nat_status nat_select(const nat_select_params* params, const int64_t* d_cu_seqlens, int32_t B,
                                 int64_t N, int32_t* d_cut_len, uint32_t* d_mask_bits, void* stream) {
  SelectArgs a;
  nat_status st = validate_select(params, &a);
  if (st != NAT_OK) return st;
  if (!d_cu_seqlens || !d_cut_len || B <= 0 || N < 0 || N >= (int64_t(1) << 31)) return NAT_INVALID_ARG;
  if (N > 0 && !d_mask_bits) return NAT_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  ProfScope prof(PC_SELECT, s);
  return launch_mask<false>(a, MaskArgs{d_cu_seqlens, B, N, nullptr, d_cut_len, nullptr, 0, 0, d_mask_bits}, s);
}
