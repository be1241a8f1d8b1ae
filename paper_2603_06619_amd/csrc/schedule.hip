// nat_select_schedule: cut L_i drawn from an arbitrary cut-length distribution
// q_i given as integer weights, mask 1{t <= L_i} and survival function
// p_{i,t} = sum_{l >= t} q_i(l) (Sec. 4, Eq. 7-8).
// nat_select_poisson: independent Bernoulli(p_{i,t}) masks with caller-supplied
// probabilities (Sec. 3.1).
// nat_prefix_pack: the truncated batch (prompt + kept prefix per rollout) a model
// body needs to run only over kept prefixes (Sec. 4, forward truncation).
#include "nat_internal.h"
#include "philox.hip.h"

#include <type_traits>

namespace nat {

// Threads of schedule_cut_kernel's block (one block per rollout).  1024 where a rollout's chain of block scans is the
// time: rollouts longer than 1024 on average and no more of them than compute units, or two or three times as many
// very long ones.  With more rollouts blocks of 256 share the compute units better.  Whole call, 256 / 1024 threads, us:
// mean length 1500: 128 rollouts 10.2 / 9.0, 512 12.2 / 14.3, 16384 148 / 319; 4000: 128 15.8 / 12.1, 512 21.9 / 23.3,
// 2048 47 / 71; 8000: 256 30 / 21, 512 39 / 37, 768 48 / 52, 2048 81 / 112; 16000: 768 97 / 92, 1024 116 / 123; 30000: 512
// 144 / 116, 768 176 / 169, 1024 237 / 249.
static int schedule_threads(int64_t N, int32_t B) {
  const int64_t mean = N / B;
  return (mean > 1024 && B <= 256) || (mean > 6000 && B <= 512) || (mean > 12000 && B <= 768) ? 1024 : 256;
}

// Inclusive scan of one 64-bit value per thread over the block; *total = block sum.
// `wave_tot` is a word of LDS per wavefront; the caller separates successive calls with a barrier.
template <int kThreads>
__device__ __forceinline__ uint64_t block_scan_u64(uint64_t v, uint64_t* wave_tot, uint64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t incl = v;
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t up = __shfl_up((unsigned long long)incl, off);
    if (lane >= off) incl += up;
  }
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint64_t before = 0, all = 0;
  for (int w = 0; w < kThreads / 64; ++w) {
    const uint64_t t = wave_tot[w];
    if (w < wave) before += t;
    all += t;
  }
  *total = all;
  return before + incl;
}

// One block per rollout: total weight, the cut by inversion of the running sum, and the
// survival function for every position.  Bound by the chain of block scans over the longest rollout (4 positions per
// thread and scan) in a small batch, by the bytes in a large one.  See schedule_threads.
template <int kThreads>
__global__ void __launch_bounds__(kThreads)
schedule_cut_kernel(uint32_t key0, uint32_t key1, uint32_t step, int32_t rollout_id_base,
                    const float* __restrict__ drop_zero_adv,
                    const uint32_t* __restrict__ weights, const int64_t* __restrict__ cu, int64_t N,
                    int32_t* __restrict__ cut_len, double* __restrict__ pi) {
  __shared__ uint64_t wave_tot[kThreads / 64];
  const int i = blockIdx.x;
  // offsets are clamped to the N positions the caller's arrays hold
  const int64_t start = cu[i] < 0 ? 0 : cu[i] > N ? N : cu[i];
  const int64_t stop = cu[i + 1] > N ? N : cu[i + 1];
  const int64_t T = stop - start;
  if (T <= 0) {
    if (threadIdx.x == 0) cut_len[i] = 0;
    return;
  }
  const uint32_t* a = weights + start;
  double* p = pi + start;

  uint64_t part = 0;
  for (int64_t j = threadIdx.x; j < T; j += kThreads) part += a[j];
  uint64_t A;
  block_scan_u64<kThreads>(part, wave_tot, &A);
  __syncthreads();
  if (A == 0) {                                   // no schedule: keep the rollout whole, p = 1
    for (int64_t j = threadIdx.x; j < T; j += kThreads) p[j] = 1.0;
    if (threadIdx.x == 0) cut_len[i] = (drop_zero_adv && drop_zero_adv[i] == 0.f) ? 0 : (int32_t)T;
    return;
  }
  const u32x4 rnd = philox4x32_10(u32x4{0u, (uint32_t)(rollout_id_base + i), 2u, step}, key0, key1);
  uint64_t r = __umul64hi(((uint64_t)rnd.x << 32) | (uint64_t)rnd.y, A);         // in [0, A)
  const bool dropped = drop_zero_adv && drop_zero_adv[i] == 0.f;                 // keeps nothing: no position
  if (dropped) {                                                                 // qualifies below
    r = ~0ull;
    if (threadIdx.x == 0) cut_len[i] = 0;
  }

  const double den = (double)A;
  uint64_t carry = 0;                              // running sum of all earlier positions
  constexpr int kPer = 4;                          // consecutive positions per thread and iteration
  for (int64_t base = 0; base < T; base += kThreads * kPer) {
    const int64_t j0 = base + (int64_t)threadIdx.x * kPer;
    uint32_t v[kPer];
    uint64_t mine = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      v[e] = j0 + e < T ? a[j0 + e] : 0u;
      mine += v[e];
    }
    uint64_t chunk_total;
    uint64_t run = carry + block_scan_u64<kThreads>(mine, wave_tot, &chunk_total) - mine;   // sum of positions before j0
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (j0 + e < T) {
        p[j0 + e] = (double)(A - run) / den;      // sum_{l >= t} a_l over A, exact integers below 2^53
        if (run <= r && r < run + v[e]) cut_len[i] = (int32_t)(j0 + e + 1);   // exactly one position qualifies
      }
      run += v[e];
    }
    carry += chunk_total;
    __syncthreads();
  }
}

// cu_packed = exclusive scan of P_i + L_i, cu_loss = exclusive scan of L_i, totals = (rows, longest).
__global__ void __launch_bounds__(1024)
prefix_scan_kernel(const int32_t* __restrict__ prompt_len, const int64_t* __restrict__ cu,
                   const int32_t* __restrict__ cut_len, int B, int32_t* __restrict__ cu_packed,
                   int32_t* __restrict__ cu_loss, int32_t* __restrict__ totals, int32_t* __restrict__ h_totals) {
  __shared__ int wave_rows[16], wave_loss[16], wave_max[16];
  __shared__ int carry_rows, carry_loss;
  if (threadIdx.x == 0) { carry_rows = 0; carry_loss = 0; }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int longest = 0;
  for (int base = 0; base < B; base += 1024) {
    const int i = base + threadIdx.x;
    int L = 0, rows = 0;
    if (i < B) {
      const int64_t T = cu[i + 1] - cu[i];
      const int64_t c = cut_len[i];
      L = (int)(c < 0 ? 0 : c > T ? T : c);
      rows = (prompt_len ? prompt_len[i] : 0) + L;
      longest = rows > longest ? rows : longest;
    }
    int in_rows = rows, in_loss = L;
    for (int off = 1; off < 64; off <<= 1) {
      const int ur = __shfl_up(in_rows, off), ul = __shfl_up(in_loss, off);
      if (lane >= off) { in_rows += ur; in_loss += ul; }
    }
    if (lane == 63) { wave_rows[wave] = in_rows; wave_loss[wave] = in_loss; }
    __syncthreads();
    int before_rows = carry_rows, before_loss = carry_loss;
    for (int w = 0; w < wave; ++w) { before_rows += wave_rows[w]; before_loss += wave_loss[w]; }
    if (i < B) { cu_packed[i] = before_rows + in_rows - rows; cu_loss[i] = before_loss + in_loss - L; }
    __syncthreads();
    if (threadIdx.x == 1023) { carry_rows = before_rows + in_rows; carry_loss = before_loss + in_loss; }
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) { const int o = __shfl_xor(longest, off); longest = o > longest ? o : longest; }
  if (lane == 0) wave_max[wave] = longest;
  __syncthreads();
  if (threadIdx.x == 0) {
    int m = 0;
    for (int w = 0; w < 16; ++w) m = wave_max[w] > m ? wave_max[w] : m;
    cu_packed[B] = carry_rows;
    cu_loss[B] = carry_loss;
    totals[0] = carry_rows;
    totals[1] = m;
    if (h_totals) {
      host_store(h_totals, carry_rows);
      host_store(h_totals + 1, m);
    }
  }
}

// One lane per row of the truncated batch.
__global__ void __launch_bounds__(256)
prefix_rows_kernel(const int32_t* __restrict__ prompt_len, const int64_t* __restrict__ cu, int B, int shift,
                   int64_t rows_cap, int64_t kept_cap, const int32_t* __restrict__ cu_packed,
                   const int32_t* __restrict__ cu_loss, int32_t* __restrict__ src_idx,
                   int32_t* __restrict__ position_ids, int32_t* __restrict__ loss_row,
                   const int32_t* __restrict__ input_ids, int32_t* __restrict__ input_ids_packed) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= rows_cap || m >= (int64_t)cu_packed[B]) return;
  const int i = rollout_of_pos(cu_packed, 0, B, m);
  const int j = (int)(m - cu_packed[i]);
  const int P = prompt_len ? prompt_len[i] : 0;
  // rows of the full input before rollout i: all earlier prompts and all earlier full responses
  const int64_t full_start = (int64_t)(cu_packed[i] - cu_loss[i]) + cu[i];
  const int64_t src = full_start + j;
  src_idx[m] = (int32_t)src;
  position_ids[m] = j;
  if (input_ids) input_ids_packed[m] = input_ids[src];
  if (j >= P) {
    const int64_t k = (int64_t)cu_loss[i] + (j - P);
    if (k < kept_cap) loss_row[k] = (int32_t)(m - shift);
  }
}

// Both of the above in one launch, for up to kScanRollouts rollouts: every block scans them itself, four to a thread (three loads and two barriers),
// and finds its rows' rollouts in LDS instead of by a chain of loads; the first one writes the offsets and totals.  At most kPackBlocks blocks, eight to a
// compute unit, take all rows between them, so that the scan is paid once.  Two launches / this one with 1024 / 2048 / 4096 blocks, us: 0.32 million
// rows 10.5 / 7.4 / 7.1 / 7.5, 2.3 20.0 / 16.4 / 17.3 / 22.9, 8.6 42.6 / 31.8 / 27.6 / 32.2, 19 125.8 / 79.5 / 64.0 / 66.8 (19 with a block per 256 rows: 127).
constexpr int kScanRollouts = 1024, kPackBlocks = 2048;
__global__ void __launch_bounds__(256)
prefix_pack_kernel(const int32_t* __restrict__ prompt_len, const int64_t* __restrict__ cu, const int32_t* __restrict__ cut_len, int B, int shift,
                   int64_t rows_cap, int64_t kept_cap, int32_t* __restrict__ cu_packed, int32_t* __restrict__ cu_loss,
                   int32_t* __restrict__ totals, int32_t* __restrict__ h_totals, int32_t* __restrict__ src_idx, int32_t* __restrict__ position_ids,
                   int32_t* __restrict__ loss_row, const int32_t* __restrict__ input_ids, int32_t* __restrict__ input_ids_packed) {
  constexpr int kPer = kScanRollouts / 256;
  __shared__ int at_row[kScanRollouts + 1], at_loss[kScanRollouts + 1], wave_rows[4], wave_loss[4], wave_max[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i0 = threadIdx.x * kPer;
  int L[kPer], rows[kPer], in_rows = 0, in_loss = 0, longest = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    L[e] = rows[e] = 0;
    if (i0 + e < B) {
      const int64_t T = cu[i0 + e + 1] - cu[i0 + e], c = cut_len[i0 + e];
      L[e] = (int)(c < 0 ? 0 : c > T ? T : c);
      rows[e] = (prompt_len ? prompt_len[i0 + e] : 0) + L[e];
      longest = rows[e] > longest ? rows[e] : longest;
    }
    in_rows += rows[e];
    in_loss += L[e];
  }
  int run_rows = -in_rows, run_loss = -in_loss;              // the scan includes this thread's own
  for (int off = 1; off < 64; off <<= 1) {
    const int ur = __shfl_up(in_rows, off), ul = __shfl_up(in_loss, off);
    if (lane >= off) { in_rows += ur; in_loss += ul; }
  }
  for (int off = 32; off > 0; off >>= 1) { const int o = __shfl_xor(longest, off); longest = o > longest ? o : longest; }
  if (lane == 63) { wave_rows[wave] = in_rows; wave_loss[wave] = in_loss; wave_max[wave] = longest; }
  __syncthreads();
  run_rows += in_rows;
  run_loss += in_loss;
  for (int w = 0; w < wave; ++w) { run_rows += wave_rows[w]; run_loss += wave_loss[w]; }
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (i0 + e < B) { at_row[i0 + e] = run_rows; at_loss[i0 + e] = run_loss; }
    run_rows += rows[e];
    run_loss += L[e];
    if (i0 + e == B - 1) { at_row[B] = run_rows; at_loss[B] = run_loss; }
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i <= B; i += 256) { cu_packed[i] = at_row[i]; cu_loss[i] = at_loss[i]; }
    if (threadIdx.x == 0) {
      int m = 0;
      for (int w = 0; w < 4; ++w) m = wave_max[w] > m ? wave_max[w] : m;
      totals[0] = at_row[B];
      totals[1] = m;
      if (h_totals) {
        host_store(h_totals, at_row[B]);
        host_store(h_totals + 1, m);
      }
    }
  }
  const int64_t n_rows = rows_cap < at_row[B] ? rows_cap : at_row[B];
  for (int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x; m < n_rows; m += (int64_t)gridDim.x * 256) {
    const int i = rollout_of_pos(at_row, 0, B, m), row0 = at_row[i], loss0 = at_loss[i];
    const int j = (int)(m - row0), P = prompt_len ? prompt_len[i] : 0;
    const int64_t src = (int64_t)(row0 - loss0) + cu[i] + j;   // behind all earlier prompts and all earlier full responses
    src_idx[m] = (int32_t)src;
    position_ids[m] = j;
    if (input_ids) input_ids_packed[m] = input_ids[src];
    if (j >= P) {
      const int64_t k = (int64_t)loss0 + (j - P);
      if (k < kept_cap) loss_row[k] = (int32_t)(m - shift);
    }
  }
}

}  // namespace nat

using namespace nat;

static nat_status check_common(const nat_select_params* params, const void* a, const int64_t* cu, int32_t B,
                               int64_t N) {
  if (!params || !cu || B <= 0 || N < 0 || N >= (int64_t(1) << 31)) return NAT_INVALID_ARG;
  if (N > 0 && !a) return NAT_INVALID_ARG;
  return NAT_OK;
}

extern "C" nat_status nat_select_schedule(const nat_select_params* params, const uint32_t* d_weights,
                                          const int64_t* d_cu_seqlens, int32_t B, int64_t N,
                                          int32_t* d_cut_len, uint32_t* d_mask_bits, double* d_pi, void* stream) {
  nat_status st = check_common(params, d_weights, d_cu_seqlens, B, N);
  if (st != NAT_OK) return st;
  if (!d_cut_len || (N > 0 && (!d_mask_bits || !d_pi))) return NAT_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  ProfScope prof(PC_SCHEDULE, s);
  auto go = [&](auto threads) {
    constexpr int kThreads = decltype(threads)::value;
    schedule_cut_kernel<kThreads><<<(unsigned)B, kThreads, 0, s>>>(
        (uint32_t)(params->seed & 0xFFFFFFFFull), (uint32_t)(params->seed >> 32), params->step,
        params->rollout_id_base, params->d_drop_zero_adv, d_weights, d_cu_seqlens, N, d_cut_len, d_pi);
  };
  if (schedule_threads(N, B) == 1024) go(std::integral_constant<int, 1024>{});
  else go(std::integral_constant<int, 256>{});
  NAT_LAUNCH_CHECK();
  return launch_prefix_mask(d_cu_seqlens, B, N, d_cut_len, d_mask_bits, s);
}

extern "C" nat_status nat_select_poisson(const nat_select_params* params, const double* d_pi,
                                         const int64_t* d_cu_seqlens, int32_t B, int64_t N,
                                         uint32_t* d_mask_bits, void* stream) {
  nat_status st = check_common(params, d_pi, d_cu_seqlens, B, N);
  if (st != NAT_OK) return st;
  if (N > 0 && !d_mask_bits) return NAT_INVALID_ARG;
  if (N == 0) return NAT_OK;
  hipStream_t s = (hipStream_t)stream;
  ProfScope prof(PC_SCHEDULE, s);
  SelectArgs a{};
  a.key0 = (uint32_t)(params->seed & 0xFFFFFFFFull);
  a.key1 = (uint32_t)(params->seed >> 32);
  a.step = params->step;
  a.rollout_id_base = params->rollout_id_base;
  a.drop_zero_adv = params->d_drop_zero_adv;
  return launch_poisson_mask(a, d_pi, d_cu_seqlens, B, N, d_mask_bits, s);
}

extern "C" nat_status nat_prefix_pack(const int32_t* d_prompt_len, const int64_t* d_cu_seqlens,
                                      const int32_t* d_cut_len, int32_t B, int32_t next_token_shift,
                                      int64_t rows_cap, int64_t kept_cap,
                                      int32_t* d_cu_packed, int32_t* d_cu_loss, int32_t* d_src_idx,
                                      int32_t* d_position_ids, int32_t* d_loss_row, int32_t* d_totals,
                                      int32_t* h_totals, const int32_t* d_input_ids,
                                      int32_t* d_input_ids_packed, void* stream) {
  if (!d_cu_seqlens || !d_cut_len || !d_cu_packed || !d_cu_loss || !d_totals || B <= 0 || rows_cap < 0 ||
      kept_cap < 0 || rows_cap >= (int64_t(1) << 31) || kept_cap >= (int64_t(1) << 31))
    return NAT_INVALID_ARG;
  if (next_token_shift != 0 && next_token_shift != 1) return NAT_INVALID_ARG;
  if (next_token_shift == 1 && !d_prompt_len) return NAT_INVALID_ARG;
  if (rows_cap > 0 && (!d_src_idx || !d_position_ids)) return NAT_INVALID_ARG;
  if (rows_cap > 0 && kept_cap > 0 && !d_loss_row) return NAT_INVALID_ARG;
  if ((d_input_ids != nullptr) != (d_input_ids_packed != nullptr)) return NAT_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  int32_t* pinned = pinned_words(h_totals);
  {
    ProfScope prof(PC_PREFIX_PACK, s);
    if (B <= kScanRollouts) {
      const int64_t blocks = rows_cap > 0 ? (rows_cap + 255) / 256 : 1;
      prefix_pack_kernel<<<(unsigned)(blocks < kPackBlocks ? blocks : kPackBlocks), 256, 0, s>>>(d_prompt_len, d_cu_seqlens, d_cut_len, B, next_token_shift, rows_cap, kept_cap, d_cu_packed,
                                                          d_cu_loss, d_totals, pinned, d_src_idx, d_position_ids, d_loss_row, d_input_ids,
                                                          d_input_ids_packed);
      NAT_LAUNCH_CHECK();
    } else {
      prefix_scan_kernel<<<1, 1024, 0, s>>>(d_prompt_len, d_cu_seqlens, d_cut_len, B, d_cu_packed, d_cu_loss, d_totals, pinned);
      NAT_LAUNCH_CHECK();
      if (rows_cap > 0) {
        prefix_rows_kernel<<<(unsigned)((rows_cap + 255) / 256), 256, 0, s>>>(
            d_prompt_len, d_cu_seqlens, B, next_token_shift, rows_cap, kept_cap, d_cu_packed, d_cu_loss, d_src_idx,
            d_position_ids, d_loss_row, d_input_ids, d_input_ids_packed);
        NAT_LAUNCH_CHECK();
      }
    }
  }
  if (h_totals && !pinned) NAT_HIP_TRY(hipMemcpyAsync(h_totals, d_totals, 2 * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  return NAT_OK;
}
