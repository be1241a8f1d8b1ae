// fp32 path of nat_loss_fwd_bwd and nat_logp_fwd (small heads: the tiny fp32 workload, gradient
// checks), one token chunk at a time:
//   logits    z = H W^T                         (f32_gemm_kernel)
//   token     log-sum-exp with the true row maximum, log-prob of the target, ratio / clipped
//             surrogate (Eq. 1, Eq. 3), then dz = c (onehot - softmax) over z;
//   dH        dH = dz W                         (f32_gemm_kernel)
//   dW        dW (+)= dz^T H, chunks in order   (f32_gemm_kernel)
// Every sum has a fixed order.
#include "nat_internal.h"
#include "grpo_scalar.hip.h"

#include <type_traits>

namespace nat {

constexpr int kF32Threads = 256;
// Larger hidden sizes have always been refused on this path, and are; its kernels have no such bound of their own.
constexpr int kF32MaxHidden = 15360;

__device__ __forceinline__ float wave_max_f(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// ------------------------------------------------------------------- GEMM ----
// C[m][n] = sum_k A(m, k) B(n, k) in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and
// sums, 157 TFLOP/s against 79 for unpacked vector FMAs).  One workgroup per 32 x 32 tile of C: the problems
// of this path are small (a 601 x 256 dH has 152 such tiles for 256 CUs, and a contraction of 4096), so
// the contraction axis is split over the eight wavefronts of the workgroup, whose partial tiles are added in
// order through LDS.  Each wavefront streams its own range of k from memory (L2) 32 at a time, the loads of the
// next 32 in flight under the products of the current ones; nothing in the loop waits for another wavefront.
// An MFMA operand of a lane is (row l % 32, k = 8 (j / 4) + 4 (l / 32) + j % 4 for product j of a step), the same k
// for both operands.  A k-major operand is read as that, 32 consecutive floats per half-wavefront.  A
// k-contiguous one is read in whole 128-byte pieces of its rows and turned through the wavefront's own LDS (read
// lane by lane from 32 rows at once it cost four times the address cycles and bound the kernel).
// The logits (both operands k-contiguous) are summed in groups of 8 products, a wavefront's groups in a chain of H / 64 and the
// wavefronts in fp64: no logit is rounded more often than by 64 lanes with H / 64 products each and a tree over them
// (in one chain of H / 8 per wavefront its error was 1.5 times that at H = 256, 2.6 times at H = 4096; the groups cost the
// launch 1.5 of 28 us at H = 256, 5 of 65 at H = 1024).  Operands are then read four products at a time: with all
// sixteen in registers the kernel needs 163, and only one workgroup fits a compute unit (35 us).
// Measured at 601 tokens, V = 4096, H = 256: logits 27 us, dH 31 us, dW 30 us (44 TFLOP/s; latency of the short
// ranges); one block per token (logits, dH) and per vocabulary row (dW) on the vector ALU took 2500 us for the three.
// 64 x 64 tiles (half the reads) and sixteen wavefronts were slower or equal.
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kF32Waves = 8, kF32Step = 32;
constexpr int kF32Row = 36;      // floats per LDS row of 32: 16-byte aligned, and 16 rows at one k cover all 64 banks once

// operand (row, k): k-contiguous (KMajor = false) p[row * ld + k], k-major p[k * ld + row]; rows past the end
// read the last one.  Vec: 16-byte loads (leading dimension a multiple of 4; bases are 16-byte aligned).
template <bool KMajor, bool Vec>
struct F32Operand {
  const float* p;
  int64_t ld;
  int row0, rows, lane;
  float* turn;                   // [32][kF32Row] of this wavefront (k-contiguous operands)

  // raw values of the 32 k from k0 on; kTail: entries at or beyond k_end are zero (read from the last valid
  // place; with Vec, k_end is a multiple of 4: the contraction's length is the leading dimension)
  template <bool kTail>
  __device__ __forceinline__ void fetch(float (&r)[16], int k0, int k_end) const {
    auto row_of = [&](int i) { return (int64_t)(row0 + i < rows ? row0 + i : rows - 1); };
    if constexpr (KMajor) {
      const float* col = p + row_of(lane & 31);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int k = k0 + 8 * (j >> 2) + 4 * (lane >> 5) + (j & 3);
        const float x = col[(int64_t)(!kTail || k < k_end ? k : k_end - 1) * ld];
        r[j] = !kTail || k < k_end ? x : 0.f;
      }
    } else if constexpr (Vec) {
      const int k = k0 + 4 * (lane & 7);
      const bool in = !kTail || k < k_end;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 x = *reinterpret_cast<const float4*>(p + row_of(8 * i + (lane >> 3)) * ld + (in ? k : k_end - 4));
        r[4 * i] = in ? x.x : 0.f; r[4 * i + 1] = in ? x.y : 0.f; r[4 * i + 2] = in ? x.z : 0.f; r[4 * i + 3] = in ? x.w : 0.f;
      }
    } else {
      const int k = k0 + (lane & 31);
      const bool in = !kTail || k < k_end;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float x = p[row_of(2 * i + (lane >> 5)) * ld + (in ? k : k_end - 1)];
        r[i] = in ? x : 0.f;
      }
    }
  }
  // LDS operations of one wavefront execute in order: no barrier between its writes and its reads
  __device__ __forceinline__ void put(const float (&r)[16]) const {
    if constexpr (!KMajor && Vec) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<float4*>(turn + (8 * i + (lane >> 3)) * kF32Row + 4 * (lane & 7)) = make_float4(r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]);
    } else if constexpr (!KMajor) {
#pragma unroll
      for (int i = 0; i < 16; ++i) turn[(2 * i + (lane >> 5)) * kF32Row + (lane & 31)] = r[i];
    }
  }
  // operands of products 4 q .. 4 q + 3 of a step (k-contiguous)
  __device__ __forceinline__ float4 read4(int q) const {
    return *reinterpret_cast<const float4*>(turn + (lane & 31) * kF32Row + 8 * q + 4 * (lane >> 5));
  }
  __device__ __forceinline__ void get(const float (&r)[16], float (&v)[16]) const {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (KMajor) {
        v[4 * q] = r[4 * q]; v[4 * q + 1] = r[4 * q + 1]; v[4 * q + 2] = r[4 * q + 2]; v[4 * q + 3] = r[4 * q + 3];
      } else {
        const float4 x = read4(q);
        v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
      }
    }
  }
};

template <bool KMajorA, bool KMajorB, bool Vec>
__global__ void __launch_bounds__(kF32Waves * 64, !KMajorA && !KMajorB && Vec ? 4 : 1)   // logits: two workgroups per compute unit
f32_gemm_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, int M, int N, int K,
                int tiles_n, float* __restrict__ C, int64_t ldc, int accumulate) {
  constexpr bool kGroups = !KMajorA && !KMajorB;             // the logits
  constexpr int kTurn = 32 * kF32Row, kTurns = (KMajorA ? 0 : 1) + (KMajorB ? 0 : 1), kPart = 32 * 33;
  __shared__ __attribute__((aligned(16))) float lds[kF32Waves * (kTurns * kTurn > kPart ? kTurns * kTurn : kPart)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
  const int m0 = (int)(blockIdx.x / tiles_n) * 32, n0 = (int)(blockIdx.x % tiles_n) * 32;
  float* turn = lds + wave * kTurns * kTurn;
  const F32Operand<KMajorA, Vec> a{A, lda, m0, M, lane, turn};
  const F32Operand<KMajorB, Vec> b{B, ldb, n0, N, lane, turn + (KMajorA ? 0 : kTurn)};
  const int per = ((K + kF32Waves - 1) / kF32Waves + 7) / 8 * 8;          // k per wavefront, a multiple of 8
  const int k_first = wave * per;
  const int k_end = k_first + per < K ? k_first + per : K;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  if (k_first < k_end) {
    float ra[16], rb[16], va[16], vb[16];
    auto fetch = [&](int k) {
      if (k + kF32Step <= k_end) {                            // wave-uniform
        a.template fetch<false>(ra, k, k_end);
        b.template fetch<false>(rb, k, k_end);
      } else {
        a.template fetch<true>(ra, k, k_end);
        b.template fetch<true>(rb, k, k_end);
      }
    };
    fetch(k_first);
    for (int k = k_first; k < k_end; k += kF32Step) {
      a.put(ra);
      b.put(rb);
      __builtin_amdgcn_wave_barrier();
      if constexpr (kGroups) {
        if (k + kF32Step < k_end) fetch(k + kF32Step);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 x = a.read4(q), y = b.read4(q);
          f32x16 group;
#pragma unroll
          for (int r = 0; r < 16; ++r) group[r] = 0.f;
          group = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, group, 0, 0, 0);
          group = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, group, 0, 0, 0);
          group = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, group, 0, 0, 0);
          group = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, group, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[r] += group[r];
        }
        __builtin_amdgcn_wave_barrier();
      } else {
        a.get(ra, va);
        b.get(rb, vb);
        if (k + kF32Step < k_end) fetch(k + kF32Step);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 16; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(va[j], vb[j], acc, 0, 0, 0);
      }
    }
  }
  __syncthreads();
  // acc[r] of lane l is C[m0 + 8 (r / 4) + 4 (l / 32) + r % 4][n0 + l % 32]
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[wave * kPart + (8 * (r >> 2) + 4 * lhi + (r & 3)) * 33 + l32] = acc[r];
  __syncthreads();
#pragma unroll
  for (int e = threadIdx.x; e < 1024; e += kF32Waves * 64) {
    const int i = e >> 5, j = e & 31;
    typename std::conditional<kGroups, double, float>::type s = 0;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) s += lds[w * kPart + i * 33 + j];
    if (m0 + i < M && n0 + j < N) {
      float* c = C + (int64_t)(m0 + i) * ldc + n0 + j;
      *c = accumulate ? *c + (float)s : (float)s;
    }
  }
}

// A launch holds fewer than 2^32 work-items, 2^23 tiles (of more, HIP runs what is left modulo 2^32 and reports nothing): larger
// products, a chunk of 2^33 logits, take several.
template <bool KMajorA, bool KMajorB>
static nat_status f32_gemm(const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N, int K, float* C,
                           int64_t ldc, int accumulate, hipStream_t s) {
  constexpr int64_t kMaxTiles = ((int64_t(1) << 32) - 1) / (kF32Waves * 64), kMaxCols = 1 << 20;
  // 16-byte reads of a k-contiguous operand need its rows to start on 16 bytes
  const bool vec = (KMajorA || lda % 4 == 0) && (KMajorB || ldb % 4 == 0);
  for (int64_t n0 = 0; n0 < N; n0 += kMaxCols) {
    const int cols = (int)(N - n0 < kMaxCols ? N - n0 : kMaxCols), tiles_n = (cols + 31) / 32;
    const int64_t max_rows = kMaxTiles / tiles_n * 32;
    for (int64_t m0 = 0; m0 < M; m0 += max_rows) {
      const int rows = (int)(M - m0 < max_rows ? M - m0 : max_rows);
      const unsigned grid = (unsigned)((rows + 31) / 32) * (unsigned)tiles_n;
      const float *a = A + (KMajorA ? m0 : m0 * lda), *b = B + (KMajorB ? n0 : n0 * ldb);
      float* c = C + m0 * ldc + n0;
      auto go = [&](auto wide) {
        f32_gemm_kernel<KMajorA, KMajorB, decltype(wide)::value><<<grid, kF32Waves * 64, 0, s>>>(a, lda, b, ldb, rows, cols, K, tiles_n, c, ldc, accumulate);
      };
      if constexpr (KMajorA && KMajorB) go(std::true_type{});         // no k-contiguous operand: nothing to widen
      else if (vec) go(std::true_type{});
      else go(std::false_type{});
      NAT_LAUNCH_CHECK();
    }
  }
  return NAT_OK;
}

// ------------------------------------------------------------- per token ----
// log-sum-exp pieces of one token's logits, one block per token: the maximum m, sum of e^(z-m) and of
// e^(z-m) (z-m), all threads.  The sums and what follows from them (log-sum-exp, log-prob, ratio, surrogate) are formed
// in fp64: a loss whose terms cancel is left with the rounding of its log-probs, 5e-7 each in fp32.
__device__ __forceinline__ double wave_sum_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
// A row of at most kF32RowRegs * 256 logits stays in registers between the passes over it (kRegs of them: `row`), a longer one is read again (0): with the
// loads ahead (f32_token_kernel), whole loss call at V = 4096, H = 256, us: 100 tokens 58.1 -> 55.5, 601 94.5 -> 92.3.  The passes go over all kRegs, so a
// short row has fewer.  1024 tokens, read again / sixteen always / so, us: log-probs V = 2048, H = 4 18.6 / 19.7 / 18.5, V = 700, H = 64 14.1 / 15.0 / 13.8, V = 300, H =
// 1024 20.1 / 21.2 / 19.7; loss V = 31, H = 1024 38.4 / 40.6 / 38.6, V = 1000, H = 64 43.9 / 44.0 / 42.7.
constexpr int kF32RowRegs = 16;
// launch(integral_constant) with the registers for a row of V logits: 1, 2, 4, 8 or 16, or 0
template <class F>
static void with_row_regs(int V, F&& launch) {
  if (V <= kF32Threads) launch(std::integral_constant<int, 1>{});
  else if (V <= 2 * kF32Threads) launch(std::integral_constant<int, 2>{});
  else if (V <= 4 * kF32Threads) launch(std::integral_constant<int, 4>{});
  else if (V <= 8 * kF32Threads) launch(std::integral_constant<int, 8>{});
  else if (V <= kF32RowRegs * kF32Threads) launch(std::integral_constant<int, kF32RowRegs>{});
  else launch(std::integral_constant<int, 0>{});
}
struct F32RowSums { float m; double s, t; };
struct F32RowShared { float m[4]; double s[4], t[4]; };
template <int kRegs>
__device__ __forceinline__ F32RowSums f32_row_sums(const float* __restrict__ z, int V, F32RowShared& sh, float (&row)[kRegs + 1]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float m = -INFINITY;
  if (kRegs > 0) {
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
      const int v = threadIdx.x + i * kF32Threads;
      row[i] = v < V ? z[v] : -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < kRegs; ++i) m = fmaxf(m, row[i]);
  } else {
#pragma unroll 4
    for (int v = threadIdx.x; v < V; v += kF32Threads) m = fmaxf(m, z[v]);
  }
  m = wave_max_f(m);
  if (lane == 0) sh.m[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(sh.m[0], sh.m[1]), fmaxf(sh.m[2], sh.m[3]));
  double s = 0.0, t = 0.0;
  auto add = [&](float x) {
    const float zc = x - m, e = expf(zc);
    s += (double)e;
    t = fma((double)e, (double)zc, t);
  };
  if (kRegs > 0) {
#pragma unroll
    for (int i = 0; i < kRegs; ++i)
      if ((int)threadIdx.x + i * kF32Threads < V) add(row[i]);
  } else {
#pragma unroll 4
    for (int v = threadIdx.x; v < V; v += kF32Threads) add(z[v]);
  }
  s = wave_sum_d(s);
  t = wave_sum_d(t);
  if (lane == 0) { sh.s[wave] = s; sh.t[wave] = t; }
  __syncthreads();
  return F32RowSums{m, (sh.s[0] + sh.s[1]) + (sh.s[2] + sh.s[3]), (sh.t[0] + sh.t[1]) + (sh.t[2] + sh.t[3])};
}

// One block per token.  Bound by latency: what only the first thread needs (ids, weights, the target's logit) is loaded ahead of the reductions.
template <int kRegs>
__global__ void __launch_bounds__(kF32Threads)
f32_token_kernel(const int32_t* __restrict__ ids, const float* __restrict__ old_logp, const float* __restrict__ adv,
                 const int32_t* __restrict__ kept_seq, const float* __restrict__ kept_w,
                 int chunk_start, int V, float eps_lo, float eps_hi, float grad_scale, KlArgs klp,
                 float* __restrict__ dz /*[chunk, V]: logits in, gradients out*/, float* __restrict__ logp_out,
                 float* __restrict__ term, float* __restrict__ kl_out, float* __restrict__ entropy_out,
                 int32_t* __restrict__ diag) {
  __shared__ F32RowShared sh;
  __shared__ float bcast[2];
  const int kc = blockIdx.x;                 // token within the chunk
  const int k = chunk_start + kc;
  float* z = dz + (size_t)kc * V;
  const int y = ids[k];
  const bool bad_id = y < 0 || y >= V;
  float z_y = 0.f, w = 0.f, A = 0.f, old = 0.f, ref = 0.f;
  if (!bad_id) {
    z_y = z[y];
    w = kept_w[k];
    A = adv[kept_seq[k]];
    old = old_logp[k];
    if (klp.beta != 0.f) ref = klp.ref_logp[k];
  }
  float row[kRegs + 1];
  const F32RowSums sums = f32_row_sums<kRegs>(z, V, sh, row);
  if (threadIdx.x == 0) {
    const double log_s = log(sums.s), lse = (double)sums.m + log_s;
    // -sum p log p = log(sum) - (sum of e (z - m)) / sum
    if (entropy_out) entropy_out[k] = (float)(log_s - sums.t / sums.s);
    bcast[0] = (float)lse;
    if (bad_id) {                            // no such token: left out (no loss term, zero gradient)
      if (logp_out) logp_out[k] = __builtin_nanf("");
      if (kl_out) kl_out[k] = __builtin_nanf("");
      term[k] = 0.f;
      bcast[1] = 0.f;
      if (diag) atomicAdd(diag + NAT_DIAG_BAD_ID, 1);
    } else {
      const double logp = (double)z_y - lse;
      const TokenScalars ts = grpo_token_scalars(logp, old, A, w, eps_lo, eps_hi, grad_scale, klp.beta, klp.kind, ref);
      if (logp_out) logp_out[k] = (float)logp;
      if (kl_out) kl_out[k] = ts.kl;
      term[k] = w * ts.L;
      bcast[1] = ts.c;
      if (diag) {
        if (ts.clipped) atomicAdd(diag + NAT_DIAG_CLIPPED, 1);
        if (A != 0.f) atomicAdd(diag + NAT_DIAG_NONZERO_ADV, 1);
      }
    }
  }
  __syncthreads();
  const float lse = bcast[0], c = bcast[1];
  auto put = [&](int v, float x) { z[v] = c * ((v == y ? 1.f : 0.f) - expf(x - lse)); };
  if (kRegs > 0) {
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
      const int v = threadIdx.x + i * kF32Threads;
      if (v < V) put(v, row[i]);
    }
  } else {
    for (int v = threadIdx.x; v < V; v += kF32Threads) put(v, z[v]);
  }
}

static int f32_chunk_rows(int32_t N_k, int32_t V, size_t ws_bytes) {
  const size_t fixed = (size_t)N_k * sizeof(float) + 256;
  if (ws_bytes <= fixed) return 0;
  size_t rows = (ws_bytes - fixed) / ((size_t)V * sizeof(float));
  if (rows > (size_t)N_k) rows = N_k;
  return (int)rows;
}

size_t loss_f32_workspace_bytes(int32_t N_k, int32_t H, int32_t V, bool minimal) {
  (void)H;
  int rows = N_k < 1 ? 1 : N_k;
  const int cap = minimal ? 1 : 4096;
  if (rows > cap) rows = cap;
  return (size_t)N_k * sizeof(float) + 256 + (size_t)rows * V * sizeof(float);
}

nat_status loss_f32_run(const LossArgs& a) {
  if (a.H > kF32MaxHidden) return NAT_BAD_SHAPE;
  const int rows = f32_chunk_rows(a.N_k, a.V, a.ws_bytes);
  if (rows < 1) return NAT_WORKSPACE_TOO_SMALL;
  float* term = (float*)a.ws;
  float* dz = (float*)((char*)a.ws + (((size_t)a.N_k * sizeof(float) + 255) / 256) * 256);
  hipStream_t s = a.stream;
  {
    ProfScope prof(PC_F32_PATH, s);
    for (int c0 = 0; c0 < a.N_k; c0 += rows) {
      const int n = a.N_k - c0 < rows ? a.N_k - c0 : rows;
      const float* hid = (const float*)a.hidden + (size_t)c0 * a.H;
      nat_status st = f32_gemm<false, false>(hid, a.H, (const float*)a.W, a.H, n, a.V, a.H, dz, a.V, 0, s);
      if (st != NAT_OK) return st;
      auto token = [&](auto kernel) {
        kernel<<<n, kF32Threads, 0, s>>>(a.ids, a.old_logp, a.adv, a.kept_seq, a.kept_w, c0, a.V, a.eps_lo, a.eps_hi, a.grad_scale,
                                         KlArgs{a.ref_logp, a.beta_kl, a.kl_kind}, dz, a.logp, term, a.kl_out, a.entropy_out, a.diag);
      };
      with_row_regs(a.V, [&](auto regs) { token(f32_token_kernel<decltype(regs)::value>); });
      NAT_LAUNCH_CHECK();
      st = f32_gemm<false, true>(dz, a.V, (const float*)a.W, a.H, n, a.H, a.V, (float*)a.dH + (size_t)c0 * a.H, a.H, 0, s);
      if (st != NAT_OK) return st;
      st = f32_gemm<true, true>(dz, a.V, hid, a.H, a.V, a.H, n, a.dW, a.H, (c0 > 0 || a.accumulate_dw) ? 1 : 0, s);
      if (st != NAT_OK) return st;
    }
  }
  ProfScope prof(PC_LOSS_REDUCE, s);
  loss_reduce_kernel<<<1, 1024, 0, s>>>(term, a.N_k, a.loss);
  NAT_LAUNCH_CHECK();
  return NAT_OK;
}


// Forward pass alone: log-prob of the target and entropy of one token per block.
template <int kRegs>
__global__ void __launch_bounds__(kF32Threads)
f32_logp_kernel(const float* __restrict__ z_scratch /*[chunk, V]*/, const int32_t* __restrict__ ids, int chunk_start, int V,
                float* __restrict__ logp_out, float* __restrict__ entropy_out, int32_t* __restrict__ diag) {
  __shared__ F32RowShared sh;
  const int kc = blockIdx.x, k = chunk_start + kc;
  const float* z = z_scratch + (size_t)kc * V;
  float row[kRegs + 1];
  const F32RowSums sums = f32_row_sums<kRegs>(z, V, sh, row);
  if (threadIdx.x == 0) {
    const int yk = ids[k];
    if (yk < 0 || yk >= V) {
      logp_out[k] = __builtin_nanf("");
      if (diag) atomicAdd(diag + NAT_DIAG_BAD_ID, 1);
    } else {
      logp_out[k] = (float)((double)z[yk] - ((double)sums.m + log(sums.s)));
    }
    if (entropy_out) entropy_out[k] = (float)(log(sums.s) - sums.t / sums.s);
  }
}

size_t logp_f32_workspace_bytes(int32_t N_k, int32_t H, int32_t V, bool minimal) {
  (void)H;
  int rows = N_k < 1 ? 1 : N_k;
  const int cap = minimal ? 1 : 4096;
  if (rows > cap) rows = cap;
  return 256 + (size_t)rows * V * sizeof(float);
}

nat_status logp_f32_run(const LogpArgs& a) {
  if (a.H > kF32MaxHidden) return NAT_BAD_SHAPE;
  if (a.ws_bytes < 256 + (size_t)a.V * sizeof(float)) return NAT_WORKSPACE_TOO_SMALL;
  size_t rows = (a.ws_bytes - 256) / ((size_t)a.V * sizeof(float));
  if (rows > (size_t)a.N_k) rows = a.N_k;
  hipStream_t s = a.stream;
  ProfScope prof(PC_F32_PATH, s);
  for (int c0 = 0; c0 < a.N_k; c0 += (int)rows) {
    const int n = a.N_k - c0 < (int)rows ? a.N_k - c0 : (int)rows;
    const nat_status st = f32_gemm<false, false>((const float*)a.hidden + (size_t)c0 * a.H, a.H, (const float*)a.W, a.H, n,
                                                 a.V, a.H, (float*)a.ws, a.V, 0, s);
    if (st != NAT_OK) return st;
    with_row_regs(a.V, [&](auto regs) {
      f32_logp_kernel<decltype(regs)::value><<<n, kF32Threads, 0, s>>>((const float*)a.ws, a.ids, c0, a.V, a.logp, a.entropy, a.diag);
    });
    NAT_LAUNCH_CHECK();
  }
  return NAT_OK;
}

}  // namespace nat
