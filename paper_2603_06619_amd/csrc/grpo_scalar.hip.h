// Per-token scalar part of the loss (Eq. 1, Eq. 3) and the fixed-order loss
// reduction, shared by the bf16 and fp32 paths.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "nat.h"

namespace nat {

// KL term of Eq. 4 (sampled-token forms; the footnote to Eq. 4 names the first).
struct KlArgs {
  const float* ref_logp;   // [N_k] log-probability of the sampled token under the reference policy
  float beta;              // 0 disables the term (ref_logp is then not read)
  int kind;                // NAT_KL_LOG_RATIO or NAT_KL_NONNEG
};

struct TokenScalars { float L; float c; float kl; bool clipped; };   // clipped: A != 0 and dS/dlogp = 0

// r = exp(logp - old_logp); S = min(r A, clip(r, 1-eps_lo, 1+eps_hi) A);
// dS/dlogp = r A on the unclipped branch (boundaries inclusive), else 0;
// with d = ref_logp - logp:  KL = -d (log-ratio form) or exp(d) - d - 1 (non-negative form),
// dKL/dlogp = 1 or 1 - exp(d);
// token objective L = S - beta KL;  c = dLoss/dlogp = -grad_scale * w * (dS/dlogp - beta dKL/dlogp).
// T: precision of the log-prob and of everything formed from it (float on the bf16 path, double on the fp32 path).
// A behaviour log-prob equal to the log-prob as it is reported (rounded to fp32) gives r = 1 exactly in both.
__device__ __forceinline__ float exp_of(float x) { return expf(x); }
__device__ __forceinline__ double exp_of(double x) { return exp(x); }
__device__ __forceinline__ float min_of(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double min_of(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float max_of(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double max_of(double a, double b) { return fmax(a, b); }
// logp - other, 0 where they agree as fp32 numbers
__device__ __forceinline__ float logp_minus(float logp, float other) { return logp - other; }
__device__ __forceinline__ double logp_minus(double logp, float other) {
  const double d = logp - (double)other;
  return (float)logp == other && d - d == 0.0 ? 0.0 : d;
}
template <class T>
__device__ __forceinline__ TokenScalars grpo_token_scalars(T logp, float old_logp, float A, float w,
                                                           float eps_lo, float eps_hi, float grad_scale,
                                                           float beta_kl, int kl_kind, float ref_logp) {
  const T lo = (T)(1.f - eps_lo), hi = (T)(1.f + eps_hi);
  const T r = exp_of(logp_minus(logp, old_logp));
  const T r_clip = min_of(max_of(r, lo), hi);
  const T S = min_of(r * (T)A, r_clip * (T)A);
  const bool active = (A > 0.f && r <= hi) || (A < 0.f && r >= lo);
  T g = active ? r * (T)A : (T)0;
  TokenScalars out;
  out.clipped = A != 0.f && !active;
  T L = S;
  out.kl = 0.f;
  if (beta_kl != 0.f) {
    const T d = -logp_minus(logp, ref_logp);
    T kl, dkl;
    if (kl_kind == NAT_KL_NONNEG) {
      const T ed = exp_of(d);
      kl = ed - d - (T)1;
      dkl = (T)1 - ed;
    } else {
      kl = -d;
      dkl = (T)1;
    }
    out.kl = (float)kl;
    L = S - (T)beta_kl * kl;
    g -= (T)beta_kl * dkl;
  }
  out.L = (float)L;
  out.c = (float)(-(T)grad_scale * (T)w * g);
  return out;
}

// loss = -sum_k term[k], one block, fixed order: lane-strided fp64 partial sums,
// then a fixed binary tree over the 1024 partials.
static __global__ void __launch_bounds__(1024)
loss_reduce_kernel(const float* __restrict__ term, int n, float* __restrict__ loss) {
  __shared__ double part[1024];
  double s = 0.0;
  for (int k = threadIdx.x; k < n; k += 1024) s += (double)term[k];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int half = 512; half > 0; half >>= 1) {
    if ((int)threadIdx.x < half) part[threadIdx.x] += part[threadIdx.x + half];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = (float)(-part[0]);
}

}  // namespace nat
