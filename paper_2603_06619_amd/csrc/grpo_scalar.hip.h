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
// All of it in fp64.  A behaviour log-prob equal to the log-prob as it is reported (rounded to fp32) gives r = 1 exactly.
// logp - other, 0 where they agree as fp32 numbers
__device__ __forceinline__ double logp_minus(double logp, float other) {
  const double d = logp - (double)other;
  return (float)logp == other && d - d == 0.0 ? 0.0 : d;
}
__device__ __forceinline__ TokenScalars grpo_token_scalars(double logp, float old_logp, float A, float w,
                                                           float eps_lo, float eps_hi, float grad_scale,
                                                           float beta_kl, int kl_kind, float ref_logp) {
  const double lo = (double)(1.f - eps_lo), hi = (double)(1.f + eps_hi);
  const double r = exp(logp_minus(logp, old_logp));
  const double r_clip = fmin(fmax(r, lo), hi);
  const double S = fmin(r * (double)A, r_clip * (double)A);
  const bool active = (A > 0.f && r <= hi) || (A < 0.f && r >= lo);
  double g = active ? r * (double)A : (double)0;
  TokenScalars out;
  out.clipped = A != 0.f && !active;
  double L = S;
  out.kl = 0.f;
  if (beta_kl != 0.f) {
    const double d = -logp_minus(logp, ref_logp);
    double kl, dkl;
    if (kl_kind == NAT_KL_NONNEG) {
      const double ed = exp(d);
      kl = ed - d - (double)1;
      dkl = (double)1 - ed;
    } else {
      kl = -d;
      dkl = (double)1;
    }
    out.kl = (float)kl;
    L = S - (double)beta_kl * kl;
    g -= (double)beta_kl * dkl;
  }
  out.L = (float)L;
  out.c = (float)(-(double)grad_scale * (double)w * g);
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
