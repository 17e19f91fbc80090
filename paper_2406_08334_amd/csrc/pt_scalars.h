// What the scalar kernel and an update that takes the scalar work along share: the constants of an update, and values that pass between
// workgroups of one launch.
#pragma once

#include "pt_common.h"

// Values other workgroups of the same launch have written (or will read): past this XCD's caches.
template <class T> __device__ __forceinline__ T ld_agent(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class T> __device__ __forceinline__ void st_agent(T* p, T x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Whether a sum of squares holds an infinity or a NaN (pt_close_sum).
__device__ __forceinline__ bool pt_not_finite(double x) { return (uint32_t(__double2hiint(x)) & 0x7ff00000u) == 0x7ff00000u; }

// The nine fp32 constants of this update from the fp64 hyper-parameters and the step's device scalars (Adam bias
// correction with t = applied updates + 1; clip coefficient min(1, c/(norm+1e-6)); unscale by the loss scale).
// Those that need no norm; bc1 = 1 - beta1^t, bc2 = 1 - beta2^t.
__device__ __forceinline__ void pt_step_consts(float (&c)[9], const pt_hparams& hp, double bc1, double bc2) {
  c[0] = float(hp.beta1);
  c[1] = float(hp.beta2);
  c[2] = float(1.0 - hp.beta1);
  c[3] = float(1.0 - hp.beta2);
  c[4] = float(1.0 - hp.lr * hp.weight_decay);
  c[5] = float(hp.lr / bc1);
  c[6] = float(1.0 / sqrt(bc2));
  c[7] = float(hp.eps);
}
// The gradient multiplier; clip: the clip coefficient.
__device__ __forceinline__ float pt_grad_mult(double& clip, double max_norm, double norm, double loss_scale) {
  clip = 1.0;
  if (max_norm > 0.0) {
    const double q = max_norm / (norm + 1e-6);
    clip = q < 1.0 ? q : 1.0;
  }
  return float(clip / loss_scale);
}
