// What the scalar kernel and an update that takes the scalar work along share: the constants of an update, values that pass between
// workgroups of one launch, and the arguments of such an update.
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

// ---- an update that derives its own constants (k_adamw_fused) --------------------------------------
//
// The sums it takes first, if a plan's wait: units of PT_REDUCE_SEG partial sums at most, [lo, hi) of unit u, chunk by chunk; chunk first + i
// has chunk_units[i] of them, possibly none.  `trees`: of 64 lanes, in the longest unit.
constexpr uint32_t FUSED_UNITS = 24, FUSED_TREES = 8, FUSED_CHUNKS = 8;
// What its workgroups publish: FUSED_COPIES copies of the words of the update (FUSED_LINE words apart), then the trees' sums.
constexpr uint32_t FUSED_COPIES = 16, FUSED_LINE = 32, FUSED_PUB_WORDS = FUSED_COPIES * FUSED_LINE + FUSED_UNITS * FUSED_TREES * 2;
struct PtFused {
  const double* part = nullptr;
  uint32_t lo[FUSED_UNITS] = {}, hi[FUSED_UNITS] = {};
  uint32_t units = 0, trees = 0, first = 0, n = 0;
  uint8_t chunk_units[FUSED_CHUNKS] = {};
  uint32_t C = 0;
  double* chunk_sq = nullptr;
  uint32_t* chunk_flag = nullptr;
  PtDevState* st = nullptr;
  uint64_t* pub = nullptr;
  uint32_t no = 0;                 // of this launch in its context, from 1 on
  uint32_t end_step = 0;           // number of the step that ends with it
  uint32_t tries = 0;              // looks for what another workgroup publishes, before a wave does the work itself
  pt_hparams hp{};
};
// Its workgroups that take sums: workgroup 1 + k the tree k % trees of the units 2 * (k / trees) and 2 * (k / trees) + 1.
inline uint32_t pt_fused_summers(const PtFused& f) { return (f.units + 1) / 2 * f.trees; }
