// The step's scalars in device memory and what is done to them: loss-scale machine, step counter, the end of a step and its taking back;
// what the kernels that derive them are called with.
// Without a HIP compiler these are ordinary functions, so that the sequences of launches can be played through on the host.
#pragma once

#include <cstdint>

#include "ptchunk.h"

#ifdef __HIPCC__
#define PT_STEP_FN __device__ __forceinline__
#define PT_SCALAR __attribute__((address_space(4)))      // loaded through the scalar cache
#else
#define PT_STEP_FN inline
#define PT_SCALAR
#endif

// ---- device-resident scalars of a context ---------------------------------------
// One instance per context, in device memory.  Written only by the single-thread
// scalar kernels; read (uniformly) by the bulk kernels.
struct PtDevState {
  double sqnorm;
  double norm;
  double clip_coef;
  double loss_scale;
  double growth;
  double backoff;
  int32_t found_inf;
  int32_t step;          // applied updates so far
  int32_t good_steps;
  int32_t growth_interval;
  int32_t scaler_enabled;
  int32_t override_active;
  float override_grad_mult;
  // constants of the update in flight (see pt_update_consts)
  float c[9];
  int32_t skip;
  uint32_t ticket;       // workgroups of the scalar kernel that have finished (0 between launches)
  // a step that was ended together with its constants (pt_end_early): its number, and what the end has changed
  uint32_t ended;
  int32_t old_step, old_good_steps, old_override;
  double old_loss_scale;
};

// The end of a step - loss-scale machine and step counter (dynamic loss scaling with skip on non-finite gradients; the counter
// does not move on a skipped step) - from the step's found_inf; a forced multiplier lasts one step.
PT_STEP_FN void pt_advance(PtDevState& s, bool found_inf) {
  if (found_inf) {
    if (s.scaler_enabled) {
      const double b = s.loss_scale * s.backoff;
      s.loss_scale = b > 1.0 ? b : 1.0;
      s.good_steps = 0;
    }
  } else {
    s.step += 1;
    if (s.scaler_enabled) {
      s.good_steps += 1;
      if (s.good_steps >= s.growth_interval) {
        s.loss_scale = s.loss_scale * s.growth;
        s.good_steps = 0;
      }
    }
  }
  s.override_active = 0;
}

// The update reads nothing but the constants and `skip`, so the step can end here, without a launch of its own behind the update
// (4.8 us; pt_step_end then launches nothing; a step of 0.8 M parameters 22.3 -> 18.7 us, of 7 M 54.0 -> 52.5).  What changes is kept: a call
// of the same step that depends on it takes the end back first (pt_reopen_step).  Contexts with graphs, and those whose steps
// go on behind an update, end in the kernel (pt_prepare_consts).  s: the state this step began with.
PT_STEP_FN void pt_end_early(PtDevState* st, PtDevState s, bool found_inf, uint32_t step_no) {
  st->old_step = s.step; st->old_good_steps = s.good_steps; st->old_override = s.override_active; st->old_loss_scale = s.loss_scale;
  pt_advance(s, found_inf);
  st->step = s.step; st->good_steps = s.good_steps; st->override_active = s.override_active; st->loss_scale = s.loss_scale;
  st->ended = step_no;
}

// The end of a step, unless that has come with its constants: `early` is the number of the step that is known to have ended so, or
// 0.  (What `ended` still holds of a step closed without a launch is never asked for again.)
PT_STEP_FN void pt_end_step(PtDevState* st, uint32_t early) {
  if (early && st->ended == early) { st->ended = 0; return; }
  PtDevState s = *st;
  pt_advance(s, s.found_inf != 0);
  st->step = s.step; st->loss_scale = s.loss_scale; st->good_steps = s.good_steps; st->override_active = s.override_active;
}

// Takes the early end of that step back, unless that has happened or the step is closed.
PT_STEP_FN void pt_take_back(PtDevState* st, uint32_t early) {
  if (st->ended != early) return;
  st->step = st->old_step; st->loss_scale = st->old_loss_scale; st->good_steps = st->old_good_steps;
  st->override_active = st->old_override;
  st->ended = 0;
}

// ---- arguments of the scalar kernel ---------------------------------------------

struct pt_pack_plan;

// A per-chunk reduction of partial sums, to be launched or put off (see pt_norm.hip).  tile_begin == NULL: chunk first+i owns
// partials [i*per_chunk, (i+1)*per_chunk), else [tile_begin[c], tile_begin[c+1]) * per_tile.  seg_sum / seg_flag: room for n * segs
// sums where a chunk has more partials than one workgroup takes (segs > 1).
struct PtPendingReduce {
  const double* part = nullptr;
  const uint32_t* flag = nullptr;
  const uint32_t* tile_begin = nullptr;
  uint32_t first = 0, n = 0, per_chunk = 0, segs = 1;
  uint32_t per_tile = 1;                 // partial sums per entry of tile_begin
  double* seg_sum = nullptr;
  uint32_t* seg_flag = nullptr;
  const pt_pack_plan* plan = nullptr;    // owner of part / flag / tile_begin (NULL: the context)
};
struct PtScalarArgs {
  PtPendingReduce r;             // r.n == 0: nothing to reduce (grid 1 x 1)
  double* chunk_sq;
  uint32_t* chunk_flag;
  uint32_t C;
  uint32_t* ticket;
  PtDevState* st;                // NULL: the norm for a caller without a context, into out_*
  double* out_sq_norm;
  int32_t* out_found_inf;
  int do_finalize, do_prepare;
  uint32_t end_step;             // do_prepare: number of the step that ends with it, or 0
  pt_hparams hp;
  PtDevState* mirror;            // pinned host memory that receives the constants, or NULL
};

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

// What the kernel is called with.  The first workgroup alone reads `work`, from where the arguments lie (fused_work): as an ordinary argument it
// would be loaded by every wave.
struct FusedArgs {
  const PT_SCALAR uint64_t* table;
  uint32_t table_cols, no;
  uint64_t units;
  const PT_SCALAR uint32_t* nd_begin;
  const PT_SCALAR uint64_t* nd_ranges;
  const uint64_t* pub;
  int zero_grads;
  uint32_t summers;
  uint32_t tiles, total, doubled;                // of a chunk, of all chunks; workgroups that take two
  uint32_t inv_lo, inv_hi;                       // 2^58 / tiles, rounded up
  PtFused work;
};
