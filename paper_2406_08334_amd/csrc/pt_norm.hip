// Global gradient norm: per-block fp64 partial sums of squares over gradient
// chunks, a fixed-order per-chunk reduction, and the finalize step.
//
// HBM-bound: 2 bytes read per element.  Each lane issues 16-byte loads that are
// contiguous across the wavefront (1 KiB per wave instruction), converts every
// 16-bit word to fp64 and accumulates squares in fp64 (two 16-bit significands
// multiply exactly, so only the additions round); the loss scale and the scan for
// non-finite words cost nothing per element (pt_close_sum).  Reduction order is fixed:
// lane-serial, then a 64-lane shuffle tree, then the four waves through LDS, then
// one slot per block - no floating-point atomics, so results are bitwise reproducible.
//
// Three shapes by the size of the call (norm_shape), all with the same order of additions.  Up to 1024 workgroups (four a
// compute unit, all of them running at once) a lane has all of its loads in flight: what such a call costs is how often it
// waits.  8.4e6 words 9.3 us with four loads, 8.8 with sixteen (from there on down the host's two launches were the limit; without a
// context it is one launch now, 6.9 us), 3.3e7
// 15.9 and 15.3; 1e8 34.8 and 41.7.  Large arenas are read fastest with few bytes in flight: two loads a lane, and unused LDS that
// leaves four workgroups on a compute unit instead of eight.  8.1e8 words 233 us (6.9 TB/s; 7.05 without the scalar kernel's 5 us),
// with four loads 239, one load 291, two loads and no limit 241, six workgroups 237, three 245; 2.5e8 77.0 / 78.5 / 96.3 / 79.2 / 77.9 /
// 81.4.  The line is where a second set of 1024 workgroups is three quarters full: below it eight at once are faster or
// it makes no difference (4.5e7 fp16 words 19.7 us either way, 6e7 23.7 with the limit and 25.3 without).  In between four loads
// are as good as two or better (6e7 23.65, 1e8 34.8 against 35.1).  fp32 chunks are twice the bytes for as many
// workgroups and gain from the limit from four full sets on: 6.7e7 words 50.8 us with it and two loads, 47.3 with four loads and
// without it, 1.3e8 88.6 and 86.7, 4e8 239 and 241.
#include "pt_common.h"
#include "pt_scalars.h"

#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <mutex>

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int NB_THREADS = PT_REDUCE_THREADS;
struct NormShape { int unroll; uint32_t lds; };        // 16-byte loads of a lane in flight, unused LDS of a workgroup
inline NormShape norm_shape(uint64_t elems, bool fp32) {
  if (elems <= 1024ull * PT_NORM_BLOCK_ELEMS) return {16, 0};
  return elems < (fp32 ? 4096ull : 1792ull) * PT_NORM_BLOCK_ELEMS ? NormShape{4, 0} : NormShape{2, 36000};
}
typedef void (*norm_kernel_t)(const uint64_t*, uint32_t, uint64_t, const PtDevState*, double*, uint32_t*);
struct OneTicket;
typedef void (*norm_arena_kernel_t)(const void*, uint64_t, double, double*, uint32_t*, OneTicket*, OneTicket*, double*, int32_t*);

template <int DT>
__device__ __forceinline__ double word_to_f64(uint32_t w16) {
  if (DT == PT_BF16) {
    return (double)__uint_as_float(w16 << 16);
  } else {
    __half_raw r; r.x = (unsigned short)w16;
    return (double)__half2float(__half(r));
  }
}

template <int DT>
__device__ __forceinline__ void accum_vec(const u32x4& q, double& a0, double& a1) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double x0 = word_to_f64<DT>(w[k] & 0xffffu), x1 = word_to_f64<DT>(w[k] >> 16);
    a0 = fma(x0, x0, a0);
    a1 = fma(x1, x1, a1);
  }
}

__device__ __forceinline__ void accum_vec_f32(const u32x4& q, double& a0, double& a1) {
#pragma unroll
  for (int k = 0; k < 4; k += 2) {
    const double x0 = (double)__uint_as_float(q[k]), x1 = (double)__uint_as_float(q[k + 1]);
    a0 = fma(x0, x0, a0);
    a1 = fma(x1, x1, a1);
  }
}

// One block's share of a chunk: the fp64 sum of (g/scale)^2 and the non-finite flag over elements
// [b*PT_NORM_BLOCK_ELEMS, min(S, (b+1)*PT_NORM_BLOCK_ELEMS)) of the chunk at `base`; valid in thread 0.  U 16-byte loads of a lane
// are in flight together; neither U nor the end of a chunk changes the order of the additions.
template <int DT, int U, bool F32 = false>
__device__ __forceinline__ void sqnorm_block(const PT_GLOBAL u32x4* base, uint64_t S, uint32_t b, double inv_scale,
                                             double& acc, uint32_t& flag) {
  constexpr uint32_t PER_VEC = F32 ? 4 : 8, BLOCK_VECS = PT_NORM_BLOCK_ELEMS / PER_VEC;
  static_assert(BLOCK_VECS % (U * NB_THREADS) == 0, "a whole block is a number of whole rounds");
  const uint64_t v0 = uint64_t(b) * BLOCK_VECS, left = S / PER_VEC - v0;
  base += v0;
  double a0 = 0.0, a1 = 0.0;
  auto take = [&](const u32x4& q) {
    if constexpr (F32) accum_vec_f32(q, a0, a1);
    else accum_vec<DT>(q, a0, a1);
  };
  if (left >= BLOCK_VECS) {
    for (uint32_t v = threadIdx.x; v < BLOCK_VECS; v += U * NB_THREADS) {
      u32x4 q[U];
#pragma unroll
      for (int r = 0; r < U; ++r) q[r] = __builtin_nontemporal_load(base + v + r * NB_THREADS);
#pragma unroll
      for (int r = 0; r < U; ++r) take(q[r]);
    }
  } else {                               // the end of a chunk: what lies beyond it counts as zeros
    for (uint32_t v = threadIdx.x; v < left; v += U * NB_THREADS) {
      u32x4 q[U];
#pragma unroll
      for (int r = 0; r < U; ++r) {
        q[r] = u32x4{0, 0, 0, 0};
        if (v + r * NB_THREADS < left) q[r] = __builtin_nontemporal_load(base + v + r * NB_THREADS);
      }
#pragma unroll
      for (int r = 0; r < U; ++r) take(q[r]);
    }
  }
  pt_close_sum(a0 + a1, inv_scale, acc, flag);
  pt_block_sum(acc, flag);
}

// grid = (norm_blocks, n_chunks).  Block (b, i) reduces its share of chunk first+i, whose base
// pointer comes from the context's pointer table.
template <int DT, int U>
__global__ void __launch_bounds__(NB_THREADS)
k_sqnorm(const uint64_t* __restrict__ grad_row, uint32_t first, uint64_t S,
         const PtDevState* __restrict__ st, double* __restrict__ part, uint32_t* __restrict__ flagout) {
  const uint32_t b = blockIdx.x, i = blockIdx.y;
  const PT_GLOBAL u32x4* base = (const PT_GLOBAL u32x4*)(grad_row[first + i]);   // global_* loads
  double acc;
  uint32_t flag;
  sqnorm_block<DT, U>(base, S, b, 1.0 / st->loss_scale, acc, flag);
  if (threadIdx.x == 0) {
    size_t slot = size_t(first + i) * gridDim.x + b;
    part[slot] = acc;
    flagout[slot] = flag;
  }
}

// The same reduction over fp32 gradient chunks (accumulated micro-batches): 4 bytes read per
// element, every value widened to fp64 before it is squared.
template <int U>
__global__ void __launch_bounds__(NB_THREADS)
k_sqnorm_f32(const uint64_t* __restrict__ grad_row, uint32_t first, uint64_t S,
             const PtDevState* __restrict__ st, double* __restrict__ part, uint32_t* __restrict__ flagout) {
  const uint32_t b = blockIdx.x, i = blockIdx.y;
  const PT_GLOBAL u32x4* base = (const PT_GLOBAL u32x4*)(grad_row[first + i]);
  double acc;
  uint32_t flag;
  sqnorm_block<0, U, true>(base, S, b, 1.0 / st->loss_scale, acc, flag);
  if (threadIdx.x == 0) {
    size_t slot = size_t(first + i) * gridDim.x + b;
    part[slot] = acc;
    flagout[slot] = flag;
  }
}

template <int DT> norm_kernel_t pick_norm(int u) { return u == 16 ? k_sqnorm<DT, 16> : u == 4 ? k_sqnorm<DT, 4> : k_sqnorm<DT, 2>; }
inline norm_kernel_t pick_norm_f32(int u) { return u == 16 ? k_sqnorm_f32<16> : u == 4 ? k_sqnorm_f32<4> : k_sqnorm_f32<2>; }

// ---- the scalar work of a step in one launch ---------------------------------------------------
//
// Grid (segs, n): workgroup (s, i) adds up partial sums [s * PT_REDUCE_SEG, (s + 1) * PT_REDUCE_SEG) of chunk first+i
// (lane-strided serial sums, then the fixed block tree); the workgroup that finishes last adds the segments of each chunk
// in order, then - do_finalize - the values of all chunks in chunk order, and publishes norm and found_inf, and - do_prepare -
// derives the nine fp32 constants of the update.  Every order is fixed: who comes last does not change a bit.
//
// Latency is all it costs, so the chain is kept short: a lane's eight loads are in flight together, two waves take the
// powers of beta while the others wait for the sums, the chunk values pass through LDS, nothing that was just computed is
// read back, and no cache is written back or invalidated: what workgroups hand each other goes past the caches
// (agent scope), and a workgroup counts itself in when its store has arrived.  Reduction,
// finalize and constants: 15 chunks, 1.2e8 elements: 8.8 us in two launches and 5.5 us of a gap behind an event before, 6.8 us
// in one launch now (a kernel that does nothing takes 4.7 there); 47 chunks, 1.56e9 elements: 14.0 -> 8.8 us; one block's two
// chunks 6.5 -> 4.4 us.  With fences for the whole L2 instead: 9.5, 17 and 7.6 us.
static_assert(PT_FUSED_ROW == PT_REDUCE_SEG / 8, "the same order of additions");
constexpr int SC_SUM = PT_REDUCE_SEG / 8, SC_THREADS = SC_SUM + 128;     // two more waves for the powers

// Leaves the constants of this update, and whether it is skipped, where the update reads them.
__device__ __forceinline__ void prepare_body(PtDevState* st, const pt_hparams& hp, double bc1, double bc2, double norm, double loss_scale,
                                             bool override_active, float override_grad_mult, int32_t found_inf, PtDevState* mirror) {
  float c[9];
  double clip = 1.0;
  pt_step_consts(c, hp, bc1, bc2);
  c[8] = override_active ? override_grad_mult : pt_grad_mult(clip, hp.max_norm, norm, loss_scale);
  st->clip_coef = clip;
  const int32_t skip = found_inf ? 1 : 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) st->c[k] = c[k];
  st->skip = skip;
  // The host-side update reads its constants there after waiting for the event behind this kernel - no stream, no copy,
  // nothing that could queue up behind the resident update.
  if (mirror) {
#pragma unroll
    for (int k = 0; k < 9; ++k) mirror->c[k] = c[k];
    mirror->skip = skip;
    __threadfence_system();
  }
}

// Partial sums of chunk first + i.
__device__ __forceinline__ uint32_t partials_of(const PtPendingReduce& r, uint32_t i, uint32_t& lo) {
  if (!r.tile_begin) { lo = i * r.per_chunk; return r.per_chunk; }
  lo = r.tile_begin[r.first + i] * r.per_tile;
  return r.tile_begin[r.first + i + 1] * r.per_tile - lo;
}

__global__ void __launch_bounds__(SC_THREADS) k_scalars(const PtScalarArgs a) {
  __shared__ double s_sum[SC_SUM / 64], s_val[SC_SUM], s_bc[2];
  __shared__ uint32_t s_flag[SC_SUM / 64], s_f[SC_SUM], s_last;
  const PtPendingReduce& r = a.r;
  const uint32_t tid = threadIdx.x, c = r.first + blockIdx.y;
  const bool alone = r.segs == 1 && !a.do_finalize && !a.do_prepare;      // a chunk's sum each, and nothing behind it
  uint32_t lo = 0, hi = 0;
  if (r.n) hi = partials_of(r, blockIdx.y, lo);          // a number here
  hi = min(hi, (blockIdx.x + 1) * PT_REDUCE_SEG) + lo;
  lo = min(hi, lo + blockIdx.x * PT_REDUCE_SEG);
  double acc = 0.0;
  uint32_t f = 0;
  PtDevState s;                                          // what the last lines need of it, on its way while the sums are taken
  if (a.do_prepare) s = *a.st;
  if (tid < SC_SUM) {
    double x[8];
    uint32_t y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t k = lo + tid + j * SC_SUM;
      x[j] = k < hi ? r.part[k] : 0.0;
      y[j] = k < hi ? r.flag[k] : 0u;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) { acc += x[j]; f |= y[j]; }
    pt_wave_sum(acc, f);
    if ((tid & 63) == 0) { s_sum[tid >> 6] = acc; s_flag[tid >> 6] = f; }
  } else if (a.do_prepare && (tid & 63) == 0) {
    const double t = double(s.step + 1);
    s_bc[(tid - SC_SUM) >> 6] = 1.0 - pow(tid == SC_SUM ? a.hp.beta1 : a.hp.beta2, t);
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int i = 1; i < SC_SUM / 64; ++i) { acc += s_sum[i]; f |= s_flag[i]; }
    if (lo < hi) {
      const size_t slot = size_t(blockIdx.y) * r.segs + blockIdx.x;
      st_agent(r.segs > 1 ? r.seg_sum + slot : a.chunk_sq + c, acc);
      st_agent(r.segs > 1 ? r.seg_flag + slot : a.chunk_flag + c, f);
    }
    const uint32_t total = alone ? 1u : gridDim.x * gridDim.y;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    s_last = total == 1 || __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == total - 1 ? 1u : 0u;
  }
  __syncthreads();
  if (!s_last || alone) return;
  if (tid == 0) st_agent(a.ticket, 0u);
  double sq = 0.0, norm = 0.0;
  uint32_t inf = 0;
  // the chunks of this launch, or - to finalize - all of them
  const uint32_t c0 = a.do_finalize ? 0 : r.first, c1 = a.do_finalize ? a.C : r.first + r.n;
  for (uint32_t base = c0; base < c1; base += SC_SUM) {
    const uint32_t cc = base + tid;
    if (tid < SC_SUM && cc < c1) {
      double t;
      uint32_t g, p0;
      const uint32_t ns = r.segs > 1 && cc >= r.first && cc - r.first < r.n
                              ? (partials_of(r, cc - r.first, p0) + PT_REDUCE_SEG - 1) / PT_REDUCE_SEG : 0;
      if (ns) {
        t = 0.0; g = 0;
        for (uint32_t k = 0; k < ns; ++k) {
          t += ld_agent(r.seg_sum + size_t(cc - r.first) * r.segs + k);
          g |= ld_agent(r.seg_flag + size_t(cc - r.first) * r.segs + k);
        }
        a.chunk_sq[cc] = t;
        a.chunk_flag[cc] = g;
      } else {
        t = ld_agent(a.chunk_sq + cc);
        g = ld_agent(a.chunk_flag + cc);
      }
      s_val[tid] = t;
      s_f[tid] = g;
    }
    if (!a.do_finalize) continue;
    __syncthreads();
    if (tid == 0) {
      const uint32_t k1 = min(uint32_t(SC_SUM), c1 - base);
      for (uint32_t k = 0; k < k1; ++k) { sq += s_val[k]; inf |= s_f[k]; }
    }
    __syncthreads();
  }
  if (tid != 0) return;
  if (a.do_finalize) {
    norm = sqrt(sq);
    if (a.st) {
      a.st->sqnorm = sq;
      a.st->norm = norm;
      a.st->found_inf = inf ? 1 : 0;
      a.st->override_active = s.override_active = 0;
    } else {
      a.out_sq_norm[0] = sq;
      a.out_sq_norm[1] = norm;
      *a.out_found_inf = inf ? 1 : 0;
    }
  }
  if (a.do_prepare) {
    if (!a.do_finalize) { norm = s.norm; inf = uint32_t(s.found_inf); }
    prepare_body(a.st, a.hp, s_bc[0], s_bc[1], norm, s.loss_scale, s.override_active != 0, s.override_grad_mult, int32_t(inf), a.mirror);
    if (a.end_step) pt_end_early(a.st, s, inf != 0, a.end_step);
  }
}

// The constants of a prepared step into pinned host memory, for a host-side update that nothing pointed to.
__global__ void k_mirror(const PtDevState* st, PtDevState* mirror) {
  if (threadIdx.x < 9) mirror->c[threadIdx.x] = st->c[threadIdx.x];
  if (threadIdx.x == 9) mirror->skip = st->skip;
  __threadfence_system();
}

}  // namespace

// ---- scalar work of a step: put off and fused -----------------------------------------------
//
// The finalize is put off to the first call that needs its result - normally the update, which then derives its constants in
// the same launch - and the reduction of a small plan's partial sums (PT_FUSE_MAX_*) with it: for a small state launches are
// what a step costs.  What waits runs on the stream of the call that needs it, which is ordered behind the packs anyway.
// Every other reduction belongs to its own call.  A program that packs eagerly and replays a graph of norm, update and step
// end makes no call that could launch it, and the plan may be gone by then.  It costs a launch of 4 us: put off and at once,
// 33 chunks of 95 528 elements 39 and 43 us, 14 of 5e6 354 and 357-360, 15 of 2^23 616 and 619, 47 of 2^25 7.76 ms both.

constexpr uint32_t PT_FUSE_MAX_CHUNKS = 8;
constexpr uint32_t PT_FUSE_MAX_PARTIALS = 16384;
// Where an update takes all of this along in its own launch (k_adamw_fused).  One wave adds the chunks up one after the other, which takes longer
// than a launch if there are many: chunks of 2^18, k_scalars in front and not, 128 of them 169.1 and 166.0 us a step, 160 211.4 and 208.7, 208
// 268.8 and 266.6, 224 295.5 and 296.1, 256 331.5 and 334.1.  (Chunks of 256 elements, where nothing hides it: call behind call, which the host
// decides, 192 63.7 and 60.6, a step alone 128 56.4 and 57.8, 192 72.4 and 77.7.)  There is no lower line: one chunk of 768 elements 13.5 and 9.5,
// of 12 700 13.6 and 9.6, eight of 512 15.1 and 11.4, nine of 4096 18.6 and 15.3, 64 of 256 30.3 and 27.6.
constexpr uint32_t PT_FUSED_MAX_CHUNKS = 208;

static int launch_scalars(pt_ctx* ctx, const PtPendingReduce* r, bool finalize, const pt_hparams* hp, uint32_t end_step, PtDevState* mirror,
                          hipStream_t stream) {
  PtScalarArgs a{};
  if (r) a.r = *r;
  a.chunk_sq = ctx->d_chunk_sq; a.chunk_flag = ctx->d_chunk_flag; a.C = ctx->C; a.ticket = &ctx->d_state->ticket; a.st = ctx->d_state;
  a.do_finalize = finalize ? 1 : 0;
  a.do_prepare = hp ? 1 : 0;
  if (hp) a.hp = *hp;
  a.end_step = end_step;
  a.mirror = mirror;
  hipLaunchKernelGGL(k_scalars, dim3(a.r.segs, r ? std::max(1u, r->n) : 1u), dim3(SC_THREADS), 0, stream, a);
  PT_LAUNCH_CHECK(ctx, "k_scalars");
  return PT_OK;
}

// Everything put off, the constants of `hp` behind it if there are any, in one launch.
static int launch_pending(pt_ctx* ctx, const pt_hparams* hp, uint32_t end_step, PtDevState* mirror, hipStream_t stream) {
  const int rc = launch_scalars(ctx, ctx->pend_reduce.n ? &ctx->pend_reduce : nullptr, ctx->pend_finalize, hp, end_step, mirror, stream);
  if (rc != PT_OK) return rc;
  ctx->pend_reduce = PtPendingReduce{};
  ctx->pend_finalize = false;
  return PT_OK;
}

int pt_flush_pending(pt_ctx* ctx, hipStream_t stream) {
  if (!ctx->pend_reduce.n && !ctx->pend_finalize) return PT_OK;
  // one that was asked for under capture, in a step that had ended early: the end follows its found_inf
  if (ctx->pend_finalize)
    if (const int rc = pt_reopen_step(ctx, stream); rc != PT_OK) return rc;
  return launch_pending(ctx, nullptr, 0, nullptr, stream);
}

// A call is about to write partial sums: a finalize that is still waiting takes the old ones first.
int pt_before_partials(pt_ctx* ctx, hipStream_t stream) { return ctx->pend_finalize ? pt_flush_pending(ctx, stream) : int(PT_OK); }

int pt_reduce_plan(pt_ctx* ctx, const pt_pack_plan* plan, hipStream_t stream) {
  if (plan->touched.empty()) return PT_OK;
  PtPendingReduce r;
  r.part = plan->d_tile_sq; r.flag = plan->d_tile_flag; r.tile_begin = plan->d_chunk_tile_begin;
  r.first = plan->touched.front(); r.n = plan->touched.back() - r.first + 1; r.per_tile = plan->subs;
  r.segs = plan->segs; r.seg_sum = plan->d_seg_sum; r.seg_flag = plan->d_seg_flag;
  r.plan = plan;
  const bool small = plan->touched.size() <= PT_FUSE_MAX_CHUNKS && ctx->C <= 64 && plan->n_tiles <= PT_FUSE_MAX_PARTIALS;
  // the same partial sums again: taken once, with the values they will then hold
  if (small && ctx->pend_reduce.n && ctx->pend_reduce.plan == plan) return PT_OK;
  // whatever is pending comes first: a later reduction of the same chunk replaces an earlier one
  const int rc = pt_flush_pending(ctx, stream);
  if (rc != PT_OK || !small) return rc != PT_OK ? rc : launch_scalars(ctx, &r, false, nullptr, 0, nullptr, stream);
  ctx->pend_reduce = r;
  return PT_OK;
}

int pt_prepare_consts(pt_ctx* ctx, const pt_hparams* hp, bool host_part, hipStream_t stream) {
  if (ctx->prepared) {
    if (std::memcmp(&ctx->prepared_hp, hp, sizeof *hp) == 0) return PT_OK;
    if (ctx->stream_pending)
      return pt_fail(ctx, PT_ERR_STATE, "hyper-parameters changed while a streamed update of this step is in flight");
  }
  // The event that lets a host-side update read the constants early costs the update behind it 5 us: recorded only where such
  // a call can be on its way, or has been made before.
  const bool mirror = host_part || ctx->host_pool != nullptr;
  ctx->mirrored = false;
  int rc = pt_reopen_step(ctx, stream);              // other hyper-parameters: the constants are derived anew
  if (rc != PT_OK) return rc;
  // The launch is the step's end too (pt_end_early), but not in a graph, whose replays may be followed by a step end outside it, nor
  // in a context that has graphs, nor where a step of the context has gone on behind it.
  const bool end = !ctx->captured && !ctx->goes_on;
  rc = launch_pending(ctx, hp, end ? ctx->step_no : 0, mirror ? ctx->h_state_dev : nullptr, stream);
  if (rc != PT_OK) return rc;
  if (end) ctx->ended_early = ctx->step_no;
  if (mirror) {
    PT_HIP(ctx, hipEventRecord(ctx->ev_scalar, stream));
    ctx->mirrored = true;
  }
  ctx->prepared = true;
  ctx->prepared_hp = *hp;
  return PT_OK;
}

// The update takes the scalar work along where it covers all chunks, a finalize waits, nothing but the update depends on the constants
// (no host-side update: its event would be behind the whole update), and the step can end with them (pt_prepare_consts).
bool pt_fuse_scalars(pt_ctx* ctx, const pt_hparams* hp, PtFused* f) {
  if (ctx->pub_no == UINT32_MAX) return false;         // the numbers of launches don't come round again
  if (ctx->prepared || !ctx->pend_finalize || ctx->host_pool || ctx->captured || ctx->goes_on || ctx->ended_early) return false;
  if (ctx->opt_adamw_grid || ctx->opt_adamw_unroll || ctx->opt_adamw_threads || !pt_adamw_hints(ctx)) return false;
  if (ctx->C > PT_FUSED_MAX_CHUNKS) return false;
  const PtPendingReduce& r = ctx->pend_reduce;
  if (r.n > FUSED_CHUNKS || (r.n && ctx->C > 64)) return false;
  if (r.n) {
    uint32_t most = 0;
    for (uint32_t i = 0; i < r.n; ++i) {
      uint32_t lo = r.plan->tile_begin[i] * r.per_tile;
      const uint32_t hi = r.plan->tile_begin[i + 1] * r.per_tile;
      for (; lo < hi; lo += PT_REDUCE_SEG) {
        if (f->units == FUSED_UNITS) return false;
        f->lo[f->units] = lo;
        f->hi[f->units] = std::min(hi, lo + PT_REDUCE_SEG);
        most = std::max(most, f->hi[f->units] - lo);
        ++f->units;
        ++f->chunk_units[i];
      }
    }
    f->trees = (std::min(most, PT_FUSED_ROW) + 63) / 64;
    if (ctx->S / 256 * ctx->C <= 2 * pt_fused_summers(*f)) return false;       // they are among the workgroups of the update
    f->part = r.part; f->first = r.first; f->n = r.n;
  }
  f->C = ctx->C; f->chunk_sq = ctx->d_chunk_sq; f->chunk_flag = ctx->d_chunk_flag; f->st = ctx->d_state; f->pub = ctx->d_pub;
  f->no = ++ctx->pub_no;                              // also if the launch fails: no two have the same
  f->end_step = ctx->step_no;
  f->tries = ctx->opt_fused_tries;
  f->hp = *hp;
  return true;
}

void pt_fused_launched(pt_ctx* ctx, const PtFused& f) {
  ctx->pend_reduce = PtPendingReduce{};
  ctx->pend_finalize = false;
  ctx->mirrored = false;
  ctx->ended_early = ctx->step_no;
  ctx->prepared = true;
  ctx->prepared_hp = f.hp;
}

int pt_mirror_consts(pt_ctx* ctx, hipStream_t stream) {
  if (ctx->mirrored) return PT_OK;
  hipLaunchKernelGGL(k_mirror, dim3(1), dim3(64), 0, stream, ctx->d_state, ctx->h_state_dev);
  PT_LAUNCH_CHECK(ctx, "k_mirror");
  PT_HIP(ctx, hipEventRecord(ctx->ev_scalar, stream));
  ctx->mirrored = true;
  return PT_OK;
}

extern "C" int pt_chunk_grad_sqnorm(pt_ctx* ctx, const void* const* grad_chunks, uint32_t first_chunk,
                                    uint32_t n_chunks, int finalize, void* stream) {
  if (!ctx) return PT_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (uint64_t(first_chunk) + n_chunks > ctx->C)
    return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_grad_sqnorm: chunks [%u, %u) outside the context's %u chunks",
                   first_chunk, first_chunk + n_chunks, ctx->C);
  if (finalize < 0 || finalize > PT_FINALIZE_CARRY)
    return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_grad_sqnorm: finalize must be 0, PT_FINALIZE_STRICT or PT_FINALIZE_CARRY");
  PtPendingReduce r;                             // of a recompute
  if (grad_chunks && n_chunks) {
    pt_capturing(ctx, st);                       // without chunks the call launches nothing
    int rc = pt_table_bind(ctx, ROW_PACK, first_chunk, n_chunks, grad_chunks + first_chunk, false, st);
    if (rc != PT_OK || (rc = pt_reopen_step(ctx, st)) != PT_OK || (rc = pt_before_partials(ctx, st)) != PT_OK) return rc;
    const NormShape shape = norm_shape(ctx->S * n_chunks, ctx->grad_f32);
    norm_kernel_t kern = ctx->grad_f32          ? pick_norm_f32(shape.unroll)
                         : ctx->dtype == PT_BF16 ? pick_norm<PT_BF16>(shape.unroll)
                                                 : pick_norm<PT_FP16>(shape.unroll);
    hipLaunchKernelGGL(kern, dim3(ctx->norm_blocks, n_chunks), dim3(NB_THREADS), shape.lds, st, pt_row(ctx, ROW_PACK), first_chunk,
                       ctx->S, ctx->d_state, ctx->d_norm_part, ctx->d_norm_flag);
    PT_LAUNCH_CHECK(ctx, "k_sqnorm");
    r.part = ctx->d_norm_part + size_t(first_chunk) * ctx->norm_blocks;
    r.flag = ctx->d_norm_flag + size_t(first_chunk) * ctx->norm_blocks;
    r.first = first_chunk; r.n = n_chunks; r.per_chunk = ctx->norm_blocks; r.segs = ctx->norm_segs;
    if (r.segs > 1) {
      r.seg_sum = ctx->d_norm_seg_sum + size_t(first_chunk) * r.segs;
      r.seg_flag = ctx->d_norm_seg_flag + size_t(first_chunk) * r.segs;
    }
    if ((rc = pt_flush_pending(ctx, st)) != PT_OK) return rc;      // a waiting sum of the same chunk is replaced
    // a recompute covers the whole chunk: whatever plan packed it, its value is complete now
    for (uint32_t c = first_chunk; c < first_chunk + n_chunks; ++c) { ctx->chunk_fresh[c] = 1; ctx->chunk_packed_by[c] = 0; }
  }
  int refused = PT_OK;
  if (finalize && ctx->stream_pending)
    refused = pt_fail(ctx, PT_ERR_STATE, "pt_chunk_grad_sqnorm: a streamed update is still open (its kernels read the "
                      "step's scalars); close the step with pt_step_end first");
  else if (finalize && finalize != PT_FINALIZE_CARRY) {
    for (uint32_t c = 0; c < ctx->C && refused == PT_OK; ++c)
      if (!ctx->chunk_fresh[c])
        refused = pt_fail(ctx, PT_ERR_STATE, "pt_chunk_grad_sqnorm: chunk %u has no sum of squares from this step (nothing "
                          "packed, accumulated or recomputed for it since the last pt_step_end); its old value would enter "
                          "the norm - finalize with PT_FINALIZE_CARRY if that is meant", c);
  }
  const bool final = finalize && refused == PT_OK;
  // a recompute's own launch takes the sum over the chunks along (recompute, norm and step end of 4e6 words 13.9 -> 12.6 us,
  // of 6.7e7 28.9 -> 27.7)
  if (r.n)
    if (const int rc = launch_scalars(ctx, &r, final, nullptr, 0, nullptr, st); rc != PT_OK) {
      std::fill_n(ctx->chunk_fresh.begin() + first_chunk, n_chunks, uint8_t(0));
      return rc;
    }
  if (final) {
    if (const int rc = pt_reopen_step(ctx, st); rc != PT_OK) return rc;
    // Else it runs with the first call that needs it: the update (in the launch that derives its constants), a read-back, or
    // pt_step_end.
    ctx->pend_finalize = !r.n;
    ctx->norm_finalized = true;
    ctx->prepared = false;
  }
  return refused;
}

// ---- the norm for callers that cannot allocate -------------------------------------------------
// Same kernels and the same reduction order as pt_chunk_grad_sqnorm(grad_chunks, ..., finalize), but
// without a context: the block partials and per-chunk sums live in one file-scope device array
// instead of memory a context allocated, and the gradient chunks are addressed as one arena.

namespace {

constexpr uint32_t PT_STATIC_MAX_PARTIALS = 1u << 19;   // blocks of PT_NORM_BLOCK_ELEMS elements: 2^34 elements
constexpr uint32_t PT_STATIC_MAX_CHUNKS = 4096;
constexpr int PT_STATIC_MAX_DEVICES = 64;

constexpr uint32_t PT_ONE_MAX_BLOCKS = 1024, PT_ONE_MAX_WAVES = 16, PT_ONE_TICKETS = 16, ONE_COUNTERS = 16;
// Workgroups count themselves in on 16 counters, a line of memory each, and the last of each on one more: 256 of them on a single
// one waited for each other for 2 us.
struct OneTicket { struct alignas(128) Line { uint32_t n; } line[ONE_COUNTERS + 1]; };

// workgroups of the reduction: n * ceil(per_chunk / PT_REDUCE_SEG) <= n + partials / PT_REDUCE_SEG
constexpr uint32_t PT_STATIC_MAX_SEGS = PT_STATIC_MAX_CHUNKS + PT_STATIC_MAX_PARTIALS / PT_REDUCE_SEG;

struct PtStaticScratch {
  double part[PT_STATIC_MAX_PARTIALS];
  double chunk_sq[PT_STATIC_MAX_CHUNKS];
  double seg_sum[PT_STATIC_MAX_SEGS];
  uint32_t flag[PT_STATIC_MAX_PARTIALS];
  uint32_t chunk_flag[PT_STATIC_MAX_CHUNKS];
  uint32_t seg_flag[PT_STATIC_MAX_SEGS];
  OneTicket ticket;
  // Of calls in one launch: a counter each, in turn, which its last workgroup leaves at 0.  A call also clears the one half way
  // round, so that what calls that overlapped in time have left in one does not stay.
  OneTicket tickets[PT_ONE_TICKETS];
};

}  // namespace

// 6.1 MiB per GPU the library runs on, held until the process ends.  In host code this name is only a
// stand-in for the symbol: the device address comes from hipGetSymbolAddress (scratch_of_current_device).
static __device__ __align__(256) unsigned char scratch[sizeof(PtStaticScratch)];

namespace {

// As k_sqnorm, for chunks that lie back to back in one arena; the loss scale comes by value.
//
// ONE: the workgroup that finishes last adds the partial sums up, in the order k_scalars has, and writes the results: one launch
// instead of two, which is what a call costs the host (8.8 -> 5.3 us).  No workgroup waits for another one.  Two launches and one:
// 2.6e5 words 8.8 -> 5.3 us, 4.2e6 8.8 -> 6.1, 8.4e6 8.8 -> 7.0 (with one counter 9.1), 1.7e7 10.2 -> 9.4 (13.5), 200 chunks of two
// workgroups 13.0 -> 8.8.
template <int DT, int U, bool ONE>
__global__ void __launch_bounds__(NB_THREADS)
k_sqnorm_arena(const void* __restrict__ arena, uint64_t S, double loss_scale, double* __restrict__ part, uint32_t* __restrict__ flagout,
               OneTicket* __restrict__ ticket, OneTicket* __restrict__ other_ticket, double* __restrict__ out_sq_norm,
               int32_t* __restrict__ out_found_inf) {
  const uint32_t b = blockIdx.x, i = blockIdx.y;
  const PT_GLOBAL u32x4* base = (const PT_GLOBAL u32x4*)((uint64_t)(uintptr_t)arena + 2ull * S * i);
  double acc;
  uint32_t flag;
  sqnorm_block<DT, U>(base, S, b, 1.0 / loss_scale, acc, flag);
  const size_t slot = size_t(i) * gridDim.x + b;
  if constexpr (!ONE) {
    if (threadIdx.x == 0) {
      if (b == 0 && i == 0) ticket->line[0].n = 0;       // whatever calls that overlapped in time have left there
      part[slot] = acc;
      flagout[slot] = flag;
    }
  } else {
    __shared__ double s_tree[PT_ONE_MAX_BLOCKS];
    __shared__ uint32_t s_last;
    const uint32_t total = gridDim.x * gridDim.y;
    if (threadIdx.x == 0) {
      if (slot == 0) for (uint32_t k = 0; k <= ONE_COUNTERS; ++k) st_agent(&other_ticket->line[k].n, 0u);
      st_agent(part + slot, acc);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const uint32_t k = uint32_t(slot) % ONE_COUNTERS, mine = (total - k + ONE_COUNTERS - 1) / ONE_COUNTERS;
      uint32_t last = __hip_atomic_fetch_add(&ticket->line[k].n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mine - 1;
      if (last) last = __hip_atomic_fetch_add(&ticket->line[ONE_COUNTERS].n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                       == min(total, ONE_COUNTERS) - 1;
      s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x <= ONE_COUNTERS) st_agent(&ticket->line[threadIdx.x].n, 0u);
    // As many lanes as a chunk has partial sums; `w` of them, a power of two, add theirs up in a tree, one lane the trees of a chunk
    // one after the other.
    const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6, per = gridDim.x, n = gridDim.y;
    uint32_t lg = 0;
    while (lg < 6 && (1u << lg) < per) ++lg;
    const uint32_t w = 1u << lg, trees = (per + w - 1) / w, all = n * trees;
    constexpr uint32_t WAVES = NB_THREADS / 64, R = PT_ONE_MAX_WAVES / WAVES;
    double x[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      const uint32_t v = ((wid + r * WAVES) << (6 - lg)) + (lane >> lg), c = v / trees, k = (v - c * trees) * w + (lane & (w - 1));
      x[r] = v < all && k < per ? ld_agent(part + size_t(c) * per + k) : 0.0;
    }
    for (uint32_t off = w >> 1; off > 0; off >>= 1)
#pragma unroll
      for (uint32_t r = 0; r < R; ++r) x[r] += __shfl_down(x[r], off, 64);
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      const uint32_t v = ((wid + r * WAVES) << (6 - lg)) + (lane >> lg);
      if ((lane & (w - 1)) == 0 && v < all) s_tree[v] = x[r];
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double sq = 0.0;
    if (trees == 1) {
#pragma unroll 8
      for (uint32_t c = 0; c < n; ++c) sq += s_tree[c];
    } else {
      for (uint32_t c = 0; c < n; ++c) {
        double t = s_tree[c * trees];
        for (uint32_t k = 1; k < trees; ++k) t += s_tree[c * trees + k];
        sq += t;
      }
    }
    out_sq_norm[0] = sq;
    out_sq_norm[1] = sqrt(sq);
    // a sum of squares is finite if and only if every number is (pt_close_sum)
    *out_found_inf = pt_not_finite(sq) ? 1 : 0;
  }
}

// Waves that take the partial sums of n chunks with `per` each in one launch.
inline uint64_t one_waves(uint64_t per, uint64_t n) {
  uint64_t w = 1;
  while (w < 64 && w < per) w *= 2;
  return (n * ((per + w - 1) / w) * w + 63) / 64;
}
// One launch where all workgroups run at once (norm_shape), the last one's four waves have at most four loads a lane (eight cost 0.7 us,
// more than the rest of what a larger call gains: 960 workgroups 16.8 -> 16.1) and no lane has two partial sums of a chunk (one
// chunk of 1024: 15.0 -> 15.5).
inline bool norm_in_one(uint64_t per_chunk, uint64_t n_chunks) {
  return per_chunk <= SC_SUM && per_chunk * n_chunks <= PT_ONE_MAX_BLOCKS && one_waves(per_chunk, n_chunks) <= PT_ONE_MAX_WAVES;
}

template <int DT> norm_arena_kernel_t pick_norm_arena(int u, bool one) {
  return one ? k_sqnorm_arena<DT, 16, true>
         : u == 16 ? k_sqnorm_arena<DT, 16, false> : u == 4 ? k_sqnorm_arena<DT, 4, false> : k_sqnorm_arena<DT, 2, false>;
}

std::mutex g_scratch_mutex;
void* g_scratch_addr[PT_STATIC_MAX_DEVICES] = {};

}  // namespace

// Device address of `scratch` on the current device, looked up once per device (every GPU holds its
// own copy of the array at its own address).
int pt_static_scratch_setup(void** out, int* device) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return pt_fail(nullptr, PT_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= PT_STATIC_MAX_DEVICES)
    return pt_fail(nullptr, PT_ERR_UNSUPPORTED, "device %d: at most %d devices are supported", dev, PT_STATIC_MAX_DEVICES);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return pt_fail(nullptr, PT_ERR_HIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_addr[dev] = p;
  }
  if (out) *out = g_scratch_addr[dev];
  if (device) *device = dev;
  return PT_OK;
}

extern "C" int pt_chunk_grad_sqnorm_noalloc(const void* grad_arena, int dtype, uint64_t chunk_elems, uint32_t n_chunks,
                                            double loss_scale, double* out_sqnorm_norm, int32_t* out_found_inf,
                                            void* stream) {
  if (!grad_arena || !out_sqnorm_norm || !out_found_inf)
    return pt_fail(nullptr, PT_ERR_INVALID_ARG, "pt_chunk_grad_sqnorm_noalloc: NULL pointer");
  if (dtype != PT_BF16 && dtype != PT_FP16)
    return pt_fail(nullptr, PT_ERR_INVALID_ARG, "pt_chunk_grad_sqnorm_noalloc: dtype %d is neither PT_BF16 nor PT_FP16", dtype);
  if (chunk_elems == 0 || n_chunks == 0)
    return pt_fail(nullptr, PT_ERR_INVALID_ARG, "pt_chunk_grad_sqnorm_noalloc: chunk_elems and n_chunks must be > 0");
  if (chunk_elems % 8 != 0 || (reinterpret_cast<uintptr_t>(grad_arena) & 15u))
    return pt_fail(nullptr, PT_ERR_ALIGNMENT,
                   "pt_chunk_grad_sqnorm_noalloc: chunk_elems must be a multiple of 8 and the arena 16-byte aligned");
  if ((reinterpret_cast<uintptr_t>(out_sqnorm_norm) & 7u) || (reinterpret_cast<uintptr_t>(out_found_inf) & 3u))
    return pt_fail(nullptr, PT_ERR_ALIGNMENT, "pt_chunk_grad_sqnorm_noalloc: misaligned output pointer");
  if (!(loss_scale >= 1.0) || !(loss_scale <= 1.8446744073709552e19))
    return pt_fail(nullptr, PT_ERR_INVALID_ARG, "pt_chunk_grad_sqnorm_noalloc: loss_scale must be in [1, 2^64]");
  const uint64_t blocks_per_chunk = (chunk_elems + PT_NORM_BLOCK_ELEMS - 1) / PT_NORM_BLOCK_ELEMS;
  if (n_chunks > PT_STATIC_MAX_CHUNKS || blocks_per_chunk * n_chunks > PT_STATIC_MAX_PARTIALS)
    return pt_fail(nullptr, PT_ERR_UNSUPPORTED,
                   "pt_chunk_grad_sqnorm_noalloc: %u chunks of %llu elements exceed the static scratch (at most %u chunks "
                   "and %u blocks of %u elements, i.e. 2^34 elements); use pt_chunk_grad_sqnorm with a context",
                   n_chunks, (unsigned long long)chunk_elems, PT_STATIC_MAX_CHUNKS, PT_STATIC_MAX_PARTIALS,
                   PT_NORM_BLOCK_ELEMS);
  void* base = nullptr;
  int dev = 0;
  int rc = pt_static_scratch_setup(&base, &dev);
  if (rc != PT_OK) return rc;
  // every address below derives from the looked-up device address, never from the array's name
  PtStaticScratch* sc = static_cast<PtStaticScratch*>(base);
  hipStream_t st = (hipStream_t)stream;
  dim3 grid((uint32_t)blocks_per_chunk, n_chunks);
  const NormShape shape = norm_shape(chunk_elems * n_chunks, false);
  // Nothing here has to start at zero: each launch writes every partial and per-chunk slot that the
  // next one reads (n_chunks * blocks_per_chunk partials, n_chunks sums), so stale contents of an
  // earlier, larger call are never read.
  // Never under capture: a replay would use the same counter every time, and clear another one.  A count that calls which overlapped
  // have left in it would stay, and no workgroup of a later replay would be the last.  Two launches clear theirs themselves.
  const bool one = norm_in_one(blocks_per_chunk, n_chunks) && !pt_is_capturing(st);
  static std::atomic<uint32_t> calls[PT_STATIC_MAX_DEVICES];       // so far, a number each: every device has its own counters
  const uint32_t call = one ? calls[dev].fetch_add(1, std::memory_order_relaxed) : 0;
  norm_arena_kernel_t kern = dtype == PT_BF16 ? pick_norm_arena<PT_BF16>(shape.unroll, one) : pick_norm_arena<PT_FP16>(shape.unroll, one);
  hipLaunchKernelGGL(kern, grid, dim3(NB_THREADS), shape.lds, st, grad_arena, chunk_elems, loss_scale, sc->part, sc->flag,
                     one ? sc->tickets + call % PT_ONE_TICKETS : &sc->ticket, sc->tickets + (call + PT_ONE_TICKETS / 2) % PT_ONE_TICKETS,
                     out_sqnorm_norm, out_found_inf);
  if (hipGetLastError() != hipSuccess) return pt_fail(nullptr, PT_ERR_HIP, "pt_chunk_grad_sqnorm_noalloc: launch of k_sqnorm_arena failed");
  if (one) return PT_OK;
  PtScalarArgs a{};
  a.r.part = sc->part; a.r.flag = sc->flag; a.r.n = n_chunks; a.r.per_chunk = (uint32_t)blocks_per_chunk;
  a.r.segs = pt_segs(blocks_per_chunk); a.r.seg_sum = sc->seg_sum; a.r.seg_flag = sc->seg_flag;
  a.chunk_sq = sc->chunk_sq; a.chunk_flag = sc->chunk_flag; a.C = n_chunks; a.ticket = &sc->ticket.line[0].n;
  a.out_sq_norm = out_sqnorm_norm; a.out_found_inf = out_found_inf;
  a.do_finalize = 1;
  hipLaunchKernelGGL(k_scalars, dim3(a.r.segs, n_chunks), dim3(SC_THREADS), 0, st, a);
  if (hipGetLastError() != hipSuccess) return pt_fail(nullptr, PT_ERR_HIP, "pt_chunk_grad_sqnorm_noalloc: launch of k_scalars failed");
  return PT_OK;
}
