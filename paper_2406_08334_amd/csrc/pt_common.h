// Internal declarations shared by the translation units of libptchunk.so.
// Not part of the public boundary (that is include/ptchunk.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "ptchunk.h"
#include "pt_step.h"

// Device (global) address space qualifier for pointers rebuilt from integer addresses: the
// compiler then emits global_* memory instructions instead of flat_* ones.
#define PT_GLOBAL __attribute__((address_space(1)))

// Rows of the per-context device pointer table.  Each row has n_chunks + n_slots
// entries; entries [n_chunks, n_chunks + n_slots) are the device chunk buffers
// of the streamed path.
enum PtRow : int {
  ROW_GRAD = 0,
  ROW_MASTER = 1,
  ROW_M = 2,
  ROW_V = 3,
  ROW_P16 = 4,
  ROW_PACK = 5,    // gradient chunks as seen by pack / sqnorm
  ROW_UNPACK = 6,  // source chunks of unpack
  N_ROWS = 7
};

constexpr uint32_t PT_MAX_SLOTS = 8;
constexpr uint32_t PT_DIRECT_CHUNKS = 16;         // host chunks one launch of the in-place streamed update takes
constexpr uint32_t PT_ADAMW_LDS = 14848;           // unused LDS of an update workgroup: 11 workgroups fit a unit's 160 KiB
constexpr uint32_t PT_NORM_BLOCK_ELEMS = 32768;  // elements one block of the norm kernel reduces
constexpr uint32_t PT_PACK_TILE_ELEMS = 8192;    // chunk-space tile of a pack plan
constexpr uint32_t PT_PACK_SUBS = 4;             // waves that share a tile of the default size: a quarter each

struct PtTile {        // one piece of work of the pack / unpack / accumulate kernels, shared by `subs` waves of its plan
  uint64_t tensor_addr;  // byte address of the first element on the tensor side
  uint64_t chunk_off;    // first element on the chunk side
  uint32_t chunk;
  uint32_t len;          // 1 .. tile size of the plan
  uint32_t phase;        // chunk_off modulo the tile size: the waves' quarters are cut on its grid
  uint32_t pad;
};

struct pt_pack_plan {
  pt_ctx* ctx = nullptr;
  uint32_t n_tiles = 0;
  uint32_t subs = 1, sub_elems = 0;        // waves per tile, elements of the tile each of them takes
  PtTile* d_tiles = nullptr;
  uint32_t* d_chunk_tile_begin = nullptr;  // n_chunks + 1 entries (tiles sorted by chunk)
  double* d_tile_sq = nullptr;             // [n_tiles * subs]
  uint32_t* d_tile_flag = nullptr;
  uint32_t segs = 1;                       // reduction workgroups per chunk, for the chunk with the most tiles
  double* d_seg_sum = nullptr;             // [chunks from the first to the last touched one * segs], if segs > 1
  uint32_t* d_seg_flag = nullptr;
  uint64_t total_elems = 0;
  uint32_t kept_tiles = 0;                 // the first ones, whose unpacked words are to stay in the Infinity Cache
  uint64_t id = 0;                         // never reused within a context (a destroyed plan's address may be)
  std::vector<uint32_t> touched;           // chunks that own at least one tile
  std::vector<uint32_t> tile_begin;        // d_chunk_tile_begin from the first to behind the last touched chunk
};

namespace pt_host { class Pool; }

constexpr uint32_t PT_FUSED_ROW = 512;            // partial sums an update that derives its constants loads from a row's start on
constexpr uint32_t PT_REDUCE_SEG = 4096;         // partial sums one workgroup adds up, eight per lane
inline uint32_t pt_segs(uint64_t partials) { return uint32_t(partials ? (partials + PT_REDUCE_SEG - 1) / PT_REDUCE_SEG : 1); }

struct pt_ctx {
  int device = 0;
  int dtype = PT_BF16;
  uint64_t S = 0;          // chunk_elems
  uint32_t C = 0;          // n_chunks
  uint32_t norm_blocks = 0;  // blocks per chunk of the norm kernel
  uint32_t table_cols = 0;   // C + PT_MAX_SLOTS
  // launch-shape options (pt_ctx_set_option)
  uint32_t opt_adamw_grid = 0;      // workgroups of the update kernel; 0 = one per tile
  uint32_t opt_adamw_unroll = 0;    // 4-element units per lane per tile: 1, 2, 4 or 8; 0 = the library's shape (pt_adamw_shape)
  uint32_t opt_adamw_threads = 0;   // workgroup size of the update kernel: 256, 512, or 0 = the library's shape
  uint32_t opt_adamw_nt = 2;        // non-temporal hints on the update's loads and stores: 0 no, 1 or 2 yes (pt_adamw_hints)
  uint32_t opt_pack_tile_elems = PT_PACK_TILE_ELEMS;  // read when a pack plan is created
  uint32_t opt_in_place = 1;        // streamed update in place: 0 never, 1 where it can be, 2 or not at all
  bool scaler = false;
  bool grad_f32 = false;            // gradient chunks hold fp32 (accumulated micro-batches), option "grad_fp32"
  uint32_t opt_fused_tries = 1u << 13;  // looks of an update's waves for the constants that its first workgroup publishes
  uint32_t opt_zero_grads = 0;      // pt_chunk_adamw_step zeroes the gradient chunks it has read

  PtDevState* d_state = nullptr;
  uint64_t* d_table = nullptr;          // [N_ROWS][table_cols]
  std::vector<uint64_t> h_table;        // host shadow of d_table
  double* d_chunk_sq = nullptr;         // [C]
  uint32_t* d_chunk_flag = nullptr;     // [C]
  double* d_norm_part = nullptr;        // [C * norm_blocks]
  uint32_t* d_norm_flag = nullptr;      // [C * norm_blocks]
  uint32_t norm_segs = 1;               // reduction workgroups per chunk of a recompute
  double* d_norm_seg_sum = nullptr;     // [C * norm_segs], if norm_segs > 1
  uint32_t* d_norm_seg_flag = nullptr;

  uint64_t* d_pub = nullptr;            // constants published by an update that derives them itself (pt_scalars.h)
  uint32_t pub_no = 0;                  // such launches so far

  // host-side step bookkeeping
  std::vector<uint64_t> chunk_packed_by;   // [C] id of the pack plan whose partial sum is the chunk's value in this step, 0 = none
  uint64_t plan_ids = 0;
  std::vector<uint8_t> chunk_fresh;     // [C] 1 = the chunk's sum of squares was taken in this step (since pt_step_end)
  bool norm_finalized = false;
  bool prepared = false;
  uint32_t step_no = 1;                 // steps opened so far; never 0
  // Number of the step whose constants' launch has advanced the step counter and loss scale too, as long as no kernel that took that
  // into account has been launched and the step is open; 0: none.  A call under capture launches nothing, so it leaves this
  // as it is: then the device's own `ended` says whether a replay has closed the step or taken its end back.
  uint32_t ended_early = 0;
  bool captured = false;                // a call of this context has been captured into a graph
  bool goes_on = false;                 // an early end has been taken back: this context's steps do more behind their first update
  PtPendingReduce pend_reduce;                // scalar work put off to be fused into one launch (pt_norm.hip); n == 0: none
  bool pend_finalize = false;
  bool mirrored = false;                // the prepared constants are in h_state, with ev_scalar behind them
  pt_hparams prepared_hp{};

  // streamed path
  uint32_t n_slots = 0;
  void* slot_mem[PT_MAX_SLOTS] = {};
  hipStream_t s_up = nullptr, s_comp = nullptr, s_down = nullptr;
  hipEvent_t ev_fork = nullptr;
  hipEvent_t ev_up[PT_MAX_SLOTS] = {}, ev_k[PT_MAX_SLOTS] = {}, ev_down[PT_MAX_SLOTS] = {};
  // outcome of the duplex self-test of pt_stream_reserve: tested (the chunk buffers were large enough and the
  // scratch could be pinned), ok (upload and offload overlapped), offload streams tried
  uint32_t opt_force_unhealthy = 0;     // tests: the next look at a finished step finds it serialised whatever it measured
  uint32_t stream_rebuilds = 0;         // times the side streams were replaced after a serialised step
  void* h_trial = nullptr;              // pinned scratch of the trial copies (kept while chunk buffers are reserved)
  double link_one_dir_Bps = 0.0;        // one-direction rate of the link, from the reservation's trial copies
  hipEvent_t ev_t0 = nullptr, ev_t1 = nullptr;   // first upload may start / last offload done (timed)
  bool health_pending = false;
  uint64_t health_bytes = 0;            // bytes per direction of the step the two events bracket
  uint32_t health_chunks = 0;
  uint32_t opt_duplex_reject = 0;       // the self-test rejects that many offload streams whatever it measures (tests)
  bool duplex_tested = false, duplex_ok = false;
  uint32_t duplex_attempts = 0;
  bool slot_used[PT_MAX_SLOTS] = {};
  bool stream_pending = false;          // a streamed update of this step has not been joined yet ...
  bool slots_pending = false, direct_pending = false;   // ... through the chunk buffers / in place
  uint32_t last_slot = 0;
  hipEvent_t ev_direct = nullptr;       // behind the last in-place launch on s_comp
  bool direct_used = false;             // ev_direct has been recorded

  // weight-decay groups: per chunk, sorted disjoint element ranges kept out of the decay
  uint32_t* d_nd_begin = nullptr;        // [C + 1] indices into d_nd_ranges (NULL: no ranges set)
  uint64_t* d_nd_ranges = nullptr;       // pairs (lo, hi)
  std::vector<uint32_t> h_nd_begin;
  std::vector<uint64_t> h_nd_ranges;

  // host-side update: a pinned landing buffer for the step's constants and the event behind the kernel that fills it
  PtDevState* h_state_dev = nullptr;    // h_state as the device addresses it (the scalar kernels leave the constants there)
  hipEvent_t ev_scalar = nullptr;
  PtDevState* h_state = nullptr;
  pt_host::Pool* host_pool = nullptr;   // worker threads of the host-side update, started on first use
  uint32_t host_pool_threads = 0;       // n_threads the pool was built for

  std::string err;
};

// ---- error plumbing ----------------------------------------------------------------
int pt_fail(pt_ctx* ctx, int status, const char* fmt, ...) noexcept;

// Runs the body of an entry point that allocates host memory; a C++ exception becomes a status
// code, so that nothing is ever thrown across the C boundary.
template <class F>
inline int pt_guarded(pt_ctx* ctx, const char* who, F&& body) noexcept {
  try {
    return body();
  } catch (const std::bad_alloc&) {
    return pt_fail(ctx, PT_ERR_NOMEM, "%s: out of host memory", who);
  } catch (...) {
    return pt_fail(ctx, PT_ERR_UNSUPPORTED, "%s: unexpected C++ exception", who);
  }
}

#define PT_HIP(ctx, call)                                                              \
  do {                                                                                 \
    hipError_t e__ = (call);                                                           \
    if (e__ != hipSuccess)                                                             \
      return pt_fail((ctx), PT_ERR_HIP, "%s failed: %s (%s:%d)", #call,                \
                     hipGetErrorString(e__), __FILE__, __LINE__);                      \
  } while (0)

#define PT_LAUNCH_CHECK(ctx, name)                                                     \
  do {                                                                                 \
    hipError_t e__ = hipGetLastError();                                                \
    if (e__ != hipSuccess)                                                             \
      return pt_fail((ctx), PT_ERR_HIP, "launch of %s failed: %s", (name),             \
                     hipGetErrorString(e__));                                          \
  } while (0)

// ---- fixed-order reductions (device) ---------------------------------------------------
// Sum of `acc` and OR of `flag` over a wave, by a 64-lane shuffle tree: a fixed order, no atomics, so a result does
// not depend on timing.  Valid in lane 0 only.
__device__ __forceinline__ void pt_wave_sum(double& acc, uint32_t& flag) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  flag = __any(flag != 0) ? 1u : 0u;
}

// Closes a lane's sum of squares of stored gradients: the sum of the unscaled ones, and whether any was infinite or NaN.  Squares of
// 16-bit or fp32 numbers and sums of 2^40 of them stay far inside fp64's range, so the sum is finite if and only if every number
// is.  The loss scale is taken out here instead of from every number: a power of two gives the same bits either way, any
// other scale fewer roundings.  Widening, squaring and adding is then all a number costs; with the scaling and the bits of each
// word looked at it was two to three times the instructions, which calls feel that don't fill
// the memory's queues: norm of 8.4e6 words 9.9 -> 9.1 us, of 6e7 25.4 -> 23.9; a step of 7.1e6 parameters, of which pack is
// 8 us, 52.4 -> 51.5.
__device__ __forceinline__ void pt_close_sum(double sum, double inv_scale, double& acc, uint32_t& flag) {
  flag = (uint32_t(__double2hiint(sum)) & 0x7ff00000u) == 0x7ff00000u;
  acc = sum * inv_scale * inv_scale;
}

// The same over a workgroup of 256 threads: the tree per wave, then the four waves one after the other through LDS.
// Valid in thread 0 only.
constexpr int PT_REDUCE_THREADS = 256;

__device__ __forceinline__ void pt_block_sum(double& acc, uint32_t& flag) {
  __shared__ double s_sum[PT_REDUCE_THREADS / 64];
  __shared__ uint32_t s_flag[PT_REDUCE_THREADS / 64];
  double w = acc;
  uint32_t f = flag;
  pt_wave_sum(w, f);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) { s_sum[wid] = w; s_flag[wid] = f; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = s_sum[0];
    uint32_t g = s_flag[0];
#pragma unroll
    for (int i = 1; i < PT_REDUCE_THREADS / 64; ++i) { t += s_sum[i]; g |= s_flag[i]; }
    acc = t; flag = g;
  }
}

// The part of tile t that the wave blockIdx.x takes: elements [lo, hi) of the tile, possibly none.
__device__ __forceinline__ void pt_sub_range(const PtTile& t, uint32_t sub, uint32_t sub_elems, uint32_t& lo, uint32_t& hi) {
  const uint64_t end = uint64_t(t.phase) + t.len, a = uint64_t(sub) * sub_elems;      // on the tile's grid
  const uint64_t l = a > t.phase ? a : t.phase, h = a + sub_elems < end ? a + sub_elems : end;
  lo = uint32_t(l - t.phase);
  hi = h > l ? uint32_t(h - t.phase) : lo;
}

// Stores 8 or 16 bytes at byte `off` of `base`, which is the same in every lane, with a cache policy: none, the non-temporal hint, through the
// L2 at once instead of when its line is evicted (agent scope, sc1), or both.
//
// Stores that go through at once are the faster ones wherever the traffic is a mix of reads and writes, at every size, warm or cold: an
// evicted line is written at another time than its neighbours.  The update (all of its stores with the hint and through): 6.8e7
// parameters 355 -> 347 us a step, 6.67e8 3235 -> 3182, 1.4e7 88.4 -> 86.2; through without the hint 367, 3257, 90.0; neither 397,
// 3578, 96.8.  Words and sums that are to stay in the Infinity Cache (pt_in_cache) go through without the hint: packed words plainly and
// so 6.8e7 343.3 -> 340.3, 1.24e8 596.7 -> 591.7, 1.4e7 86.4 -> 85.2 (with the hint 353, 612, 89); sums added to with the hint and so, one
// call behind 2 GB of other traffic: 7.3e6 18.5 -> 17.3, 1.6e7 31.6 -> 29.2, 3e7 53.1 -> 50.0, 5.3e7 89.2 -> 84.3; sums the update zeroes
// likewise: four micro-batches and update 7e6 108.3 -> 104.3, 3e7 337 -> 335, 1.24e8 1350 -> 1334, 3.3e8 3603 -> 3585.  Sums
// beyond it have the hint alone (through: 3.3e8 3655).  All figures of arrays that both sides share: where a process's arrays lie moves its steps by
// 1 % either way.
constexpr int PT_PLAIN = 0, PT_NT = 2, PT_THROUGH = 16, PT_NT_THROUGH = 18;
typedef int pt_i32x4 __attribute__((ext_vector_type(4)));
typedef int pt_i32x2 __attribute__((ext_vector_type(2)));
template <int POLICY, class T>
__device__ __forceinline__ void pt_store(T v, PT_GLOBAL void* base, uint32_t off) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)base, 0, 0xffffffffu, 0x27000);
  if constexpr (sizeof(T) == 16) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(pt_i32x4, v), r, off, 0, POLICY);
  else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(pt_i32x2, v), r, off, 0, POLICY);
}

// ---- helpers implemented in pt_ctx.hip ---------------------------------------------
// Makes rows[r][first .. first+n) of the device pointer table equal to ptrs[0..n), for each of n_binds rows; uploads (on
// `stream`, which it synchronises) only when something changed.
// allow_null: NULL entries are accepted (and stored as 0).
struct PtBind { int row; const void* const* ptrs; };
int pt_table_bind(pt_ctx* ctx, const PtBind* binds, int n_binds, uint32_t first, uint32_t n, bool allow_null, hipStream_t stream);
inline int pt_table_bind(pt_ctx* ctx, int row, uint32_t first, uint32_t n, const void* const* ptrs, bool allow_null, hipStream_t stream) {
  const PtBind b{row, ptrs};
  return pt_table_bind(ctx, &b, 1, first, n, allow_null, stream);
}
inline const uint64_t* pt_row(const pt_ctx* ctx, int row) {
  return ctx->d_table + size_t(row) * ctx->table_cols;
}

// ---- implemented in pt_adamw.hip ------------------------------------------------------
// recast_on_skip: on a skipped step rewrite param16 = RNE(master) instead of doing nothing.
// mask_chunk0: chunk index (for the no-decay ranges) of table column first_col.
// zero_grads: overwrite the gradient chunks with zeros once read (resident chunks only).
// Launch shape of an update over n_cols chunks.  Left to itself: one wave per workgroup, one unit per lane, 11 workgroups per
// compute unit - the best of the shapes at every size measured, 0.8 M to 6.8e9 elements (figures at k_adamw).  With
// adamw_threads or adamw_unroll set: that shape without a limit, the other of the two by the size of the launch (512 threads
// from 2^28 elements on) or four units.
struct PtAdamwShape { uint32_t threads, unroll, lds; };
inline PtAdamwShape pt_adamw_shape(const pt_ctx* ctx, uint32_t n_cols) {
  if (!ctx->opt_adamw_threads && !ctx->opt_adamw_unroll) return {64, 1, PT_ADAMW_LDS};
  const uint32_t by_size = ctx->S * uint64_t(n_cols) >= (uint64_t(1) << 28) ? 512u : 256u;
  return {ctx->opt_adamw_threads ? ctx->opt_adamw_threads : by_size, ctx->opt_adamw_unroll ? ctx->opt_adamw_unroll : 4u, 0};
}
// Non-temporal hints of an update launch.  On unless switched off: in the library's shape they gain 4-15 % at every size,
// whether the state was last touched a step ago or 512 MB of other traffic earlier (update with and without hints: 16 MB
// of state 16.0 / 17.8 us, 108 MB 45.3 / 51.8, 108 MB touched just before 44.6 / 48.2, 733 MB 217 / 237).
// The gradient chunks are the exception: what pack or accumulate has written, the next accumulation or the update reads.  Pack
// stores and accumulate loads the first PT_CACHED_BYTES of them without a hint (the update all of them: it is their last
// reader), and they stay in the 256 MB Infinity Cache from call to call; traffic with hints does not take it from them, but words
// without hints beyond its size push each other out.  16-bit words, a step of 68 M parameters 370 -> 357 us, 124 M 631 -> 615,
// 200 M 1075 -> 1067, 667 M within its spread.
// fp32 sums, four micro-batches and the update, with hints and without: 3e7 elements 363 and 353 us, 5.3e7 612 and 589, 1.24e8
// 1422 and 1364, 3.3e8 3715 and 3635 (without hints on all of them 3800); 192 to 240 MB differ by less than 1 %, 300 MB costs
// 1.24e8 elements 5 %.  In training a forward and a backward pass come in between, which take the cache for themselves; then
// smaller sums are better off with the hints.  One call behind 2 GB of other traffic, with and without: 4.2e6 elements
// 13.0 and 14.1 us, 7.3e6 18.0 and 19.1, 1.6e7 30.2 and 32.1, 2.3e7 40.8 and 41.6, 3e7 51.5 and 51.3, 5.3e7 86.8 and 87.7, 1.0e8 155.4
// and 154.9.  Hence the line (below it, call behind call: 4.2e6 11.3 and 11.5, 7.3e6 16.9 and 14.8, 1.6e7 29.0 and 29.4, 2.3e7 39.4 and 38.7).
inline bool pt_adamw_hints(const pt_ctx* ctx) { return ctx->opt_adamw_nt != 0; }
constexpr uint64_t PT_CACHED_BYTES = 240ull << 20, PT_CACHED_SUMS = 3ull << 23;
inline uint64_t pt_cached_elems(const pt_ctx* ctx) { return PT_CACHED_BYTES / (ctx->grad_f32 ? 4 : 2); }
inline uint64_t pt_cached_loads(const pt_ctx* ctx) {
  return ctx->grad_f32 && ctx->S * ctx->C < PT_CACHED_SUMS ? 0 : pt_cached_elems(ctx);
}
// Whether element `off` of chunk `chunk` (of S elements each) is one of the first `cached`.
__device__ __forceinline__ bool pt_in_cache(uint32_t chunk, uint64_t S, uint64_t off, uint64_t cached) { return chunk * S + off < cached; }
struct PtFused;
// fused: the step's scalar work that the update of all chunks takes along (pt_fuse_scalars), or NULL.
int pt_launch_adamw(pt_ctx* ctx, uint32_t first_col, uint32_t n_cols, hipStream_t stream, bool recast_on_skip,
                    uint32_t mask_chunk0, bool zero_grads, const PtFused* fused = nullptr);
// The update of n chunks in pinned host memory, in place (at[i]: gradient, master, m, v, param16 of chunk i as device
// addresses; fp32 arrays 16-byte, 16-bit ones 8-byte aligned).  A skipped step recasts param16.
int pt_launch_adamw_host(pt_ctx* ctx, const uint64_t (*at)[5], uint32_t n, hipStream_t stream, uint32_t mask_chunk0);

// ---- implemented in pt_stream.hip ----------------------------------------------------------
// Destroys the streamed path's streams and events and frees its chunk buffers (no-op when none).
void pt_stream_release(pt_ctx* ctx);

// ---- implemented in pt_host.hip ------------------------------------------------------------
// Stops and joins the context's worker threads (no-op when there are none).
void pt_host_pool_destroy(pt_ctx* ctx);

// ---- implemented in pt_norm.hip ---------------------------------------------------------
// Looks up (once per device) the device address of the file-scope scratch array that
// pt_chunk_grad_sqnorm_noalloc works in; out and device may be NULL.  Called by pt_ctx_create, so that a process
// with a context never pays the lookup inside a hot call.
int pt_static_scratch_setup(void** out, int* device = nullptr);
// The reduction of a plan's tile sums (pack, accumulate) to per-chunk values: launched on `stream`, a small plan's put off until the
// norm is read or another call's sums come.
int pt_reduce_plan(pt_ctx* ctx, const pt_pack_plan* plan, hipStream_t stream);
inline bool pt_is_capturing(hipStream_t stream) {      // whether `stream` is being captured into a graph
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cs) != hipSuccess) (void)hipGetLastError();
  return cs != hipStreamCaptureStatusNone;
}
// The same; the context remembers that it ever was.  Every call that reads or changes what the end of a step changes asks first of
// all: a graph holds such a call then, and may be replayed anywhere in a later step, so those end in a kernel of their own.
// Unpacking and adding without the norm read none of it and do not ask (a question costs 0.1 us).
bool pt_capturing(pt_ctx* ctx, hipStream_t stream);
// Before a call on `stream` that reads or changes what the end of a step changes: takes an early end of this step back.
int pt_reopen_step(pt_ctx* ctx, hipStream_t stream);
// Launches, on `stream`, whatever scalar work of the step has been put off (a per-chunk reduction, the finalize).
// Every call that reads the step's scalars goes through this first.
int pt_flush_pending(pt_ctx* ctx, hipStream_t stream);
// Before a kernel on `stream` that writes partial sums.
int pt_before_partials(pt_ctx* ctx, hipStream_t stream);
// Derives this step's update constants from `hp` if that has not happened yet - in one launch together
// with any pending reduction and finalize.  host_part: chunks the calling update leaves out may be updated on the host.
int pt_prepare_consts(pt_ctx* ctx, const pt_hparams* hp, bool host_part, hipStream_t stream);
// Whether an update of all chunks can take this step's scalar work along in its own launch instead (then *fused holds the work), and what
// follows once that has been launched.
bool pt_fuse_scalars(pt_ctx* ctx, const pt_hparams* hp, PtFused* fused);
void pt_fused_launched(pt_ctx* ctx, const PtFused& fused);
// Makes sure the prepared constants are on their way to h_state, with ev_scalar behind them.
int pt_mirror_consts(pt_ctx* ctx, hipStream_t stream);
