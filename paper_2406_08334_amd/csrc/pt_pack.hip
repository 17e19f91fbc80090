// Pack gradients into chunks (and the inverse copy), one wave per quarter of a tile of a
// precomputed work list, fused with the wave's sum of squares and the
// non-finite scan.
//
// HBM-bound: 2 bytes read + 2 bytes written per element.  Tiles are cut in
// CHUNK space at multiples of the tile size (PT_PACK_TILE_ELEMS by default), so many tiny tensors and a few
// huge ones give equally sized workgroups.  Words are moved as 16-bit integers,
// never through a float.  The 16-byte vector body is aligned on the destination;
// when source and destination are not congruent modulo 16 bytes the source side
// is read with 16-byte loads at 2-byte alignment.
#include "pt_common.h"

#include <hip/hip_fp16.h>

#include <algorithm>
#include <memory>

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int PK_THREADS = 64;

// The square of one word joins the sum (two 16-bit significands multiply exactly: only the addition rounds).
template <int DT>
__device__ __forceinline__ void take(uint32_t w16, double& sum) {
  double x;
  if (DT == PT_BF16) {
    x = (double)__uint_as_float(w16 << 16);
  } else {
    __half_raw r; r.x = (unsigned short)w16;
    x = (double)__half2float(__half(r));
  }
  sum = fma(x, x, sum);
}

template <int DT>
__device__ __forceinline__ void take_vec(const u32x4& q, double& a0, double& a1) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    take<DT>(q[k] & 0xffffu, a0);
    take<DT>(q[k] >> 16, a1);
  }
}

typedef u32x4 u32x4_a2 __attribute__((aligned(2)));   // global memory takes a 16-byte load at any address

// Off the alignment every line at a lane's or a wave's end is read twice, and unpack takes it without the hint: with and
// without, from memory 15e6 words 16.4 and 16.2 us, 6e7 51.5 and 51.8 (8-byte aligned 49.4 and 47.0), 3.3e8 251 and 252
// (237 and 224); from the Infinity Cache 15e6 14.9 and 10.2, 6e7 49.8 and 33.7.  Pack, whose words come from a backward pass,
// is 5 % faster with it from memory (3e7 words 23.6 and 24.9 us).
template <int DIR, bool ALIGNED>
__device__ __forceinline__ u32x4 load_vec(const PT_GLOBAL uint16_t* s) {
  if (ALIGNED) return __builtin_nontemporal_load((const PT_GLOBAL u32x4*)s);
  return DIR == 1 ? *(const PT_GLOBAL u32x4_a2*)s : __builtin_nontemporal_load((const PT_GLOBAL u32x4_a2*)s);
}

// nvec vectors from sb to db: two per lane in flight.
template <int DT, int DIR, bool KEEP, bool ALIGNED>
__device__ __forceinline__ void move_vecs(const PT_GLOBAL uint16_t* sb, PT_GLOBAL u32x4* db, uint32_t nvec, double& a0, double& a1) {
  constexpr int U = 2, POLICY = KEEP ? PT_THROUGH : PT_NT_THROUGH;
  uint32_t i = threadIdx.x;
  for (; i + (U - 1) * PK_THREADS < nvec; i += U * PK_THREADS) {
    u32x4 q[U];
#pragma unroll
    for (int r = 0; r < U; ++r) q[r] = load_vec<DIR, ALIGNED>(sb + size_t(i + r * PK_THREADS) * 8);
#pragma unroll
    for (int r = 0; r < U; ++r) pt_store<POLICY>(q[r], db, (i + r * PK_THREADS) * 16);
    if (DIR == 0)
#pragma unroll
      for (int r = 0; r < U; ++r) take_vec<DT>(q[r], a0, a1);
  }
  for (; i < nvec; i += PK_THREADS) {
    const u32x4 q = load_vec<DIR, ALIGNED>(sb + size_t(i) * 8);
    pt_store<POLICY>(q, db, i * 16);
    if (DIR == 0) take_vec<DT>(q, a0, a1);
  }
}

// DIR 0: tensor -> chunk with sum of squares and non-finite scan (pack).
// DIR 1: chunk -> tensor (unpack), no reduction.
// cached: of packed words as many, of unpacked ones those of as many tiles.
// KEEP: words that stay in the Infinity Cache: packed ones for the update (pt_in_cache), unpacked ones for whoever reads the tensors (UNPACK_KEPT).
//
// Few bytes in flight, in address order, are moved fastest (as in the update).  One wave moves 4 KiB, two vectors a lane at a
// time, and unused LDS keeps few waves on a compute unit.  Against workgroups of four waves with 16 KiB, eight on a unit: pack of
// 1.56e9 elements 1012 -> 955 us (6.5 TB/s), 6.7e8 fp16 words 438 -> 414; unpack of 6.7e8 425 -> 404 us (6.6 TB/s).  2 KiB per wave cost
// pack 20 % (too little work behind the look-up of a tile), 8 KiB 6-8 %.
// Pack: two vectors a lane in flight and about 17 waves a unit.  With four and 17, two and 17, two and 13, two and 10, the kernel by
// itself: 7.1e6 words 7.8 / 7.1 / 8.1 / 8.0 us, 2.8e7 20.7 / 20.6 / 21.7 / 22.6, 3.4e8 209 / 207 / 210 / 223, 1.56e9 974 / 959 / 956 /
// 1021.  Whole steps, four and two in turn: 7.1e6 51.5-52.0 and 50.9-51.1 us, larger ones within 0.5 %, which is their spread; with 13
// waves no step from 6.8e7 to 1.56e9 is faster (1.24e8 617 with 17 waves, 619 with 13).  Four in flight suited pack as long as every
// word cost it two to three times the instructions.
// Unpack: the limit gives 2-5 %: 1e7 words 8.1 -> 7.9 us, 3.7e7 24.7 -> 23.7, 1.25e8 79.8 -> 77.0, 6.3e8 404 -> 386.  About 14 waves are
// better still from 2^28 words on (4.1e8 262.5 and 259.2 us, 1.4e9 858 and 849) and worse below (2.0e7 13.7 and
// 14.2 us, 5.5e7 34.5 and 35.0, 1.25e8 77.0 and 77.6); below 2^24 words it runs without a limit (1.5e7 11.6, with one 11.8).
constexpr uint32_t PACK_LDS = 9000;
inline uint32_t unpack_lds(uint64_t elems) { return elems < (1ull << 24) ? 0 : elems < (1ull << 28) ? 9000 : 11500; }
// Stores (pt_store).  Unpacked words go through the L2 without the hint, so that the forward pass finds them in the Infinity Cache: the plan's first
// 240 MB (as of packed ones, whose place in the context counts), the rest with it.  All with the hint, the first 240 MB without, one call behind 2 GB of
// other traffic and a pass that reads the tensors from the first on: 6.1e7 words 42 + 51 and 39 + 34 us, 1.0e8 65 + 75 and 60 + 47, 1.35e8 86 + 96
// and 78 + 63, 2.0e8 124 + 131 and 116 + 105, 2.6e8 160 + 162 and 152 + 143, 6.7e8 391 + 375 and 391 + 357, 1.4e9 823 + 774 and 825 + 757; the call repeated
// 38.6 and 35.7, 61.6 and 56.2, 82.0 and 75.0, 120.7 and 113.4, 156.3 and 149.1, 395.8 and 389.4, 841 and 833.  None with the hint is as fast up to 1.3e8
// words; from there on the reading pass finds nothing and waits for what is still to be written: 1.45e8 83 + 114, 2.0e8 114 + 145, 6.7e8 389 + 391,
// 1.4e9 825 + 792.  The first 120 MB: 1.0e8 61 + 59, 2.0e8 120 + 120, 6.7e8 396 + 367; 200 MB: 2.0e8 118 + 108, 6.7e8 392 + 361; 256 MB: 2.0e8 116 + 134.
// Packed words that don't fit the cache: through with the hint; with the hint alone a step, on the same arrays, takes the same within 0.3 %, 1.8e8
// parameters 865 and 865 us, 6.7e8 3185 and 3180, 1.56e9 7486 and 7462.
constexpr uint64_t UNPACK_KEPT = PT_CACHED_BYTES / 2;

template <int DT, int DIR>
__global__ void __launch_bounds__(PK_THREADS)
k_pack(const PtTile* __restrict__ tiles, const uint64_t* __restrict__ chunk_row, uint32_t subs, uint32_t sub_elems,
       const PtDevState* __restrict__ st, double* __restrict__ tile_sq, uint32_t* __restrict__ tile_flag, uint64_t S, uint64_t cached) {
  const uint32_t tile = blockIdx.x / subs;
  const PtTile t = tiles[tile];
  uint32_t lo, hi;
  pt_sub_range(t, blockIdx.x - tile * subs, sub_elems, lo, hi);
  // both sides are device (global) memory: typed so, to get global_* instead of flat_* accesses
  PT_GLOBAL uint16_t* chunk_side = (PT_GLOBAL uint16_t*)(chunk_row[t.chunk]) + t.chunk_off + lo;
  PT_GLOBAL uint16_t* tensor_side = (PT_GLOBAL uint16_t*)(t.tensor_addr) + lo;
  const PT_GLOBAL uint16_t* src = DIR == 0 ? tensor_side : chunk_side;
  PT_GLOBAL uint16_t* dst = DIR == 0 ? chunk_side : tensor_side;
  const uint32_t len = hi - lo;

  // elements before the destination reaches a 16-byte boundary
  uint32_t head = uint32_t(((16u - (uint32_t((uintptr_t)dst) & 15u)) & 15u) >> 1);
  if (head > len) head = len;
  const uint32_t nvec = (len - head) / 8;
  const uint32_t tail0 = head + nvec * 8;

  const double inv_scale = DIR == 0 ? 1.0 / st->loss_scale : 1.0;
  double a0 = 0.0, a1 = 0.0;

  const PT_GLOBAL uint16_t* sb = src + head;
  PT_GLOBAL u32x4* db = (PT_GLOBAL u32x4*)(dst + head);
  const bool aligned = ((uintptr_t)sb & 15u) == 0;
  if (DIR == 0 ? pt_in_cache(t.chunk, S, t.chunk_off, cached) : tile < cached) {
    if (aligned) move_vecs<DT, DIR, true, true>(sb, db, nvec, a0, a1);
    else move_vecs<DT, DIR, true, false>(sb, db, nvec, a0, a1);
  } else {
    if (aligned) move_vecs<DT, DIR, false, true>(sb, db, nvec, a0, a1);
    else move_vecs<DT, DIR, false, false>(sb, db, nvec, a0, a1);
  }

  // head and tail: at most 7 elements each, one lane per element
  if (threadIdx.x < head) {
    const uint16_t w = src[threadIdx.x];
    dst[threadIdx.x] = w;
    if (DIR == 0) take<DT>(w, a0);
  }
  if (threadIdx.x < len - tail0) {
    const uint32_t e = tail0 + threadIdx.x;
    const uint16_t w = src[e];
    dst[e] = w;
    if (DIR == 0) take<DT>(w, a1);
  }

  if (DIR == 0) {
    double acc;
    uint32_t flag;
    pt_close_sum(a0 + a1, inv_scale, acc, flag);
    pt_wave_sum(acc, flag);
    if (threadIdx.x == 0) {
      tile_sq[blockIdx.x] = acc;
      tile_flag[blockIdx.x] = flag;
    }
  }
}

}  // namespace

// ---- plan ----------------------------------------------------------------------------------

static void plan_free(pt_pack_plan* p) {
  if (p->d_tiles) (void)hipFree(p->d_tiles);
  if (p->d_chunk_tile_begin) (void)hipFree(p->d_chunk_tile_begin);
  if (p->d_tile_sq) (void)hipFree(p->d_tile_sq);
  if (p->d_tile_flag) (void)hipFree(p->d_tile_flag);
  if (p->d_seg_sum) (void)hipFree(p->d_seg_sum);
  if (p->d_seg_flag) (void)hipFree(p->d_seg_flag);
}

static int plan_create(pt_ctx* ctx, const pt_segment* segs, uint32_t n_segs, pt_pack_plan** out);

extern "C" int pt_pack_plan_create(pt_ctx* ctx, const pt_segment* segs, uint32_t n_segs, pt_pack_plan** out) {
  if (!ctx) return PT_ERR_INVALID_ARG;
  if (!out || (!segs && n_segs)) return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_pack_plan_create: NULL argument");
  *out = nullptr;
  return pt_guarded(ctx, "pt_pack_plan_create", [&] { return plan_create(ctx, segs, n_segs, out); });
}

static int plan_create(pt_ctx* ctx, const pt_segment* segs, uint32_t n_segs, pt_pack_plan** out) {
  // validate: inside chunks, sources present and 2-byte aligned, no overlap inside a chunk
  std::vector<uint32_t> order(n_segs);
  for (uint32_t i = 0; i < n_segs; ++i) {
    const pt_segment& s = segs[i];
    if (!s.src) return pt_fail(ctx, PT_ERR_INVALID_ARG, "segment %u: src is NULL", i);
    if (reinterpret_cast<uintptr_t>(s.src) & 1u) return pt_fail(ctx, PT_ERR_ALIGNMENT, "segment %u: src is not 2-byte aligned", i);
    if (s.len == 0) return pt_fail(ctx, PT_ERR_INVALID_ARG, "segment %u: len is 0", i);
    if (s.chunk >= ctx->C) return pt_fail(ctx, PT_ERR_INVALID_ARG, "segment %u: chunk %u outside the context's %u chunks", i, s.chunk, ctx->C);
    if (s.chunk_off >= ctx->S || s.len > ctx->S - s.chunk_off)
      return pt_fail(ctx, PT_ERR_INVALID_ARG, "segment %u: [%llu, +%llu) overruns the chunk of %llu elements", i,
                     (unsigned long long)s.chunk_off, (unsigned long long)s.len, (unsigned long long)ctx->S);
    order[i] = i;
  }
  std::sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
    if (segs[a].chunk != segs[b].chunk) return segs[a].chunk < segs[b].chunk;
    return segs[a].chunk_off < segs[b].chunk_off;
  });
  for (uint32_t k = 1; k < n_segs; ++k) {
    const pt_segment& p = segs[order[k - 1]];
    const pt_segment& q = segs[order[k]];
    if (p.chunk == q.chunk && p.chunk_off + p.len > q.chunk_off)
      return pt_fail(ctx, PT_ERR_INVALID_ARG, "segments %u and %u overlap in chunk %u", order[k - 1], order[k], p.chunk);
  }
  // cut into tiles at multiples of the tile size in chunk space
  // With fp32 gradient chunks the plan feeds the accumulate kernel, which moves 2.5 times the
  // bytes per element: half the tile (figures at k_accum).
  const uint64_t tile_elems = ctx->grad_f32 ? std::max<uint64_t>(1024, ctx->opt_pack_tile_elems / 2)
                                            : ctx->opt_pack_tile_elems;
  std::vector<PtTile> tiles;
  uint64_t room_for = 0;
  for (uint32_t i = 0; i < n_segs; ++i) room_for += segs[i].len / tile_elems + 2;
  tiles.reserve(room_for);
  std::vector<uint32_t> begin(size_t(ctx->C) + 1, 0);
  uint64_t total = 0;
  uint32_t kept = 0;
  for (uint32_t k = 0; k < n_segs; ++k) {
    const pt_segment& s = segs[order[k]];
    uint64_t done = 0;
    while (done < s.len) {
      uint64_t coff = s.chunk_off + done;
      uint64_t room = tile_elems - (coff % tile_elems);
      uint64_t run = std::min<uint64_t>(room, s.len - done);
      PtTile t;
      t.tensor_addr = uint64_t(reinterpret_cast<uintptr_t>(s.src)) + 2 * (s.src_off + done);
      t.chunk_off = coff; t.chunk = s.chunk; t.len = uint32_t(run); t.phase = uint32_t(coff % tile_elems); t.pad = 0;
      tiles.push_back(t);
      begin[s.chunk + 1] += 1;
      done += run;
      total += run;
      if (total <= UNPACK_KEPT) kept = uint32_t(tiles.size());
    }
  }
  // a tile of the default size goes to four waves; one of another size to as many, if it has 2048 (1024) elements for each
  const uint64_t least = ctx->grad_f32 ? 1024 : 2048;
  const uint32_t subs = uint32_t(std::min<uint64_t>(PT_PACK_SUBS, (tile_elems + least - 1) / least));
  const uint32_t sub_elems = uint32_t(((tile_elems + subs - 1) / subs + 7) & ~uint64_t(7));
  if (tiles.size() * subs > 0x7fffffffull) return pt_fail(ctx, PT_ERR_UNSUPPORTED, "pt_pack_plan_create: too many tiles");
  for (uint32_t c = 0; c < ctx->C; ++c) begin[c + 1] += begin[c];

  pt_pack_plan* p = new (std::nothrow) pt_pack_plan();
  if (!p) return pt_fail(ctx, PT_ERR_NOMEM, "pt_pack_plan_create: out of host memory");
  std::unique_ptr<pt_pack_plan> hold(p);            // freed on every early return and on an exception
  p->ctx = ctx; p->n_tiles = uint32_t(tiles.size()); p->total_elems = total; p->kept_tiles = kept;
  p->id = ++ctx->plan_ids;
  uint32_t most = 0;
  for (uint32_t c = 0; c < ctx->C; ++c)
    if (begin[c + 1] > begin[c]) { p->touched.push_back(c); most = std::max(most, begin[c + 1] - begin[c]); }
  if (!p->touched.empty()) p->tile_begin.assign(begin.begin() + p->touched.front(), begin.begin() + p->touched.back() + 2);
  p->subs = subs; p->sub_elems = sub_elems;
  p->segs = pt_segs(uint64_t(most) * subs);
  auto bail = [&](hipError_t e, const char* what) {
    plan_free(p);
    p->d_tiles = nullptr; p->d_chunk_tile_begin = nullptr; p->d_tile_sq = nullptr; p->d_tile_flag = nullptr;
    p->d_seg_sum = nullptr; p->d_seg_flag = nullptr;
    return pt_fail(ctx, PT_ERR_HIP, "pt_pack_plan_create: %s failed: %s", what, hipGetErrorString(e));
  };
  hipError_t e;
  size_t nt = std::max<size_t>(tiles.size(), 1);
  if ((e = hipMalloc(&p->d_tiles, nt * sizeof(PtTile))) != hipSuccess) return bail(e, "hipMalloc(tiles)");
  if ((e = hipMalloc(&p->d_chunk_tile_begin, begin.size() * sizeof(uint32_t))) != hipSuccess) return bail(e, "hipMalloc(begin)");
  if ((e = hipMalloc(&p->d_tile_sq, (nt * subs + PT_FUSED_ROW) * sizeof(double))) != hipSuccess) return bail(e, "hipMalloc(tile_sq)");
  if ((e = hipMalloc(&p->d_tile_flag, nt * subs * sizeof(uint32_t))) != hipSuccess) return bail(e, "hipMalloc(tile_flag)");
  if (p->segs > 1) {
    const size_t ns = size_t(p->touched.back() - p->touched.front() + 1) * p->segs;
    if ((e = hipMalloc(&p->d_seg_sum, ns * sizeof(double))) != hipSuccess) return bail(e, "hipMalloc(seg_sum)");
    if ((e = hipMalloc(&p->d_seg_flag, ns * sizeof(uint32_t))) != hipSuccess) return bail(e, "hipMalloc(seg_flag)");
  }
  if (!tiles.empty() &&
      (e = hipMemcpy(p->d_tiles, tiles.data(), tiles.size() * sizeof(PtTile), hipMemcpyHostToDevice)) != hipSuccess)
    return bail(e, "hipMemcpy(tiles)");
  if ((e = hipMemcpy(p->d_chunk_tile_begin, begin.data(), begin.size() * sizeof(uint32_t), hipMemcpyHostToDevice)) != hipSuccess)
    return bail(e, "hipMemcpy(begin)");
  *out = hold.release();
  return PT_OK;
}

extern "C" int pt_pack_plan_destroy(pt_pack_plan* plan) {
  if (!plan) return PT_OK;
  (void)hipDeviceSynchronize();
  // a reduction of this plan's partial sums that was put off runs now, before they are freed (the device is idle: any
  // stream will do, and the one of the pack may be gone)
  if (plan->ctx && plan->ctx->pend_reduce.n && plan->ctx->pend_reduce.plan == plan) {
    pt_ctx* ctx = plan->ctx;
    if (pt_flush_pending(ctx, nullptr) != PT_OK) {
      // the sums are lost with the plan: nothing may read them, and their chunks have no value from this step
      ctx->pend_reduce = PtPendingReduce{};
      if (ctx->pend_finalize) ctx->pend_finalize = ctx->norm_finalized = false;
      for (uint32_t c : plan->touched) ctx->chunk_fresh[c] = 0;
    }
    (void)hipDeviceSynchronize();
  }
  if (plan->ctx)      // a plan that no longer exists does not stand in another plan's way
    for (uint32_t c : plan->touched)
      if (plan->ctx->chunk_packed_by[c] == plan->id) plan->ctx->chunk_packed_by[c] = 0;
  plan_free(plan);
  delete plan;
  return PT_OK;
}

// ---- hot calls --------------------------------------------------------------------------------

template <int DIR>
static int run_pack(pt_ctx* ctx, const pt_pack_plan* plan, const void* const* chunks, int row, hipStream_t st,
                    const char* who) {
  if (!plan || !chunks) return pt_fail(ctx, PT_ERR_INVALID_ARG, "%s: NULL argument", who);
  if (plan->ctx != ctx) return pt_fail(ctx, PT_ERR_INVALID_ARG, "%s: plan belongs to another context", who);
  if (DIR == 0) pt_capturing(ctx, st);
  int rc = pt_table_bind(ctx, row, 0, ctx->C, chunks, true, st);
  if (rc != PT_OK) return rc;
  if (plan->n_tiles == 0) return PT_OK;
  // every chunk the plan touches needs a pointer (NULL is legal only for untouched chunks)
  const uint64_t* h = ctx->h_table.data() + size_t(row) * ctx->table_cols;
  for (uint32_t c : plan->touched)
    if (!h[c]) return pt_fail(ctx, PT_ERR_INVALID_ARG, "%s: chunk %u is used by the plan but its pointer is NULL", who, c);
  if (DIR == 0) {
    // A chunk's sum of squares is the partial of the LAST plan that packed into it: a second plan on the same
    // chunk in one step would silently drop the first plan's share from the norm.
    for (uint32_t c : plan->touched)
      if (ctx->chunk_packed_by[c] && ctx->chunk_packed_by[c] != plan->id)
        return pt_fail(ctx, PT_ERR_STATE, "%s: chunk %u already holds the gradients of another plan of this step; its sum of "
                       "squares would be replaced, not added to - pack a chunk with one plan per step (or recompute the "
                       "norm from the chunks with pt_chunk_grad_sqnorm(grad_chunks, ...) before packing again)", who, c);
    if ((rc = pt_reopen_step(ctx, st)) != PT_OK || (rc = pt_before_partials(ctx, st)) != PT_OK) return rc;
  }
  dim3 grid(plan->n_tiles * plan->subs);
  const size_t lds = DIR == 1 ? unpack_lds(plan->total_elems) : PACK_LDS;
  auto kern = ctx->dtype == PT_BF16 ? k_pack<PT_BF16, DIR> : k_pack<PT_FP16, DIR>;
  hipLaunchKernelGGL(kern, grid, dim3(PK_THREADS), lds, st, plan->d_tiles, pt_row(ctx, row), plan->subs, plan->sub_elems,
                     ctx->d_state, plan->d_tile_sq, plan->d_tile_flag, ctx->S,
                     DIR == 1 ? uint64_t(plan->kept_tiles) : pt_cached_elems(ctx));
  PT_LAUNCH_CHECK(ctx, who);
  if (DIR == 0) {
    rc = pt_reduce_plan(ctx, plan, st);
    if (rc != PT_OK) return rc;
    for (uint32_t c : plan->touched) { ctx->chunk_fresh[c] = 1; ctx->chunk_packed_by[c] = plan->id; }
  }
  return PT_OK;
}

extern "C" int pt_chunk_pack_grads(pt_ctx* ctx, const pt_pack_plan* plan, void* const* grad_chunks, void* stream) {
  if (!ctx) return PT_ERR_INVALID_ARG;
  if (ctx->grad_f32)
    return pt_fail(ctx, PT_ERR_STATE, "pt_chunk_pack_grads: this context holds fp32 gradient chunks; use pt_chunk_accum_grads");
  return run_pack<0>(ctx, plan, (const void* const*)grad_chunks, ROW_PACK, (hipStream_t)stream, "pt_chunk_pack_grads");
}

extern "C" int pt_chunk_unpack(pt_ctx* ctx, const pt_pack_plan* plan, const void* const* chunks, void* stream) {
  if (!ctx) return PT_ERR_INVALID_ARG;
  return run_pack<1>(ctx, plan, chunks, ROW_UNPACK, (hipStream_t)stream, "pt_chunk_unpack");
}
