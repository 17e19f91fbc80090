// Gradient accumulation over micro-batches: the 16-bit gradient tensors of one
// micro-batch are added into fp32 gradient chunks (or overwrite them, for the first
// micro-batch), over the same tile list as pack; on the last micro-batch the per-tile
// sum of squares and the non-finite scan of the ACCUMULATED values are taken on the way.
//
// HBM-bound: per element 2 bytes read + 4 written when overwriting, 6 read + 4 written
// when adding.  Work unit = 4 consecutive elements per lane: one 8-byte load on the tensor
// side, one 16-byte load and store on the chunk side, so that every wave instruction covers
// one contiguous span (512 B / 1 KiB); the body is aligned on the chunk side (16 bytes); a
// tensor side that is not congruent (8 bytes) is read with 8-byte loads at 2-byte alignment.
// Each element is one binary32 addition of the stored sum and the exactly decoded word.
#include "pt_common.h"

#include <hip/hip_fp16.h>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int AC_THREADS = 64;

template <int DT>
__device__ __forceinline__ float word_to_f32(uint32_t w16) {
  if (DT == PT_BF16) {
    return __uint_as_float(w16 << 16);
  } else {
    __half_raw r; r.x = (unsigned short)w16;
    return __half2float(__half(r));
  }
}

__device__ __forceinline__ void take(float a, double& sum) {
  const double x = (double)a;
  sum = fma(x, x, sum);
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// q: four 16-bit words; acc: the four sums they are added to (or that they replace)
template <int DT, bool OVERWRITE, bool NORM>
__device__ __forceinline__ void add4(const u32x2& q, f32x4& acc, double& a0, double& a1) {
  const float x[4] = {word_to_f32<DT>(q.x & 0xffffu), word_to_f32<DT>(q.x >> 16),
                      word_to_f32<DT>(q.y & 0xffffu), word_to_f32<DT>(q.y >> 16)};
#pragma unroll
  for (int k = 0; k < 4; ++k) acc[k] = OVERWRITE ? x[k] : acc[k] + x[k];
  if (NORM) {
    take(acc[0], a0); take(acc[1], a1);
    take(acc[2], a0); take(acc[3], a1);
  }
}

typedef u32x2 u32x2_a2 __attribute__((aligned(2)));   // global memory takes an 8-byte load at any address

template <bool ALIGNED>
__device__ __forceinline__ u32x2 load4(const PT_GLOBAL uint16_t* s) {
  if (ALIGNED) return __builtin_nontemporal_load((const PT_GLOBAL u32x2*)s);
  return __builtin_nontemporal_load((const PT_GLOBAL u32x2_a2*)s);
}

// KEEP: sums that stay in the Infinity Cache (pt_in_cache) are loaded without the hint.
template <bool KEEP> __device__ __forceinline__ f32x4 load_sums(const PT_GLOBAL f32x4* p) {
  if constexpr (KEEP) return *p;
  else return __builtin_nontemporal_load(p);
}

// nvec units of four elements from sb onto db: two per lane in flight.  NEAR: the sums are among the first that the cache can hold, and are
// stored so that they stay there (pt_store), also where they are not loaded so.
template <int DT, bool OVERWRITE, bool NORM, bool ALIGNED, bool KEEP, bool NEAR>
__device__ __forceinline__ void add_units(const PT_GLOBAL uint16_t* sb, PT_GLOBAL f32x4* db, uint32_t nvec, double& a0, double& a1) {
  constexpr int U = 2, POLICY = NEAR ? PT_THROUGH : PT_NT;
  uint32_t i = threadIdx.x;
  for (; i + (U - 1) * AC_THREADS < nvec; i += U * AC_THREADS) {
    u32x2 q[U];
    f32x4 a[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      q[r] = load4<ALIGNED>(sb + size_t(i + r * AC_THREADS) * 4);
      if (OVERWRITE) a[r] = f32x4{};
      else a[r] = load_sums<KEEP>(db + i + r * AC_THREADS);
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      add4<DT, OVERWRITE, NORM>(q[r], a[r], a0, a1);
      pt_store<POLICY>(a[r], db, (i + r * AC_THREADS) * 16);
    }
  }
  for (; i < nvec; i += AC_THREADS) {
    const u32x2 q = load4<ALIGNED>(sb + size_t(i) * 4);
    f32x4 a = {};
    if (!OVERWRITE) a = load_sums<KEEP>(db + i);
    add4<DT, OVERWRITE, NORM>(q, a, a0, a1);
    pt_store<POLICY>(a, db, i * 16);
  }
}

// As in pack: one wave adds 1024 elements, two units per lane in flight, and unused LDS (accum_lds) keeps 12 or 17 waves on a
// compute unit.  Adding 3.3e8 words: 521 us with workgroups of four waves and tiles of 4096
// taken from two ends of the list, 510 with three of those on a unit, 493 now (6.6 TB/s) - 507 with four units per lane in
// flight, 513 without the limit, 535-550 with 2048 elements per wave.
// 12 waves suit large sums; small ones, which the cache serves in part, and a first micro-batch that only writes its
// sums (6 bytes an element instead of 10), want 17.  With 12 and 17, four added and the update: 7e6 words 108.5 and 104.1 us, 1.5e7
// 199 and 189, 3e7 364 and 352, 6e7 696 and 683, 8.5e7 966 and 954, 1.24e8 1365 and 1360, 2.0e8 2302 and 2360, 3.3e8 3630 and 3720
// (four units a lane in flight with 12: 6e7 690, 2e6 44.4 -> 46.9); writing: 8e6 11.5 and 10.5, 3e7 33.9 and 30.5, 3.3e8 339 and 298;
// writing with the norm: 3e7 39.7 and 34.3, 3.3e8 401 and 326.  Four launches over 6.7e9 elements whose halves lie in different
// 96 GiB regions of the memory: 37.5 to 41.5 ms from process to process before, 38.6-38.9 now.
inline uint32_t accum_lds(bool overwrite, uint64_t elems) { return overwrite || elems < (1ull << 25) ? 9000 : 13000; }

template <int DT, bool OVERWRITE, bool NORM>
__global__ void __launch_bounds__(AC_THREADS)
k_accum(const PtTile* __restrict__ tiles, const uint64_t* __restrict__ chunk_row, uint32_t subs, uint32_t sub_elems,
        const PtDevState* __restrict__ st, double* __restrict__ tile_sq, uint32_t* __restrict__ tile_flag, uint64_t S, uint64_t cached, uint64_t near) {
  const uint32_t tile = blockIdx.x / subs;
  const PtTile t = tiles[tile];
  uint32_t lo, hi;
  pt_sub_range(t, blockIdx.x - tile * subs, sub_elems, lo, hi);
  PT_GLOBAL float* dst = (PT_GLOBAL float*)(chunk_row[t.chunk]) + t.chunk_off + lo;
  const PT_GLOBAL uint16_t* src = (const PT_GLOBAL uint16_t*)(t.tensor_addr) + lo;
  const uint32_t len = hi - lo;

  // elements before the chunk side reaches a 16-byte boundary
  uint32_t head = uint32_t(((16u - (uint32_t((uintptr_t)dst) & 15u)) & 15u) >> 2);
  if (head > len) head = len;
  const uint32_t nvec = (len - head) / 4;
  const uint32_t tail0 = head + nvec * 4;

  const double inv_scale = NORM ? 1.0 / st->loss_scale : 1.0;
  double a0 = 0.0, a1 = 0.0;

  const PT_GLOBAL uint16_t* sb = src + head;
  PT_GLOBAL f32x4* db = (PT_GLOBAL f32x4*)(dst + head);
  const bool aligned = ((uintptr_t)sb & 7u) == 0;
  if (!OVERWRITE && pt_in_cache(t.chunk, S, t.chunk_off, cached)) {
    if (aligned) add_units<DT, OVERWRITE, NORM, true, true, true>(sb, db, nvec, a0, a1);
    else add_units<DT, OVERWRITE, NORM, false, true, true>(sb, db, nvec, a0, a1);
  } else if (pt_in_cache(t.chunk, S, t.chunk_off, near)) {
    if (aligned) add_units<DT, OVERWRITE, NORM, true, false, true>(sb, db, nvec, a0, a1);
    else add_units<DT, OVERWRITE, NORM, false, false, true>(sb, db, nvec, a0, a1);
  } else {
    if (aligned) add_units<DT, OVERWRITE, NORM, true, false, false>(sb, db, nvec, a0, a1);
    else add_units<DT, OVERWRITE, NORM, false, false, false>(sb, db, nvec, a0, a1);
  }

  // head and tail: at most 3 elements each, one lane per element
  if (threadIdx.x < head) {
    const float x = word_to_f32<DT>(src[threadIdx.x]);
    const float a = OVERWRITE ? x : dst[threadIdx.x] + x;
    dst[threadIdx.x] = a;
    if (NORM) take(a, a0);
  }
  if (threadIdx.x < len - tail0) {
    const uint32_t e = tail0 + threadIdx.x;
    const float x = word_to_f32<DT>(src[e]);
    const float a = OVERWRITE ? x : dst[e] + x;
    dst[e] = a;
    if (NORM) take(a, a1);
  }

  if (NORM) {
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

typedef void (*accum_kernel_t)(const PtTile*, const uint64_t*, uint32_t, uint32_t, const PtDevState*, double*, uint32_t*, uint64_t, uint64_t, uint64_t);

template <int DT>
accum_kernel_t pick(bool overwrite, bool norm) {
  if (overwrite) return norm ? k_accum<DT, true, true> : k_accum<DT, true, false>;
  return norm ? k_accum<DT, false, true> : k_accum<DT, false, false>;
}

}  // namespace

extern "C" int pt_chunk_accum_grads(pt_ctx* ctx, const pt_pack_plan* plan, float* const* acc_chunks, int overwrite,
                                    int take_norm, void* stream) {
  if (!ctx) return PT_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (!plan || !acc_chunks) return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_accum_grads: NULL argument");
  if (plan->ctx != ctx) return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_accum_grads: plan belongs to another context");
  if (!ctx->grad_f32)
    return pt_fail(ctx, PT_ERR_STATE, "pt_chunk_accum_grads: the context holds 16-bit gradient chunks (set option grad_fp32)");
  if (take_norm) pt_capturing(ctx, st);
  int rc = pt_table_bind(ctx, ROW_PACK, 0, ctx->C, (const void* const*)acc_chunks, true, st);
  if (rc != PT_OK) return rc;
  if (plan->n_tiles == 0) return PT_OK;
  const uint64_t* h = ctx->h_table.data() + size_t(ROW_PACK) * ctx->table_cols;
  for (uint32_t c : plan->touched)
    if (!h[c]) return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_accum_grads: chunk %u is used by the plan but its pointer is NULL", c);
  if (take_norm && ((rc = pt_reopen_step(ctx, st)) != PT_OK || (rc = pt_before_partials(ctx, st)) != PT_OK)) return rc;
  accum_kernel_t kern = ctx->dtype == PT_BF16 ? pick<PT_BF16>(overwrite != 0, take_norm != 0)
                                              : pick<PT_FP16>(overwrite != 0, take_norm != 0);
  hipLaunchKernelGGL(kern, dim3(plan->n_tiles * plan->subs), dim3(AC_THREADS), accum_lds(overwrite != 0, plan->total_elems), st,
                     plan->d_tiles, pt_row(ctx, ROW_PACK), plan->subs, plan->sub_elems, ctx->d_state, plan->d_tile_sq,
                     plan->d_tile_flag, ctx->S, pt_cached_loads(ctx), pt_cached_elems(ctx));
  PT_LAUNCH_CHECK(ctx, "k_accum");
  if (take_norm) {
    rc = pt_reduce_plan(ctx, plan, st);
    if (rc != PT_OK) return rc;
    for (uint32_t c : plan->touched) ctx->chunk_fresh[c] = 1;
  }
  return PT_OK;
}
