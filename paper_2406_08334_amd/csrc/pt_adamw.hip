// Fused mixed-precision AdamW over chunks: one launch covers every chunk of a
// range through the context's device pointer table.
//
// HBM-bound: per element 14 bytes read (g16, w, m, v) and 14 written (w, m, v,
// p16); 16 read with fp32 gradient chunks, and 2 or 4 more written when the gradients are
// zeroed on the way out.  Work unit = 4 consecutive elements per lane: one 16-byte access per fp32
// array and one 8-byte access per 16-bit array, so that every wave instruction
// touches one contiguous 1 KiB (fp32) or 512 B (16-bit) span.  The launch shape keeps few bytes in
// flight, in address order (see k_adamw).
// Arithmetic: the fp32 operation sequence below with correctly rounded *, fma,
// sqrt and / (this file is compiled with contraction off and without fast-math).
#include "pt_common.h"
#include "pt_scalars.h"

#include <hip/hip_fp16.h>

#include <algorithm>

#pragma clang fp contract(off)

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// Chunk arrays are device (global) memory: typed as such so that loads and stores are
// global_* instructions instead of flat_* ones.
typedef PT_GLOBAL f32x4* gf32x4_ptr;
typedef PT_GLOBAL u32x2* gu32x2_ptr;
typedef const PT_GLOBAL f32x4* cgf32x4_ptr;
typedef const PT_GLOBAL u32x2* cgu32x2_ptr;

// NT: non-temporal hints (every byte is touched once per step).
template <bool NT, class P>
__device__ __forceinline__ auto ld_stream(P p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, class T, class P>
__device__ __forceinline__ void st_stream(T v, P p) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

template <int DT>
__device__ __forceinline__ float decode16(uint32_t w16) {
  if (DT == PT_BF16) {
    return __uint_as_float(w16 << 16);
  } else {
    __half_raw r; r.x = (unsigned short)w16;
    return __half2float(__half(r));
  }
}

template <int DT>
__device__ __forceinline__ uint32_t encode16(float x) {
  if (DT == PT_BF16) {
    const uint32_t u = __float_as_uint(x);
    const uint32_t nan = (u >> 16) | 0x0040u;                          // NaN stays NaN
    const uint32_t rne = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;       // round to nearest, ties to even
    return (u & 0x7fffffffu) > 0x7f800000u ? nan : rne;                // a select: a branch per element was compiled before
  } else {
    // The recast rounds the STORED fp32 master weight.  Without this barrier the compiler
    // folds the producing fma and the conversion into one mixed-precision fma that rounds
    // the exact result straight to fp16, which can differ from RNE16(RNE32(.)) by one ulp.
    asm volatile("" : "+v"(x));
    __half_raw r = __half_raw(__float2half_rn(x));
    return (uint32_t)r.x;
  }
}

struct Consts { float b1, b2, omb1, omb2, decay, step_size, rsb2, eps, gm; };

// Four gradient elements as they sit in a gradient chunk: four 16-bit words, or four floats
// when the chunk accumulates micro-batches in fp32.
template <bool GF32> struct GradUnit { typedef u32x2 vec; };
template <> struct GradUnit<true> { typedef f32x4 vec; };

template <int DT, bool GF32>
__device__ __forceinline__ void decode_unit(const typename GradUnit<GF32>::vec& q, float (&g)[4]) {
  if constexpr (GF32) {
    g[0] = q[0]; g[1] = q[1]; g[2] = q[2]; g[3] = q[3];
  } else {
    g[0] = decode16<DT>(q.x & 0xffffu); g[1] = decode16<DT>(q.x >> 16);
    g[2] = decode16<DT>(q.y & 0xffffu); g[3] = decode16<DT>(q.y >> 16);
  }
}

// dk: decay factor of each of the four elements (k.decay, or 1 for elements kept out of the decay)
template <int DT, bool GF32>
__device__ __forceinline__ void update_unit(const Consts& k, const float (&dk)[4],
                                            const typename GradUnit<GF32>::vec& gq, f32x4& w, f32x4& m,
                                            f32x4& v, u32x2& p2) {
  float gv[4];
  decode_unit<DT, GF32>(gq, gv);
  uint32_t pw[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    // one correctly rounded binary32 operation per line; contraction is off for this file
    float g = gv[j] * k.gm;
    float t1 = k.omb1 * g;
    float mn = __builtin_fmaf(k.b1, m[j], t1);
    float t2 = k.omb2 * g;
    t2 = t2 * g;
    float vn = __builtin_fmaf(k.b2, v[j], t2);
    float d = __builtin_fmaf(__builtin_sqrtf(vn), k.rsb2, k.eps);
    float u = mn / d;
    float t3 = w[j] * dk[j];
    float wn = __builtin_fmaf(-k.step_size, u, t3);
    m[j] = mn; v[j] = vn; w[j] = wn;
    pw[j] = encode16<DT>(wn);
  }
  p2.x = pw[0] | (pw[1] << 16);
  p2.y = pw[2] | (pw[3] << 16);
}

// blockIdx.y is the chunk (table column first_col + blockIdx.y), blockIdx.x the tile of TH x UNROLL units inside
// it; workgroups are dispatched in this order, so the traffic of a moment is one narrow window that slides over each
// array.  A grid smaller than the tiles (option adamw_grid, or a dimension beyond its limit) walks on from there.
//
// What bounds the launch is the memory's service time for four read and four write streams.  It grows with the bytes in
// flight and where all arrays fall into one of the memory's three regions of 96 GiB - what plain allocation gives a state
// of up to about 100 GB; DRAM rows that are opened too often would explain both, but no counter shows them.  What helps is
// few bytes in flight, in address order: workgroups of ONE wave, one unit per lane, and only 11 of them per compute unit
// (PT_ADAMW_LDS of unused LDS each; their loads together are 10 MB chip-wide at most) instead of 24 waves with four units
// each.  Counted over 6.8e9 elements: 26 700 reads of 128 bytes in flight instead of 30 200, each back after 2400 L2
// cycles instead of 3130.  Moving the same bytes without the arithmetic over 2^28 elements: all
// arrays in one region 5.4 -> 6.5 TB/s, spread over the regions 6.39 -> 6.55 TB/s.  The whole step of the GPT-2-XL
// shape (plain allocations): 9.35 -> 7.8 ms; 9 or 13 waves per unit 8.1 and 8.0 ms, 128 lanes 8.1, two units per lane
// 8.2, no limit on the waves 8.6 ms.
//
// Tiles start on a 128-byte line of the master array (the first one up to 7 units early, with those lanes idle), so
// that chunks whose size is no multiple of a line do not split every wave's lines between two workgroups
// (14 chunks of 5 000 200 elements: 428 -> 362 us a step).
//
// The loads are issued before the step's scalars are looked at: a skipped step reads in vain, every other one has its
// traffic under way while the scalars arrive.
//
// MASKED: some element ranges of some chunks are kept out of the weight decay (sorted,
// disjoint ranges per chunk: nd_begin[c] .. nd_begin[c+1] index pairs (lo, hi) in nd_ranges).
// A tile that no range touches, or that lies inside one range, runs the same vector path with
// one decay factor; only tiles cut by a range edge take the element-wise path.
//
// GF32: the gradient chunks hold fp32 (accumulated micro-batches) instead of 16-bit words.
// zero_grads: every gradient element is overwritten with zero once it has been read (for
// callers whose backward pass adds into the chunk); a skipped step zeroes them as well, so that the non-finite
// value that caused the skip does not stay in the sums.
// recast_on_skip: a chunk buffer of the streamed path is offloaded in full after a skipped step and its param16
// array was never uploaded, so it is refilled from the untouched master weights (param16 == RNE(master) is the
// invariant of every update).
constexpr uint32_t LINE_UNITS = 8;     // units of a 128-byte line of an fp32 array

// The five arrays of a chunk.  `back`: units from the start of the master array's 128-byte line to the chunk's start.
template <bool GF32>
struct ChunkPtrs {
  PT_GLOBAL typename GradUnit<GF32>::vec* g;
  gf32x4_ptr w, m, v;
  gu32x2_ptr p;
  uint32_t back;
};

template <bool GF32>
__device__ __forceinline__ ChunkPtrs<GF32> chunk_ptrs(uint64_t g, uint64_t w, uint64_t m, uint64_t v, uint64_t p) {
  return {(PT_GLOBAL typename GradUnit<GF32>::vec*)g, (gf32x4_ptr)w, (gf32x4_ptr)m, (gf32x4_ptr)v, (gu32x2_ptr)p,
          uint32_t(w >> 4) & (LINE_UNITS - 1)};
}

// The units of a tile in a lane's registers, if the tile is a whole one.
template <int UNROLL, bool GF32>
struct Tile {
  uint64_t ub;              // first unit; "negative" (wrapped around, above the chunk's units) for the idle lanes of the first tile
  bool full;
  typename GradUnit<GF32>::vec g[UNROLL];
  f32x4 w[UNROLL], m[UNROLL], v[UNROLL];
};

// Loads tile `tile` of a chunk.  NT: hints on the state; NTG: and on the gradient loads (host memory only: pt_adamw_hints).
template <int TH, int UNROLL, bool NT, bool NTG, bool GF32>
__device__ __forceinline__ void load_tile(Tile<UNROLL, GF32>& t, const ChunkPtrs<GF32>& x, uint64_t tile, uint64_t units) {
  constexpr uint32_t TILE_UNITS = TH * UNROLL;
  t.ub = tile * TILE_UNITS - x.back;
  t.full = t.ub < units && units - t.ub >= TILE_UNITS;
  if (t.full) {
#pragma unroll
    for (int r = 0; r < UNROLL; ++r) {
      const uint32_t o = threadIdx.x + uint32_t(r) * TH;
      t.g[r] = ld_stream<NTG>(x.g + t.ub + o);
      t.w[r] = ld_stream<NT>(x.w + t.ub + o);
      t.m[r] = ld_stream<NT>(x.m + t.ub + o);
      t.v[r] = ld_stream<NT>(x.v + t.ub + o);
    }
  }
  asm volatile("" ::: "memory");        // keeps the compiler from moving the loads behind a branch on the step's scalars
}

// Updates a tile that has been loaded.  HOST: of chunks in host memory.  c: the chunk's index in the no-decay ranges.  skip,
// recast_on_skip, zero_grads as above.
template <int TH, int DT, int UNROLL, bool NT, bool HOST, bool MASKED, bool GF32, class P32, class P64>
__device__ __forceinline__ void finish_tile(const Consts& k, int32_t skip, const ChunkPtrs<GF32>& x, Tile<UNROLL, GF32>& t, uint64_t units,
                                            uint32_t c, int recast_on_skip, int zero_grads, P32 nd_begin, P64 nd_ranges) {
  typedef typename GradUnit<GF32>::vec gvec;
  constexpr uint32_t TILE_UNITS = TH * UNROLL;
  constexpr int POLICY = !NT ? PT_PLAIN : HOST ? PT_NT : PT_NT_THROUGH;
  const gvec gzero = {};
  const uint64_t ub = t.ub;
  if (skip) {
    for (int r = 0; r < UNROLL; ++r) {
      const uint64_t u = ub + (threadIdx.x + uint32_t(r) * TH);
      if (u >= units) continue;
      if (recast_on_skip) {
        const f32x4 y = x.w[u];
        u32x2 p;
        p.x = encode16<DT>(y[0]) | (encode16<DT>(y[1]) << 16);
        p.y = encode16<DT>(y[2]) | (encode16<DT>(y[3]) << 16);
        x.p[u] = p;
      }
      if (zero_grads) st_stream<NT>(gzero, x.g + u);
    }
    return;
  }
  float dtile = k.decay;            // decay factor of the whole tile, when it has one
  bool cut = false;                 // a range edge falls inside this tile
  uint32_t r0 = 0, r1 = 0;          // ranges of this chunk from the first one that ends after the tile start
  if (MASKED) {
    r1 = nd_begin[c + 1];
    uint32_t lo = nd_begin[c], hi = r1;
    const uint64_t e0 = ub < units ? ub * 4 : 0, e1 = (ub + TILE_UNITS) * 4;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (nd_ranges[2 * size_t(mid) + 1] <= e0) lo = mid + 1; else hi = mid;
    }
    r0 = lo;
    if (r0 < r1 && nd_ranges[2 * size_t(r0)] < e1) {
      if (nd_ranges[2 * size_t(r0)] <= e0 && nd_ranges[2 * size_t(r0) + 1] >= e1) dtile = 1.0f;
      else cut = true;
    }
  }
  if (t.full && !(MASKED && cut)) {
    const float dk[4] = {dtile, dtile, dtile, dtile};
#pragma unroll
    for (int r = 0; r < UNROLL; ++r) {
      const uint32_t o = threadIdx.x + uint32_t(r) * TH;
      u32x2 p;
      update_unit<DT, GF32>(k, dk, t.g[r], t.w[r], t.m[r], t.v[r], p);
      pt_store<POLICY>(t.w[r], x.w + ub, 16 * o);
      pt_store<POLICY>(t.m[r], x.m + ub, 16 * o);
      pt_store<POLICY>(t.v[r], x.v + ub, 16 * o);
      pt_store<POLICY>(p, x.p + ub, 8 * o);
      if (zero_grads) pt_store<NT ? PT_THROUGH : PT_PLAIN>(gzero, x.g + ub, uint32_t(sizeof gzero) * o);
    }
    return;
  }
  // the first and the last tile of a chunk, and tiles with a range edge inside: unit by unit
  for (int r = 0; r < UNROLL; ++r) {
    const uint64_t u = ub + (threadIdx.x + uint32_t(r) * TH);
    if (u >= units) continue;
    float dk[4] = {dtile, dtile, dtile, dtile};
    if (MASKED && cut) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint64_t e = 4 * u + j;
        for (uint32_t q = r0; q < r1 && nd_ranges[2 * size_t(q)] <= e; ++q)
          if (e < nd_ranges[2 * size_t(q) + 1]) dk[j] = 1.0f;
      }
    }
    gvec g1 = x.g[u]; f32x4 w1 = x.w[u], m1 = x.m[u], v1 = x.v[u]; u32x2 p;
    update_unit<DT, GF32>(k, dk, g1, w1, m1, v1, p);
    x.w[u] = w1; x.m[u] = m1; x.v[u] = v1; x.p[u] = p;
    if (zero_grads) x.g[u] = gzero;
  }
}

template <int TH, int DT, int UNROLL, bool NT, bool NTG, bool MASKED, bool GF32>
__device__ __forceinline__ void update_tile(const Consts& k, int32_t skip, const ChunkPtrs<GF32>& x, uint64_t tile, uint64_t units,
                                            uint32_t c, int recast_on_skip, int zero_grads, const uint32_t* __restrict__ nd_begin,
                                            const uint64_t* __restrict__ nd_ranges) {
  Tile<UNROLL, GF32> t;
  load_tile<TH, UNROLL, NT, NTG, GF32>(t, x, tile, units);
  finish_tile<TH, DT, UNROLL, NT, NTG, MASKED, GF32>(k, skip, x, t, units, c, recast_on_skip, zero_grads, nd_begin, nd_ranges);
}

__device__ __forceinline__ Consts load_consts(const PtDevState* __restrict__ st) {
  Consts k;
  k.b1 = st->c[0]; k.b2 = st->c[1]; k.omb1 = st->c[2]; k.omb2 = st->c[3]; k.decay = st->c[4];
  k.step_size = st->c[5]; k.rsb2 = st->c[6]; k.eps = st->c[7]; k.gm = st->c[8];
  return k;
}

template <int TH, int DT, int UNROLL, bool NT, bool MASKED, bool GF32>
__global__ void __launch_bounds__(TH)
k_adamw(const uint64_t* __restrict__ table, const PtDevState* __restrict__ st, uint32_t table_cols, uint32_t first_col,
        uint32_t n_cols, uint32_t mask_chunk0, uint64_t units, uint64_t tiles, int recast_on_skip, int zero_grads,
        const uint32_t* __restrict__ nd_begin, const uint64_t* __restrict__ nd_ranges) {
  const int32_t skip = st->skip;
  const Consts k = load_consts(st);
  for (uint32_t ci = blockIdx.y; ci < n_cols; ci += gridDim.y) {
    const uint64_t* t = table + first_col + ci;
    const ChunkPtrs<GF32> x = chunk_ptrs<GF32>(t[size_t(ROW_GRAD) * table_cols], t[size_t(ROW_MASTER) * table_cols],
                                               t[size_t(ROW_M) * table_cols], t[size_t(ROW_V) * table_cols],
                                               t[size_t(ROW_P16) * table_cols]);
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x)
      update_tile<TH, DT, UNROLL, NT, false, MASKED, GF32>(k, skip, x, tile, units, mask_chunk0 + ci, recast_on_skip, zero_grads, nd_begin,
                                                  nd_ranges);
  }
}

// ---- the update that derives its own constants ---------------------------------------------------
//
// The update of every chunk of a context, with the step's scalar work (the sums of a small plan, the norm, the constants, the end of
// the step) done by its first workgroups while the others have their first loads under way: one launch instead of two.
//
// What workgroups hand each other goes past the caches word by word, each next to the number of the launch in one 8-byte store: whoever
// reads the number has the word, without an order between stores.  The first workgroup publishes the constants, FUSED_COPIES times, so
// that the 2800 waves that run by then do not all ask one line.  Those ask until they have all words; the workgroups behind the first FUSED_EARLY
// start after others have finished, hence after the words were published, and read them through the scalar cache (were they to find
// older ones, they would ask like the others).
//
// What it costs is latency, from the start of the kernel: state and constants that need no norm 1.3 us (the powers of beta 0.9 of it, while the
// sums are on their way), trees published 1.8 to 2.6, all sums 3.8, the words published 4.7 and seen 4.8 to 5.1; with sums that are there already
// seen at 3.5.  The first tiles have arrived at 0.7 to 1.5, so 2 to 3.5 us of the launch of 4.7 that it replaces stay, but the memory is
// busy from the first microsecond.  One wave that takes all trees of 3500 sums by itself is slower (the 7 M step 51.0 us instead of 48.2): that
// code runs once, so what counts is how much of it has to be fetched.  A step, with the scalar kernel in front and without: 0.8 M
// parameters 19.6 and 16.0 us, 3 M 31.6 and 29.9, 7 M 50.2 and 48.2, 1e7 81.3 and 79.1, 2.8e7 149 and 147, 4.5e7 231 and 225, 6.8e7
// 362 and 354, 1.24e8 615 and 605, 2e8 1062 and 1053.
//
// No wait is without an end and none depends on the order in which workgroups start: after `tries` looks, some milliseconds, a wave
// derives the constants by itself.  The state it needs is written by the first workgroup only when the published words have arrived; so if they
// are still not there when the state has been read, what was read is the state before the step's end.
// The workgroups that run by then take a tile more each, from the far end, and load it with their own: twice the bytes are under way while
// they wait.  3 M parameters 29.8 -> 29.0 us a step, 2.5 M 23.3 -> 21.7, 3.2 M 26.2 -> 24.7, 4.3 M 31.0 -> 29.3, 7 M 47.8 -> 46.9, 1.4e7 84.5 -> 83.8,
// from 6e7 on the same (a third one 0.5 to 1 % more up to there).  Below 6144 tiles, 1.57 M elements, the state of a few such steps
// lies in the Infinity Cache and little waits for it: 1.1 M 17.1 -> 17.3, 0.8 M in chunks of 2^18 13.9 -> 14.3, 1.4 M 18.3 -> 18.2, 1.9 M 20.7
// -> 19.7.  All tiles are counted through in one dimension of the grid for that.
constexpr uint32_t FUSED_EARLY = 4096, FUSED_RESIDENT = 256 * 11, FUSED_DOUBLED_FROM = 6144;

__device__ __forceinline__ double readlane_f64(double x, uint32_t lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}

__device__ __forceinline__ const PT_SCALAR PtFused& fused_work() {
  const PT_SCALAR FusedArgs* a = (const PT_SCALAR FusedArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));                    // loads are not moved in front of this
  return a->work;
}

// What the scalar work of a step leaves: the word of the lane (0-8: the constants, 9: skip), and what goes into the state.
struct Derived { uint32_t word; double sq, norm, clip, chunk; bool inf, has; };

// The tree `tree` of units 2 * pair and 2 * pair + 1, in lanes 0 to 31 and 32 to 63: in the order of the scalar kernel a lane's partial sums 512
// apart, then the tree over the 64 lanes.
struct Pair { double x[2][PT_REDUCE_SEG / PT_FUSED_ROW]; };
__device__ __forceinline__ void load_pair(Pair& p, const PT_SCALAR PtFused& a, uint32_t pair, uint32_t tree) {
#pragma unroll
  for (uint32_t u = 0; u < 2; ++u)
#pragma unroll
    for (uint32_t j = 0; j < PT_REDUCE_SEG / PT_FUSED_ROW; ++j) {
      // in bounds: no row begins behind the unit's sums, and a plan's have PT_FUSED_ROW more behind them
      const uint32_t row = a.lo[2 * pair + u] + j * PT_FUSED_ROW;
      p.x[u][j] = ((const PT_GLOBAL double*)a.part + (row < a.hi[2 * pair + u] ? row : 0))[tree * 64 + threadIdx.x];
    }
}
__device__ __forceinline__ double sum_pair(const Pair& p, const PT_SCALAR PtFused& a, uint32_t pair, uint32_t tree) {
  const uint32_t lane = threadIdx.x;
  double y[2] = {};
#pragma unroll
  for (uint32_t u = 0; u < 2; ++u)
#pragma unroll
    for (uint32_t j = 0; j < PT_REDUCE_SEG / PT_FUSED_ROW; ++j)
      y[u] += a.lo[2 * pair + u] + j * PT_FUSED_ROW + tree * 64 + lane < a.hi[2 * pair + u] ? p.x[u][j] : 0.0;
  const double keep = lane < 32 ? y[0] : y[1], send = lane < 32 ? y[1] : y[0];
  double t = keep + __shfl_xor(send, 32, 64);
#pragma unroll
  for (uint32_t off = 16; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
  return t;
}

// A tree's sum as it is published: two words.
__device__ __forceinline__ uint64_t* tree_words(const PT_SCALAR PtFused& a, uint32_t unit, uint32_t tree) {
  return a.pub + FUSED_COPIES * FUSED_LINE + (size_t(unit) * FUSED_TREES + tree) * 2;
}
__device__ __forceinline__ void publish_pair(const PT_SCALAR PtFused& a, uint32_t pair, uint32_t tree, double t) {
  const uint32_t half = threadIdx.x & 31;
  if (half < 2) st_agent(tree_words(a, 2 * pair + (threadIdx.x >> 5), tree) + half,
                         uint64_t(a.no) << 32 | uint32_t(half ? __double2hiint(t) : __double2loint(t)));
}

// ALONE: takes every tree itself instead of waiting for the workgroups that do.  Lane u has the sum of unit u.
template <bool ALONE>
__device__ __forceinline__ Derived derive(const PT_SCALAR PtFused& a) {
  const uint32_t lane = threadIdx.x;
  const int32_t step = ld_agent(&a.st->step);
  const double loss_scale = ld_agent(&a.st->loss_scale);
  double t = 0.0, acc = 0.0;
  uint32_t g = 0;
  if (lane < a.C) { t = ld_agent(a.chunk_sq + lane); g = ld_agent(a.chunk_flag + lane); }
  // what depends on the step counter alone, while the sums are on their way
  const double bc = 1.0 - pow(lane == 1 ? a.hp.beta2 : a.hp.beta1, double(step + 1));
  const pt_hparams hp = {a.hp.lr, a.hp.beta1, a.hp.beta2, a.hp.eps, a.hp.weight_decay, a.hp.max_norm};
  float c[9];
  pt_step_consts(c, hp, readlane_f64(bc, 0), readlane_f64(bc, 1));
  Derived d{};
  if (a.units) {
    // the units of chunk first + i, if that is the lane's
    uint32_t at = 0, begin = 0, count = 0, most = 0;
#pragma unroll
    for (uint32_t i = 0; i < FUSED_CHUNKS; ++i) {
      const uint32_t n = a.chunk_units[i];
      if (lane == a.first + i && i < a.n) { begin = at; count = n; }
      at += n;
      most = max(most, n);
    }
    const uint32_t unit = min(lane, a.units - 1);
    uint64_t lo[FUSED_TREES], hi[FUSED_TREES];
    bool alone = ALONE;
    for (uint32_t tries = ALONE ? 0 : a.tries;; --tries) {
      if (tries == 0) { alone = true; break; }
      bool all = true;
#pragma unroll
      for (uint32_t k = 0; k < FUSED_TREES; ++k) { lo[k] = ld_agent(tree_words(a, unit, k)); hi[k] = ld_agent(tree_words(a, unit, k) + 1); }
#pragma unroll
      for (uint32_t k = 0; k < FUSED_TREES; ++k)
        all = all && (k >= a.trees || (uint32_t(lo[k] >> 32) == a.no && uint32_t(hi[k] >> 32) == a.no));
      if (__all(all)) break;
    }
    if (!alone) {
#pragma unroll
      for (uint32_t k = 0; k < FUSED_TREES; ++k)
        acc = k < a.trees ? acc + __hiloint2double(uint32_t(hi[k]), uint32_t(lo[k])) : acc;
    } else {
      for (uint32_t p = 0; 2 * p < a.units; ++p) {
        double s = 0.0;
        for (uint32_t k = 0; k < a.trees; ++k) {
          Pair x;
          load_pair(x, a, p, k);
          s += sum_pair(x, a, p, k);
        }
        const double s0 = readlane_f64(s, 0), s1 = readlane_f64(s, 32);
        acc = lane == 2 * p ? s0 : lane == 2 * p + 1 ? s1 : acc;
      }
    }
    double mine = 0.0;
    for (uint32_t k = 0; k < most; ++k) {
      const double x = __shfl(acc, (begin + k) & 63, 64);
      if (k < count) mine += x;
    }
    d.has = count != 0;
    if (d.has) { t = mine; g = pt_not_finite(mine); }
  }
  d.chunk = t;
  bool inf = __any(g != 0);
  for (uint32_t k = 0; k < min(a.C, 64u); ++k) d.sq += readlane_f64(t, k);
  for (uint32_t base = 64; base < a.C; base += 64) {
    t = 0.0; g = 0;
    if (base + lane < a.C) { t = ld_agent(a.chunk_sq + base + lane); g = ld_agent(a.chunk_flag + base + lane); }
    inf = inf || __any(g != 0);
    for (uint32_t k = 0; k < min(a.C - base, 64u); ++k) d.sq += readlane_f64(t, k);
  }
  d.inf = inf;
  d.norm = sqrt(d.sq);
  c[8] = pt_grad_mult(d.clip, hp.max_norm, d.norm, loss_scale);
  const uint32_t w = lane & 15;
  d.word = inf ? 1u : 0u;
#pragma unroll
  for (uint32_t k = 0; k < 9; ++k) d.word = w == k ? __float_as_uint(c[k]) : d.word;
  return d;
}

__device__ __forceinline__ void publish(const PT_SCALAR PtFused& a, uint32_t word) {
  const uint32_t lane = threadIdx.x;
  if ((lane & 15) > 9) return;
#pragma unroll
  for (uint32_t k = 0; k < FUSED_COPIES; k += 4)
    st_agent(a.pub + size_t(k + (lane >> 4)) * FUSED_LINE + (lane & 15), uint64_t(a.no) << 32 | word);
}

// The published word of each lane, if all of them are there within `tries` looks.
__device__ __forceinline__ bool published(const uint64_t* pub, uint32_t no, uint32_t copy, uint32_t tries, uint32_t& word) {
  const uint64_t* p = pub + size_t(copy) * FUSED_LINE + min(threadIdx.x & 15, 9u);
  for (; tries > 0; --tries) {
    const uint64_t x = ld_agent(p);
    if (__all(uint32_t(x >> 32) == no)) { word = uint32_t(x); return true; }
    __builtin_amdgcn_s_sleep(1);
  }
  return false;
}

// What the scalar kernel writes besides the constants, with the published words arrived.  A wave that has given up reads the state, waits for
// what it reads, and looks for the words once more: if it has read anything from here, it finds them.
__device__ __forceinline__ void write_state(const PT_SCALAR PtFused& a, const Derived& d) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const uint32_t lane = threadIdx.x;
  if (d.has) { a.chunk_sq[lane] = d.chunk; a.chunk_flag[lane] = pt_not_finite(d.chunk); }
  if (lane < 9) a.st->c[lane] = __uint_as_float(d.word);
  if (lane != 0) return;
  PtDevState s = *a.st;
  s.override_active = 0;
  a.st->sqnorm = d.sq; a.st->norm = d.norm; a.st->clip_coef = d.clip;
  a.st->found_inf = d.inf; a.st->skip = d.inf; a.st->override_active = 0;
  pt_end_early(a.st, s, d.inf, a.end_step);
}

// Tile `at` of all chunks: its chunk, the tile within it, and the chunk's arrays.
template <bool GF32>
struct Place { uint32_t c, tile; ChunkPtrs<GF32> x; };
template <bool GF32>
__device__ __forceinline__ Place<GF32> place(const FusedArgs& a, uint32_t at) {
  Place<GF32> p;
  p.c = uint32_t((uint64_t(at) * a.inv_hi + (uint64_t(at) * a.inv_lo >> 32)) >> 26);      // at / tiles
  p.tile = at - p.c * a.tiles;
  const PT_SCALAR uint64_t* t = a.table;
  asm volatile("" : "+s"(t));                    // not moved in front of what comes before
  t += p.c;
  const uint32_t cols = a.table_cols;
  p.x = chunk_ptrs<GF32>(t[size_t(ROW_GRAD) * cols], t[size_t(ROW_MASTER) * cols], t[size_t(ROW_M) * cols], t[size_t(ROW_V) * cols],
                         t[size_t(ROW_P16) * cols]);
  return p;
}

template <int DT, bool MASKED, bool GF32>
__global__ void __launch_bounds__(64, 3) k_adamw_fused(const FusedArgs a) {
  const uint32_t at = blockIdx.x, copy = at % FUSED_COPIES;
  const bool first = at == 0, two = at < a.doubled;
  Derived d;
  uint32_t mine = 0, word[10];                   // word: the same in every lane
  if (__builtin_expect(at <= a.summers, 0)) {
    const PT_SCALAR PtFused& work = fused_work();
    if (first) {
      d = derive<false>(work);
      mine = d.word;
      publish(work, mine);
    } else {
      const uint32_t pair = (at - 1) / work.trees, tree = (at - 1) % work.trees;
      Pair p;
      load_pair(p, work, pair, tree);
      publish_pair(work, pair, tree, sum_pair(p, work, pair, tree));
    }
  }
  Tile<1, GF32> tile, tile2;
  Place<GF32> p = place<GF32>(a, at), p2;
  load_tile<64, 1, true, false, GF32>(tile, p.x, p.tile, a.units);
  if (two) {
    p2 = place<GF32>(a, a.total - 1 - at);
    load_tile<64, 1, true, false, GF32>(tile2, p2.x, p2.tile, a.units);
  }
  bool known = false;
  if (at >= FUSED_EARLY) {
    const PT_SCALAR uint64_t* w = (const PT_SCALAR uint64_t*)a.pub + copy * FUSED_LINE;
    asm volatile("" : "+s"(w));                  // behind the tile's loads, whose latency hides this one's
    known = true;
#pragma unroll
    for (uint32_t k = 0; k < 10; ++k) {
      const uint64_t q = w[k];
      word[k] = uint32_t(q);
      known = known && uint32_t(q >> 32) == a.no;
    }
  }
  if (!known) {
    if (!first && __builtin_expect(!published(a.pub, a.no, copy, fused_work().tries, mine), 0)) {
      mine = derive<true>(fused_work()).word;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // looked for when the state has been read: see write_state
      published(a.pub, a.no, copy, 1, mine);
      p = place<GF32>(a, at);                    // again: nothing is held meanwhile
      load_tile<64, 1, true, false, GF32>(tile, p.x, p.tile, a.units);
      if (two) {
        p2 = place<GF32>(a, a.total - 1 - at);
        load_tile<64, 1, true, false, GF32>(tile2, p2.x, p2.tile, a.units);
      }
    }
#pragma unroll
    for (uint32_t k = 0; k < 10; ++k) word[k] = __builtin_amdgcn_readlane(mine, k);
  }
  float c[9];
#pragma unroll
  for (uint32_t k = 0; k < 9; ++k) c[k] = __uint_as_float(word[k]);
  const Consts k = {c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8]};
  finish_tile<64, DT, 1, true, false, MASKED, GF32>(k, int32_t(word[9]), p.x, tile, a.units, p.c, 0, a.zero_grads, a.nd_begin, a.nd_ranges);
  if (__builtin_expect(two, 0))
    finish_tile<64, DT, 1, true, false, MASKED, GF32>(k, int32_t(word[9]), p2.x, tile2, a.units, p2.c, 0, a.zero_grads, a.nd_begin, a.nd_ranges);
  if (__builtin_expect(first, 0)) write_state(fused_work(), d);
}

// The update of chunks in pinned host memory, in place over the link: the kernel itself reads gradient, master, momentum
// and variance from the host's arrays and writes master, momentum, variance and param16 back.
//
// What bounds it is the link with both directions busy (14 bytes per element each way).  Both directions share it from the
// first microsecond to the last: no first upload and no last offload that run alone, and no event between streams that
// could share a hardware queue.  Requests in flight are kept to what covers the link's latency (64 waves with one unit per
// lane) because more of them queue up in front of everybody's HBM traffic, writes above all; and they all come from ONE
// XCD (workgroups are dealt round robin over the eight: only every eighth works), so that the queues of the other seven
// stay free.  If the dispatch order were another one, only that advantage would be lost.  Half of a 12-block model's chunks
// (seven of 2^23 elements): 8 workgroups 21.4 ms a step, 12: 17.0, 16: 16.7 (49 GB/s per direction), 20: 17.0.  The
// resident update of 6.4e8 elements beside it runs at 5.1 TB/s (beside the copy engines: 5.25, and those move 48 GB/s).
// Moving the bytes without the arithmetic, with a copy in HBM (6.6 TB/s by itself) beside it: 32 waves on one XCD 49.9 GB/s
// and 5.3 TB/s, 32 waves over all XCDs 49.4 and 3.7, 128 waves over all XCDs 49.2 and 0.95.
constexpr uint32_t HOST_TH = 256, HOST_GROUPS = 16, N_XCD = 8;

struct HostChunks { uint64_t at[PT_DIRECT_CHUNKS][5]; };     // g, master, m, v, param16 as the device addresses them

template <int DT, bool MASKED, bool GF32>
__global__ void __launch_bounds__(HOST_TH)
k_adamw_host(const HostChunks chunks, const PtDevState* __restrict__ st, uint32_t n_chunks, uint32_t mask_chunk0, uint64_t units,
             uint64_t tiles, const uint32_t* __restrict__ nd_begin, const uint64_t* __restrict__ nd_ranges) {
  if (blockIdx.x % N_XCD) return;
  const uint32_t groups = gridDim.x / N_XCD;
  const int32_t skip = st->skip;
  const Consts k = load_consts(st);
  uint64_t tile = blockIdx.x / N_XCD;          // the tiles of all chunks are dealt out as one sequence
  for (uint32_t ci = 0; ci < n_chunks; ++ci) {
    const uint64_t* a = chunks.at[ci];
    const ChunkPtrs<GF32> x = chunk_ptrs<GF32>(a[0], a[1], a[2], a[3], a[4]);
    for (; tile < tiles; tile += groups) {
      if (!skip) {
        update_tile<HOST_TH, DT, 1, true, true, MASKED, GF32>(k, 0, x, tile, units, mask_chunk0 + ci, 0, 0, nd_begin, nd_ranges);
        continue;
      }
      // a skipped step leaves param16 as the recast of the master weights, as the chunk buffers do
      const uint64_t u = tile * HOST_TH - x.back + threadIdx.x;
      if (u >= units) continue;
      const f32x4 y = x.w[u];
      u32x2 p;
      p.x = encode16<DT>(y[0]) | (encode16<DT>(y[1]) << 16);
      p.y = encode16<DT>(y[2]) | (encode16<DT>(y[3]) << 16);
      x.p[u] = p;
    }
    tile -= tiles;
  }
}

// Measurement aid: the update's memory access pattern with the arithmetic taken out.  Same tiles, same
// block-to-tile mapping, the same four loads and four stores per unit with the same hints; master,
// momentum and variance are stored back as loaded and param16 is re-derived from the master weight
// (which is what it holds already), so the state does not change.  What this kernel attains is what the
// memory system gives this mix of streams on this placement; the update runs within 2 % of it, on either side.
template <int TH, int DT, int UNROLL, bool NT>
__global__ void __launch_bounds__(TH)
k_adamw_pattern(const uint64_t* __restrict__ table, uint32_t table_cols, uint32_t first_col, uint32_t n_cols,
                uint64_t units, uint64_t tiles, uint32_t* __restrict__ sink) {
  constexpr uint32_t TILE_UNITS = TH * UNROLL;
  uint32_t keep = 0;
  for (uint32_t ci = blockIdx.y; ci < n_cols; ci += gridDim.y) {
    const uint32_t col = first_col + ci;
    const uint64_t wa = table[size_t(ROW_MASTER) * table_cols + col];
    cgu32x2_ptr gp = (cgu32x2_ptr)(table[size_t(ROW_GRAD) * table_cols + col]);
    gf32x4_ptr wp = (gf32x4_ptr)wa;
    gf32x4_ptr mp = (gf32x4_ptr)(table[size_t(ROW_M) * table_cols + col]);
    gf32x4_ptr vp = (gf32x4_ptr)(table[size_t(ROW_V) * table_cols + col]);
    gu32x2_ptr pp = (gu32x2_ptr)(table[size_t(ROW_P16) * table_cols + col]);
    const uint32_t back = uint32_t(wa >> 4) & (LINE_UNITS - 1);
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
      const uint64_t ub = tile * TILE_UNITS - back;
      if (!(ub < units && units - ub >= TILE_UNITS)) continue;      // first and last tiles are left out (a few KiB per chunk)
      u32x2 g[UNROLL]; f32x4 w[UNROLL], m[UNROLL], v[UNROLL];
#pragma unroll
      for (int r = 0; r < UNROLL; ++r) {
        const uint32_t o = threadIdx.x + uint32_t(r) * TH;
        g[r] = gp[ub + o];
        w[r] = ld_stream<NT>(wp + ub + o);
        m[r] = ld_stream<NT>(mp + ub + o);
        v[r] = ld_stream<NT>(vp + ub + o);
      }
#pragma unroll
      for (int r = 0; r < UNROLL; ++r) {
        const uint32_t o = threadIdx.x + uint32_t(r) * TH;
        // opaque to the optimiser, so that the stores of unchanged values are not dropped
        asm volatile("" : "+v"(w[r]), "+v"(m[r]), "+v"(v[r]));
        u32x2 p;
        p.x = encode16<DT>(w[r][0]) | (encode16<DT>(w[r][1]) << 16);
        p.y = encode16<DT>(w[r][2]) | (encode16<DT>(w[r][3]) << 16);
        keep ^= g[r].x ^ g[r].y;
        pt_store<NT ? PT_NT_THROUGH : PT_PLAIN>(w[r], wp + ub, 16 * o);
        pt_store<NT ? PT_NT_THROUGH : PT_PLAIN>(m[r], mp + ub, 16 * o);
        pt_store<NT ? PT_NT_THROUGH : PT_PLAIN>(v[r], vp + ub, 16 * o);
        pt_store<NT ? PT_NT_THROUGH : PT_PLAIN>(p, pp + ub, 8 * o);
      }
    }
  }
  if (keep == 0x9e3779b9u && sink) *sink = keep;      // keeps the gradient loads alive; practically never taken
}

typedef void (*adamw_kernel_t)(const uint64_t*, const PtDevState*, uint32_t, uint32_t, uint32_t, uint32_t, uint64_t, uint64_t,
                               int, int, const uint32_t*, const uint64_t*);
typedef void (*pattern_kernel_t)(const uint64_t*, uint32_t, uint32_t, uint32_t, uint64_t, uint64_t, uint32_t*);

// The instantiation for a launch shape: the library's own (64 lanes, one unit each), and what the options adamw_threads and
// adamw_unroll ask for.  The latter lose to the former at every size measured; they stay for the options.
template <int DT, bool NT, bool MASKED, bool GF32>
struct Kernels {
  template <int TH, int U> static adamw_kernel_t adamw() { return k_adamw<TH, DT, U, NT, MASKED, GF32>; }
  template <int TH> static adamw_kernel_t by_unroll(uint32_t u) {
    return u == 1 ? adamw<TH, 1>() : u == 2 ? adamw<TH, 2>() : u == 8 ? adamw<TH, 8>() : adamw<TH, 4>();
  }
  static adamw_kernel_t pick(const PtAdamwShape& s) {
    return s.threads == 64 ? adamw<64, 1>() : s.threads == 256 ? by_unroll<256>(s.unroll) : by_unroll<512>(s.unroll);
  }
};

template <int DT, bool NT>
adamw_kernel_t pick_flags(const PtAdamwShape& s, bool masked, bool gf32) {
  if (gf32) return masked ? Kernels<DT, NT, true, true>::pick(s) : Kernels<DT, NT, false, true>::pick(s);
  return masked ? Kernels<DT, NT, true, false>::pick(s) : Kernels<DT, NT, false, false>::pick(s);
}

template <int DT>
adamw_kernel_t pick_kernel(const PtAdamwShape& s, bool nt, bool masked, bool gf32) {
  return nt ? pick_flags<DT, true>(s, masked, gf32) : pick_flags<DT, false>(s, masked, gf32);
}

typedef void (*fused_kernel_t)(FusedArgs);
template <int DT>
fused_kernel_t pick_fused(bool masked, bool gf32) {
  if (gf32) return masked ? k_adamw_fused<DT, true, true> : k_adamw_fused<DT, false, true>;
  return masked ? k_adamw_fused<DT, true, false> : k_adamw_fused<DT, false, false>;
}

template <int TH, int DT, bool NT>
pattern_kernel_t pattern_by_unroll(uint32_t u) {
  return u == 1 ? k_adamw_pattern<TH, DT, 1, NT> : u == 2 ? k_adamw_pattern<TH, DT, 2, NT>
       : u == 8 ? k_adamw_pattern<TH, DT, 8, NT> : k_adamw_pattern<TH, DT, 4, NT>;
}

template <int DT, bool NT>
pattern_kernel_t pattern_by_shape(const PtAdamwShape& s) {
  return s.threads == 64 ? k_adamw_pattern<64, DT, 1, NT>
                         : s.threads == 256 ? pattern_by_unroll<256, DT, NT>(s.unroll) : pattern_by_unroll<512, DT, NT>(s.unroll);
}

template <int DT>
pattern_kernel_t pick_pattern(const PtAdamwShape& s, bool nt) {
  return nt ? pattern_by_shape<DT, true>(s) : pattern_by_shape<DT, false>(s);
}

// Tiles per chunk and grid of an update launch over n_cols chunks.
struct Geometry { uint64_t tiles; dim3 grid; };

Geometry geometry(const pt_ctx* ctx, const PtAdamwShape& s, uint32_t n_cols) {
  const uint64_t tile_units = uint64_t(s.threads) * s.unroll;
  Geometry g;
  g.tiles = (ctx->S / 4 + (LINE_UNITS - 1) + tile_units - 1) / tile_units;   // a chunk may start up to 7 units into its first tile
  uint64_t x = g.tiles, y = n_cols;
  if (ctx->opt_adamw_grid) {
    x = std::min<uint64_t>(x, ctx->opt_adamw_grid);
    y = std::min<uint64_t>(y, std::max<uint64_t>(1, ctx->opt_adamw_grid / x));
  }
  x = std::min<uint64_t>(x, 0xffffffffull / s.threads);       // a grid dimension holds fewer than 2^32 work items
  g.grid = dim3(uint32_t(x), uint32_t(std::min<uint64_t>(y, 65535)));
  return g;
}

// Whether the tiles of an update of all chunks in the library's shape can be counted through in one dimension of a grid (and `place`).
bool tiles_in_one_row(const pt_ctx* ctx) { return (ctx->S / 256 + 2) * ctx->C < (uint64_t(1) << 26); }

// Launches of more than 2^31 tiles of 8192 elements are refused (no memory holds them).
bool too_many_tiles(const pt_ctx* ctx, uint32_t n_cols) { return (ctx->S / 8192 + 1) * n_cols > 0x7fffffffull; }

}  // namespace

int pt_launch_adamw(pt_ctx* ctx, uint32_t first_col, uint32_t n_cols, hipStream_t stream, bool recast_on_skip,
                    uint32_t mask_chunk0, bool zero_grads, const PtFused* fused) {
  if (n_cols == 0) return PT_OK;
  if (too_many_tiles(ctx, n_cols))
    return pt_fail(ctx, PT_ERR_UNSUPPORTED, "update launch of %u chunks exceeds 2^31 tiles", n_cols);
  const PtAdamwShape shape = pt_adamw_shape(ctx, n_cols);
  const Geometry geo = geometry(ctx, shape, n_cols);
  const bool hints = pt_adamw_hints(ctx);
  const bool masked = ctx->d_nd_begin != nullptr;
  if (fused) {
    fused_kernel_t kern = ctx->dtype == PT_BF16 ? pick_fused<PT_BF16>(masked, ctx->grad_f32) : pick_fused<PT_FP16>(masked, ctx->grad_f32);
    const uint32_t total = uint32_t(geo.tiles * n_cols), doubled = total < FUSED_DOUBLED_FROM ? 0 : FUSED_RESIDENT;
    const uint64_t inv = (uint64_t(1) << 58) / geo.tiles + 1;
    const FusedArgs args{(const PT_SCALAR uint64_t*)ctx->d_table, ctx->table_cols, fused->no, ctx->S / 4, (const PT_SCALAR uint32_t*)ctx->d_nd_begin,
                         (const PT_SCALAR uint64_t*)ctx->d_nd_ranges, fused->pub, zero_grads ? 1 : 0, pt_fused_summers(*fused), uint32_t(geo.tiles),
                         total, doubled, uint32_t(inv), uint32_t(inv >> 32), *fused};
    hipLaunchKernelGGL(kern, dim3(total - doubled), dim3(shape.threads), shape.lds, stream, args);
    PT_LAUNCH_CHECK(ctx, "k_adamw_fused");
    return PT_OK;
  }
  adamw_kernel_t kern = ctx->dtype == PT_BF16 ? pick_kernel<PT_BF16>(shape, hints, masked, ctx->grad_f32)
                                              : pick_kernel<PT_FP16>(shape, hints, masked, ctx->grad_f32);
  hipLaunchKernelGGL(kern, geo.grid, dim3(shape.threads), shape.lds, stream, ctx->d_table, ctx->d_state, ctx->table_cols,
                     first_col, n_cols, mask_chunk0, ctx->S / 4, geo.tiles, recast_on_skip ? 1 : 0, zero_grads ? 1 : 0,
                     ctx->d_nd_begin, ctx->d_nd_ranges);
  PT_LAUNCH_CHECK(ctx, "k_adamw");
  return PT_OK;
}

int pt_launch_adamw_host(pt_ctx* ctx, const uint64_t (*at)[5], uint32_t n, hipStream_t stream, uint32_t mask_chunk0) {
  const bool masked = ctx->d_nd_begin != nullptr, gf32 = ctx->grad_f32;
  const uint64_t units = ctx->S / 4, tiles = (units + (LINE_UNITS - 1) + HOST_TH - 1) / HOST_TH;
  for (uint32_t i = 0; i < n; i += PT_DIRECT_CHUNKS) {
    HostChunks c{};
    const uint32_t k = std::min(n - i, PT_DIRECT_CHUNKS);
    std::memcpy(c.at, at + i, k * sizeof c.at[0]);
    auto kern = ctx->dtype == PT_BF16
        ? (masked ? (gf32 ? k_adamw_host<PT_BF16, true, true> : k_adamw_host<PT_BF16, true, false>)
                  : (gf32 ? k_adamw_host<PT_BF16, false, true> : k_adamw_host<PT_BF16, false, false>))
        : (masked ? (gf32 ? k_adamw_host<PT_FP16, true, true> : k_adamw_host<PT_FP16, true, false>)
                  : (gf32 ? k_adamw_host<PT_FP16, false, true> : k_adamw_host<PT_FP16, false, false>));
    hipLaunchKernelGGL(kern, dim3(HOST_GROUPS * N_XCD), dim3(HOST_TH), 0, stream, c, ctx->d_state, k, mask_chunk0 + i, units, tiles,
                       ctx->d_nd_begin, ctx->d_nd_ranges);
    PT_LAUNCH_CHECK(ctx, "k_adamw_host");
  }
  return PT_OK;
}

extern "C" int pt_chunk_adamw_step(pt_ctx* ctx, const pt_hparams* hp, uint32_t first_chunk, uint32_t n_chunks,
                                   const void* const* grad, float* const* master, float* const* m,
                                   float* const* v, void* const* param16, void* stream) {
  if (!ctx) return PT_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (!hp) return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_adamw_step: hp is NULL");
  if (uint64_t(first_chunk) + n_chunks > ctx->C)
    return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_adamw_step: chunks [%u, %u) outside the context's %u chunks",
                   first_chunk, first_chunk + n_chunks, ctx->C);
  if (n_chunks && (!grad || !master || !m || !v || !param16))
    return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_chunk_adamw_step: NULL pointer array");
  if (!ctx->norm_finalized)
    return pt_fail(ctx, PT_ERR_STATE, "pt_chunk_adamw_step: no finalized gradient norm in this step");
  if (n_chunks == 0) return PT_OK;
  pt_capturing(ctx, st);
  int rc;
  const PtBind binds[5] = {{ROW_GRAD, grad}, {ROW_MASTER, (const void* const*)master}, {ROW_M, (const void* const*)m},
                           {ROW_V, (const void* const*)v}, {ROW_P16, (const void* const*)param16}};
  if ((rc = pt_table_bind(ctx, binds, 5, first_chunk, n_chunks, false, st)) != PT_OK) return rc;
  PtFused fused;
  if (n_chunks == ctx->C && tiles_in_one_row(ctx) && pt_fuse_scalars(ctx, hp, &fused)) {
    if ((rc = pt_launch_adamw(ctx, 0, n_chunks, st, false, 0, ctx->opt_zero_grads != 0, &fused)) == PT_OK) pt_fused_launched(ctx, fused);
    return rc;
  }
  if ((rc = pt_prepare_consts(ctx, hp, n_chunks < ctx->C, st)) != PT_OK) return rc;
  return pt_launch_adamw(ctx, first_chunk, n_chunks, st, false, first_chunk, ctx->opt_zero_grads != 0);
}

extern "C" int pt_calib_adamw_pattern(pt_ctx* ctx, uint32_t first_chunk, uint32_t n_chunks, void* stream) {
  if (!ctx) return PT_ERR_INVALID_ARG;
  if (uint64_t(first_chunk) + n_chunks > ctx->C)
    return pt_fail(ctx, PT_ERR_INVALID_ARG, "pt_calib_adamw_pattern: chunks [%u, %u) outside the context's %u chunks",
                   first_chunk, first_chunk + n_chunks, ctx->C);
  if (ctx->grad_f32 || ctx->d_nd_begin)
    return pt_fail(ctx, PT_ERR_UNSUPPORTED, "pt_calib_adamw_pattern: 16-bit gradient chunks without no-decay runs only");
  const uint64_t* h = ctx->h_table.data();
  for (uint32_t c = first_chunk; c < first_chunk + n_chunks; ++c)
    for (int row : {ROW_GRAD, ROW_MASTER, ROW_M, ROW_V, ROW_P16})
      if (!h[size_t(row) * ctx->table_cols + c])
        return pt_fail(ctx, PT_ERR_STATE, "pt_calib_adamw_pattern: chunk %u has not been through pt_chunk_adamw_step yet "
                       "(its pointers are not in the context's table)", c);
  if (n_chunks == 0) return PT_OK;
  if (too_many_tiles(ctx, n_chunks)) return pt_fail(ctx, PT_ERR_UNSUPPORTED, "pt_calib_adamw_pattern: more than 2^31 tiles");
  const PtAdamwShape shape = pt_adamw_shape(ctx, n_chunks);
  const Geometry geo = geometry(ctx, shape, n_chunks);
  const bool hints = pt_adamw_hints(ctx);
  pattern_kernel_t kern = ctx->dtype == PT_BF16 ? pick_pattern<PT_BF16>(shape, hints) : pick_pattern<PT_FP16>(shape, hints);
  hipLaunchKernelGGL(kern, geo.grid, dim3(shape.threads), shape.lds, (hipStream_t)stream, ctx->d_table, ctx->table_cols,
                     first_chunk, n_chunks, ctx->S / 4, geo.tiles, (uint32_t*)nullptr);
  PT_LAUNCH_CHECK(ctx, "k_adamw_pattern");
  return PT_OK;
}
