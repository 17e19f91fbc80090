// What the library asks of the HIP runtime, call by call, on a stand-in for it (fake_hip.h): no GPU, nothing runs.
// Usage: host_calls <check>.  Exit code 0 = the check held.
#include "fake_hip.h"

#include <memory>
#include <random>
#include <tuple>

#include "pt_step.h"
#include "ptchunk.h"

#define EXPECT(cond)                                                                                     \
  do {                                                                                                   \
    if (!(cond)) {                                                                                       \
      fprintf(stderr, "%s:%d: check failed: %s\ncalls:\n%s", __FILE__, __LINE__, #cond, fake::text().c_str()); \
      return 1;                                                                                          \
    }                                                                                                    \
  } while (0)
#define OK(call) EXPECT((call) == PT_OK)

namespace {

const pt_hparams HP = {1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0};

// Launches that take scalar work: of the scalar kernel, and of an update that does it itself.
std::vector<fake::Op> scalars(size_t from) {
  std::vector<fake::Op> v = fake::launches("k_scalars", from);
  for (const fake::Op& o : fake::launches("k_adamw_fused", from)) v.push_back(o);
  return v;
}

// C chunks of S elements in device memory and a context for them; the plan's tensors are the chunks themselves, one each.
struct State {
  uint64_t S;
  uint32_t C;
  pt_ctx* ctx = nullptr;
  std::vector<void*> g, p;
  std::vector<float*> w, m, v;
  std::vector<pt_pack_plan*> plans;

  State(uint32_t n, uint64_t elems, bool fp32 = false, const pt_scaler_cfg* scaler = nullptr) : S(elems), C(n) {
    if (pt_ctx_create(&ctx, PT_BF16, S, C, scaler) != PT_OK || (fp32 && pt_ctx_set_option(ctx, "grad_fp32", 1) != PT_OK)) die(nullptr);
    for (uint32_t c = 0; c < C; ++c) {
      g.push_back(device(4 * S)); p.push_back(device(2 * S));
      w.push_back((float*)device(4 * S)); m.push_back((float*)device(4 * S)); v.push_back((float*)device(4 * S));
    }
  }
  ~State() {
    for (pt_pack_plan* q : plans) pt_pack_plan_destroy(q);
    pt_ctx_destroy(ctx);
  }
  static void die(const pt_ctx* c) { fprintf(stderr, "setup failed: %s\n", pt_last_error(c)); exit(3); }
  static void* device(size_t n) { void* q = nullptr; (void)hipMalloc(&q, n); return q; }
  static void* pinned(size_t n) { void* q = nullptr; (void)hipHostMalloc(&q, n, 0); return q; }
  pt_pack_plan* plan(int only = -1) {
    std::vector<pt_segment> segs;
    for (uint32_t c = 0; c < C; ++c) if (only < 0 || uint32_t(only) == c) segs.push_back({device(2 * S), 0, S, 0, c, c});
    pt_pack_plan* q = nullptr;
    if (pt_pack_plan_create(ctx, segs.data(), uint32_t(segs.size()), &q) != PT_OK) die(ctx);
    plans.push_back(q);
    return q;
  }
  int pack(pt_pack_plan* q, hipStream_t s = nullptr) { return pt_chunk_pack_grads(ctx, q, g.data(), s); }
  int accum(pt_pack_plan* q, hipStream_t s = nullptr) { return pt_chunk_accum_grads(ctx, q, (float* const*)g.data(), 0, 1, s); }
  int finalize(int how, hipStream_t s = nullptr) { return pt_chunk_grad_sqnorm(ctx, nullptr, 0, C, how, s); }
  int update(hipStream_t s = nullptr) { return update(0, C, s); }
  int update(uint32_t first, uint32_t n, hipStream_t s = nullptr) {
    return pt_chunk_adamw_step(ctx, &HP, first, n, g.data() + first, w.data() + first, m.data() + first, v.data() + first,
                               p.data() + first, s);
  }
  // one eager step, after which every pointer is known to the device
  int step(pt_pack_plan* q) {
    int rc = pack(q);
    if (rc == PT_OK) rc = finalize(PT_FINALIZE_STRICT);
    if (rc == PT_OK) rc = update();
    if (rc == PT_OK) rc = pt_step_end(ctx, nullptr);
    return rc;
  }
};

// A graph of norm, update and step end that is captured without the pack - before one or behind an eager one - holds no
// reduction, and an eager pack of a plan beyond the fused sizes (8 chunks) has launched its own: replays see the sums of
// the pack in front of them, whichever plan it was.
int captured_without_the_pack() {
  State s(9, 4096);
  pt_pack_plan* q = s.plan();
  OK(s.step(q));
  const hipStream_t cap = fake::stream(0xc0);
  for (int pending = 0; pending < 2; ++pending) {
    size_t at = fake::ops.size();
    if (pending) {
      OK(s.pack(q));
      EXPECT(fake::launches("k_scalars", at).size() == 1);
    }
    at = fake::ops.size();
    fake::capturing[0xc0] = true;
    OK(s.finalize(PT_FINALIZE_CARRY, cap));
    OK(s.update(cap));
    OK(pt_step_end(s.ctx, cap));
    fake::capturing[0xc0] = false;
    const auto in_graph = fake::launches("k_scalars", at);
    EXPECT(in_graph.size() == 1 && in_graph[0].grid.x == 1 && in_graph[0].grid.y == 1);
  }
  // eager packs between the replays
  for (int k = 0; k < 3; ++k) {
    const size_t at = fake::ops.size();
    OK(s.pack(s.plan()));
    const auto red = fake::launches("k_scalars", at);
    EXPECT(red.size() == 1 && red[0].grid.y == 9);
    OK(pt_step_end(s.ctx, nullptr));
  }
  // recomputed from the chunks
  const size_t at = fake::ops.size();
  OK(pt_chunk_grad_sqnorm(s.ctx, s.g.data(), 0, 9, 0, nullptr));
  EXPECT(fake::launches("k_scalars", at).size() == 1);
  return 0;
}

// Sums that are put off don't pile up: two plans taken in turn leave one reduction to the call that needs the norm.
int put_off_at_most_once() {
  State s(2, 4096, true);
  pt_pack_plan *a = s.plan(), *b = s.plan();
  for (int k = 0; k < 50; ++k) { OK(s.accum(a)); OK(s.accum(b)); }
  const size_t at = fake::ops.size();
  OK(s.finalize(PT_FINALIZE_STRICT));
  OK(s.update());
  EXPECT(scalars(at).size() == 1);
  return 0;
}

// A finalize that waits runs on the stream of the call that needs it out of the way: the stream it was asked for on may be
// gone by then.
int finalize_on_a_stream_that_is_gone() {
  State s(2, 4096);
  pt_pack_plan* q = s.plan();
  OK(s.step(q));
  for (int how = 0; how < 3; ++how) {
    OK(s.pack(q, fake::stream(0xa0)));
    OK(s.finalize(PT_FINALIZE_STRICT, fake::stream(0xa0)));
    const size_t at = fake::ops.size();
    if (how == 0) OK(s.pack(q, fake::stream(0xb0)));
    if (how == 1) OK(pt_chunk_grad_sqnorm(s.ctx, s.g.data(), 0, 2, 0, fake::stream(0xb0)));
    if (how == 2) OK(s.update(fake::stream(0xb0)));
    EXPECT(fake::ops.size() > at && scalars(at).size() >= 1);
    for (size_t i = at; i < fake::ops.size(); ++i) EXPECT(fake::ops[i].stream != 0xa0);
    // the waiting norm comes first
    EXPECT(fake::ops[at].what == "launch" && fake::ops[at].kernel == (how == 2 ? "k_adamw_fused" : "k_scalars"));
    OK(pt_step_end(s.ctx, fake::stream(0xb0)));
  }
  return 0;
}

// Chunks [first, C) of a state in pinned host memory, one allocation per array.
struct HostPart {
  std::vector<void*> g, p;
  std::vector<float*> w, m, v;
  uint32_t first;
  HostPart(const State& s, uint32_t from) : first(from) {
    for (uint32_t c = from; c < s.C; ++c) {
      g.push_back(State::pinned(2 * s.S)); p.push_back(State::pinned(2 * s.S));
      w.push_back((float*)State::pinned(4 * s.S)); m.push_back((float*)State::pinned(4 * s.S)); v.push_back((float*)State::pinned(4 * s.S));
    }
  }
  int stream(State& s, hipStream_t st = nullptr) {
    return pt_chunk_stream_step(s.ctx, &HP, first, uint32_t(g.size()), g.data(), w.data(), m.data(), v.data(), p.data(), st);
  }
};

// More host chunks than one launch takes, and a later launch that fails: the step's end still waits for the earlier one.
int failed_launch_in_place() {
  State s(40, 4096);
  HostPart h(s, 0);
  OK(pt_stream_reserve(s.ctx, 2));
  OK(pt_step_override(s.ctx, 1.0f, 0, nullptr));
  const size_t at = fake::ops.size();
  fake::fail_kernel = "k_adamw_host";
  fake::fail_after = 1;
  EXPECT(h.stream(s) == PT_ERR_HIP);
  fake::fail_after = -1;
  const auto run = fake::launches("k_adamw_host", at);
  EXPECT(run.size() == 1);
  OK(pt_step_end(s.ctx, fake::stream(0xa0)));
  uintptr_t behind = 0;                          // the last event behind that launch
  for (size_t i = at; i < fake::ops.size(); ++i)
    if (fake::ops[i].what == "record" && fake::ops[i].stream == run[0].stream) behind = fake::ops[i].event;
  bool waits = false;
  for (size_t i = at; i < fake::ops.size(); ++i)
    waits = waits || (behind && fake::ops[i].what == "wait" && fake::ops[i].stream == 0xa0 && fake::ops[i].event == behind);
  EXPECT(waits);
  return 0;
}

// In place only where no array that is written overlaps another one: the copies go in a fixed order (of two chunks with one
// parameter array the later one's words stay), waves of one launch do not.
int overlapping_host_arrays() {
  enum { APART, OWN_GRADIENT, ONE_GRADIENT, ONE_PARAM, NEXT_GRADIENT, OVERLAPPED_PARAM, ONE_MOMENT, N };
  for (int how = 0; how < N; ++how) {
    State s(3, 4096);
    HostPart h(s, 0);
    OK(pt_stream_reserve(s.ctx, 2));
    if (how == OWN_GRADIENT) h.p = h.g;
    if (how == ONE_GRADIENT) h.g[2] = h.g[0];                                   // only read
    if (how == ONE_PARAM) h.p[2] = h.p[0];
    if (how == NEXT_GRADIENT) h.p[0] = h.g[1];
    if (how == OVERLAPPED_PARAM) { h.p[0] = State::pinned(4 * 4096); h.p[1] = (char*)h.p[0] + 4096; }
    if (how == ONE_MOMENT) h.v[1] = h.m[1];
    OK(pt_step_override(s.ctx, 1.0f, 0, nullptr));
    const size_t at = fake::ops.size();
    OK(h.stream(s));
    const bool in_place = how <= ONE_GRADIENT;
    EXPECT(fake::launches("k_adamw_host", at).size() == (in_place ? 1u : 0u));
    EXPECT(fake::launches("k_adamw", at).size() == (in_place ? 0u : 3u));
    OK(pt_step_end(s.ctx, nullptr));
  }
  return 0;
}

// The host-side update waits for an event behind the step's scalar kernel and in front of the resident update that was
// queued before it - from a context's first host-side call on, with chunk buffers reserved or without.
int host_update_beside_the_resident_one() {
  for (int buffers = 0; buffers < 2; ++buffers) {
    State s(3, 4096);
    HostPart h(s, 2);
    if (buffers) OK(pt_stream_reserve(s.ctx, 2));
    pt_pack_plan* q = s.plan();
    for (int step = 0; step < 2; ++step) {
      OK(s.pack(q));
      OK(s.finalize(PT_FINALIZE_STRICT));
      const size_t at = fake::ops.size();
      OK(s.update(0, 2));
      OK(pt_chunk_host_adamw_step(s.ctx, &HP, 2, 1, h.g.data(), h.w.data(), h.m.data(), h.v.data(), h.p.data(), 2, nullptr));
      size_t event = 0, update = 0;
      uintptr_t waited = 0;
      for (size_t i = at; i < fake::ops.size(); ++i) {
        if (fake::ops[i].what == "launch" && fake::ops[i].kernel == "k_adamw") update = i;
        if (fake::ops[i].what == "sync event") waited = fake::ops[i].event;
      }
      for (size_t i = at; i < fake::ops.size(); ++i)
        if (fake::ops[i].what == "record" && fake::ops[i].event == waited) event = i;
      EXPECT(waited && event && update && event < update);
      OK(pt_step_end(s.ctx, nullptr));
    }
  }
  // and a step that updates every chunk on the device records no event
  State s(3, 4096);
  pt_pack_plan* q = s.plan();
  const size_t at = fake::ops.size();
  OK(s.step(q));
  for (size_t i = at; i < fake::ops.size(); ++i) EXPECT(fake::ops[i].what != "record");
  return 0;
}

// The norm holds its workgroups to four a compute unit (1024 at once) from 1792 of them on, with fp32 chunks from 4096:
// smaller arenas are read faster, or as fast, by eight.
int norm_occupancy_by_size() {
  for (const auto& [blocks, limited] : {std::pair{1u, false}, {1024u, false}, {1025u, false}, {1791u, false}, {1792u, true}, {4000u, true}}) {
    void* g = State::device(16);
    double out[2];
    int32_t inf;
    size_t at = fake::ops.size();
    OK(pt_chunk_grad_sqnorm_noalloc(g, PT_BF16, 32768, blocks, 1.0, out, &inf, nullptr));
    auto run = fake::launches("k_sqnorm_arena", at);
    EXPECT(run.size() == 1 && run[0].grid.x * run[0].grid.y == blocks && (run[0].lds != 0) == limited);
  }
  const void* at16[4096];
  for (const void*& q : at16) q = State::device(16);
  for (const auto& [blocks, fp32, limited] : {std::tuple{1791u, false, false}, {1792u, false, true}, {4095u, true, false}, {4096u, true, true}}) {
    pt_ctx* ctx = nullptr;
    OK(pt_ctx_create(&ctx, PT_FP16, 32768, blocks, nullptr));
    OK(pt_ctx_set_option(ctx, "grad_fp32", fp32));
    const size_t at = fake::ops.size();
    OK(pt_chunk_grad_sqnorm(ctx, at16, 0, blocks, 0, nullptr));
    const auto run = fake::launches(fp32 ? "k_sqnorm_f32" : "k_sqnorm", at);
    EXPECT(run.size() == 1 && (run[0].lds != 0) == limited);
    OK(pt_ctx_destroy(ctx));
  }
  return 0;
}

// A context and a plan of n elements in one chunk; the pointers are only looked at.
struct OnePlan {
  pt_ctx* ctx = nullptr;
  pt_pack_plan* q = nullptr;
  void* at = nullptr;
  OnePlan(uint64_t n, bool fp32 = false) {
    at = State::device(16);
    const pt_segment seg = {at, 0, n, 0, 0, 0};
    if (pt_ctx_create(&ctx, PT_BF16, (n + 7) / 8 * 8, 1, nullptr) != PT_OK || pt_ctx_set_option(ctx, "grad_fp32", fp32) != PT_OK ||
        pt_pack_plan_create(ctx, &seg, 1, &q) != PT_OK)
      State::die(ctx);
  }
  ~OnePlan() {
    pt_pack_plan_destroy(q);
    pt_ctx_destroy(ctx);
  }
};

// Unpack holds fewer waves on a compute unit the larger the plan is: lines at 2^24 and 2^28 elements.
int unpack_occupancy_by_size() {
  for (const auto& [n, lds] : {std::pair{(1ull << 24) - 1, size_t(0)}, {1ull << 24, 9000}, {(1ull << 28) - 1, 9000}, {1ull << 28, 11500}}) {
    OnePlan p(n);
    const size_t at = fake::ops.size();
    OK(pt_chunk_unpack(p.ctx, p.q, &p.at, nullptr));
    EXPECT(fake::launches("k_pack", at).size() == 1 && fake::launches("k_pack", at)[0].lds == lds);
  }
  return 0;
}

// Adding to sums holds fewer waves on a compute unit from 2^25 elements on; writing them never does.
int accumulate_occupancy_by_size() {
  for (const auto& [n, overwrite, lds] : {std::tuple{(1ull << 25) - 1, 0, 9000u}, {1ull << 25, 0, 13000u}, {1ull << 25, 1, 9000u}}) {
    OnePlan p(n, true);
    const size_t at = fake::ops.size();
    float* acc = (float*)p.at;
    OK(pt_chunk_accum_grads(p.ctx, p.q, &acc, overwrite, 0, nullptr));
    EXPECT(fake::launches("k_accum", at).size() == 1 && fake::launches("k_accum", at)[0].lds == lds);
  }
  return 0;
}

// The launch-shape options go back to the default shape.
int launch_shape_options_and_back() {
  State s(2, 4096);
  pt_pack_plan* q = s.plan();
  OK(s.step(q));
  const auto shape = [&] {                         // of the last update
    size_t i = fake::ops.size();
    while (fake::ops[--i].kernel.rfind("k_adamw", 0) != 0) {}
    return fake::ops[i];
  };
  const fake::Op own = shape();
  for (const char* name : {"adamw_unroll", "adamw_threads", "adamw_grid"}) {
    OK(pt_ctx_set_option(s.ctx, name, strcmp(name, "adamw_unroll") == 0 ? 4 : strcmp(name, "adamw_threads") == 0 ? 256 : 1));
    OK(s.step(q));
    EXPECT(shape().block.x != own.block.x || shape().grid.x != own.grid.x);
    OK(pt_ctx_set_option(s.ctx, name, 0));
    OK(s.step(q));
    EXPECT(shape().block.x == own.block.x && shape().grid.x == own.grid.x && shape().grid.y == own.grid.y && shape().lds == own.lds);
  }
  EXPECT(pt_ctx_set_option(s.ctx, "adamw_unroll", 3) == PT_ERR_INVALID_ARG);
  return 0;
}

// A plan whose waiting sums cannot be reduced any more takes them with it: its arrays are gone, nothing may read them, and
// the chunks have no value from this step.
int plan_destroyed_and_its_reduction_fails() {
  for (int finalized = 0; finalized < 2; ++finalized) {
    State s(2, 4096);
    pt_pack_plan* q = s.plan();
    OK(s.step(q));
    OK(s.pack(q));
    if (finalized) OK(s.finalize(PT_FINALIZE_STRICT));
    fake::fail_kernel = "k_scalars";
    fake::fail_after = 0;
    (void)pt_pack_plan_destroy(q);
    s.plans.clear();
    fake::fail_after = -1;
    const size_t at = fake::ops.size();
    if (finalized) EXPECT(s.update() == PT_ERR_STATE);
    else EXPECT(s.finalize(PT_FINALIZE_STRICT) == PT_ERR_STATE);
    OK(pt_step_end(s.ctx, nullptr));
    for (const fake::Op& o : fake::launches("k_scalars", at)) EXPECT(o.grid.x == 1 && o.grid.y == 1);
    OK(s.step(s.plan()));
  }
  return 0;
}

// Only steps through the chunk buffers are looked at for copy streams that got in each other's way; the option that sends
// every step there, or none.
int side_streams_are_judged_by_their_own_steps() {
  State s(2, 1 << 21);                            // chunk buffers large enough to try the copy streams out
  HostPart h(s, 0);
  OK(pt_stream_reserve(s.ctx, 2));
  OK(pt_ctx_set_option(s.ctx, "stream_test_unhealthy", 1));
  const auto step = [&](int in_place) {
    int rc = pt_ctx_set_option(s.ctx, "stream_in_place", in_place);
    if (rc == PT_OK) rc = pt_step_override(s.ctx, 1.0f, 0, nullptr);
    if (rc == PT_OK) rc = h.stream(s);
    return rc == PT_OK ? pt_step_end(s.ctx, nullptr) : rc;
  };
  int32_t rebuilds = -1;
  size_t at = fake::ops.size();
  for (int k = 0; k < 3; ++k) OK(step(2));
  EXPECT(fake::launches("k_adamw_host", at).size() == 3 && fake::launches("k_adamw", at).empty());
  OK(pt_stream_status(s.ctx, nullptr, nullptr, nullptr, &rebuilds));
  EXPECT(rebuilds == 0);
  at = fake::ops.size();
  for (int k = 0; k < 3; ++k) OK(step(0));
  EXPECT(fake::launches("k_adamw_host", at).empty() && fake::launches("k_adamw", at).size() == 6);
  OK(pt_stream_status(s.ctx, nullptr, nullptr, nullptr, &rebuilds));
  EXPECT(rebuilds == 1);                          // the verdict was asked for once
  h.p[0] = (char*)h.p[0] + 2;                     // off the alignment
  at = fake::ops.size();
  EXPECT(step(2) == PT_ERR_UNSUPPORTED && fake::launches("k_adamw", at).empty() && fake::launches("k_adamw_host", at).empty());
  return 0;
}

// A recompute that finalizes takes the chunks' sums and the norm in one launch of its own; one that is refused has still
// taken its chunks' sums.
int recompute_and_norm_in_one_launch() {
  State s(12, 4096);
  size_t at = fake::ops.size();
  OK(pt_chunk_grad_sqnorm(s.ctx, s.g.data(), 0, 12, PT_FINALIZE_STRICT, nullptr));
  EXPECT(fake::launches("k_scalars", at).size() == 1 && fake::launches("k_scalars", at)[0].grid.y == 12);
  at = fake::ops.size();
  pt_step_report rep;
  OK(pt_step_report_read(s.ctx, &rep, nullptr));
  EXPECT(fake::launches("k_scalars", at).empty());
  OK(s.update());                                // the constants
  EXPECT(fake::launches("k_scalars", at).size() == 1 && fake::launches("k_scalars", at)[0].grid.y == 1);
  OK(pt_step_end(s.ctx, nullptr));
  at = fake::ops.size();
  EXPECT(pt_chunk_grad_sqnorm(s.ctx, s.g.data(), 0, 5, PT_FINALIZE_STRICT, nullptr) == PT_ERR_STATE);
  EXPECT(fake::launches("k_scalars", at).size() == 1 && fake::launches("k_scalars", at)[0].grid.y == 5);
  EXPECT(s.update() == PT_ERR_STATE);
  OK(pt_chunk_grad_sqnorm(s.ctx, s.g.data(), 5, 7, PT_FINALIZE_STRICT, nullptr));
  EXPECT(fake::launches("k_scalars", at).size() == 2);
  OK(s.update());
  return 0;
}

// The launch that derives a step's constants is its end too: pt_step_end launches nothing, unless a call of the same step that
// depends on the step counter or loss scale came in between (which takes the end back), or the context has graphs.
int step_ends_with_its_constants() {
  std::unique_ptr<State> own;                      // a context each: taking an end back and a capture change its later steps
  pt_pack_plan* q = nullptr;
  pt_step_report rep;
  const hipStream_t cap = fake::stream(0xc0);
  enum { NOTHING, REPORT, AGAIN, PACK, FINALIZE, RECOMPUTE, OVERRIDE, STATE, OTHER, NO_UPDATE, CAPTURED, AFTERWARDS, N };
  for (int how = 0; how < N; ++how) {
    if (how != AFTERWARDS) { own.reset(new State(2, 4096)); q = own->plan(); }
    State& s = *own;
    OK(s.pack(q));
    OK(s.finalize(PT_FINALIZE_STRICT));
    size_t at = fake::ops.size();
    if (how != NO_UPDATE) OK(s.update());
    if (how == REPORT) OK(pt_step_report_read(s.ctx, &rep, nullptr));
    if (how == AGAIN) OK(s.update(1, 1));
    if (how == PACK) OK(s.pack(q));
    if (how == FINALIZE) OK(s.finalize(PT_FINALIZE_CARRY));
    if (how == RECOMPUTE) OK(pt_chunk_grad_sqnorm(s.ctx, s.g.data(), 0, 1, 0, nullptr));
    if (how == OVERRIDE) OK(pt_step_override(s.ctx, 1.0f, 0, nullptr));
    if (how == STATE) OK(pt_ctx_set_state(s.ctx, 3, 1.0, 0, nullptr));
    pt_hparams hp = HP;
    hp.lr = 1.0;
    if (how == OTHER) OK(pt_chunk_adamw_step(s.ctx, &hp, 0, 2, s.g.data(), s.w.data(), s.m.data(), s.v.data(), s.p.data(), nullptr));
    const bool taken_back = how >= PACK && how <= OTHER;
    EXPECT(fake::launches("k_reopen", at).size() == (taken_back ? 1u : 0u));
    at = fake::ops.size();
    if (how == CAPTURED) fake::capturing[0xc0] = true;
    OK(pt_step_end(s.ctx, how == CAPTURED ? cap : nullptr));
    fake::capturing[0xc0] = false;
    const bool of_its_own = taken_back || how >= NO_UPDATE;
    EXPECT(fake::launches("k_step_end", at).size() == (of_its_own ? 1u : 0u));
  }
  return 0;
}

// ---- steps that end with their constants, and graphs ----------------------------------------------
//
// A stand-in for the device that runs the step's scalar kernels: at once, or when the graph is replayed they were captured into.  A
// call sequence has to give the same values whether steps end with their constants or in a kernel of their own (which is
// what a context does that has been captured into a graph; here into one that is never replayed).
struct Launch {
  std::string kernel;
  PtDevState* st;
  PtScalarArgs a;
  PtFused f;
  uint32_t no;
  float mult;
  int32_t inf, step, good;
  double scale;
  bool reads_scale;
};
std::vector<Launch>* graph = nullptr;              // what is captured now
bool reads_scale = false, inf_now = false;         // of the call in flight: its kernel reads the loss scale; gradients hold an infinity
std::vector<double> seen;

void run(const Launch& l) {
  PtDevState* st = l.st;
  if (l.kernel == "k_step_end") pt_end_step(st, l.no);
  else if (l.kernel == "k_reopen") pt_take_back(st, l.no);
  else if (l.kernel == "k_override") { st->override_active = 1; st->override_grad_mult = l.mult; st->found_inf = l.inf; }
  else if (l.kernel == "k_set_state") { st->step = l.step; st->loss_scale = l.scale; st->good_steps = l.good; }
  else if (l.kernel == "k_adamw") seen.insert(seen.end(), {1.0, st->c[0], st->c[8], double(st->skip)});
  else if (l.kernel == "k_adamw_fused") {          // norm, constants and end of the step, and the update with them
    PtDevState s = *st;
    st->found_inf = st->skip = inf_now; st->override_active = s.override_active = 0;
    st->c[0] = float(s.step + 1); st->c[8] = float(1.0 / s.loss_scale);
    pt_end_early(st, s, inf_now, l.f.end_step);
    seen.insert(seen.end(), {1.0, st->c[0], st->c[8], double(st->skip)});
  }
  else if (l.kernel == "k_scalars" && st) {
    PtDevState s = *st;
    if (l.a.do_finalize) { st->found_inf = s.found_inf = inf_now; st->override_active = s.override_active = 0; }
    if (l.a.do_prepare) {
      st->c[0] = float(s.step + 1);                // the number of the update
      st->c[8] = s.override_active ? s.override_grad_mult : float(1.0 / s.loss_scale);
      st->skip = s.found_inf;
      if (l.a.end_step) pt_end_early(st, s, s.found_inf != 0, l.a.end_step);
    }
  } else if (l.reads_scale) seen.insert(seen.end(), {2.0, st->loss_scale});
}

void on_launch(const fake::Op& op, void** args) {
  Launch l{};
  l.kernel = op.kernel;
  if (op.kernel == "k_step_end" || op.kernel == "k_reopen") { l.st = *(PtDevState**)args[0]; l.no = *(uint32_t*)args[1]; }
  else if (op.kernel == "k_override") { l.st = *(PtDevState**)args[0]; l.mult = *(float*)args[1]; l.inf = *(int32_t*)args[2]; }
  else if (op.kernel == "k_set_state") { l.st = *(PtDevState**)args[0]; l.step = *(int32_t*)args[1]; l.scale = *(double*)args[2]; l.good = *(int32_t*)args[3]; }
  else if (op.kernel == "k_scalars") { l.a = *(PtScalarArgs*)args[0]; l.st = l.a.st; }
  else if (op.kernel == "k_adamw") l.st = *(PtDevState**)args[1];
  else if (op.kernel == "k_adamw_fused") { l.f = ((FusedArgs*)args[0])->work; l.st = l.f.st; }
  else if (op.kernel == "k_pack" || op.kernel == "k_accum") { l.st = *(PtDevState**)args[4]; l.reads_scale = reads_scale; }
  else if (op.kernel == "k_sqnorm" || op.kernel == "k_sqnorm_f32") { l.st = *(PtDevState**)args[3]; l.reads_scale = true; }
  else if (op.kernel == "k_init_state") {
    PtDevState* st = *(PtDevState**)args[0];
    memset(st, 0, sizeof *st);
    st->loss_scale = *(double*)args[1]; st->growth = *(double*)args[2]; st->backoff = *(double*)args[3];
    st->growth_interval = *(int32_t*)args[4]; st->scaler_enabled = *(int32_t*)args[5];
    return;
  } else return;
  if (fake::capturing[op.stream]) graph->push_back(l);
  else run(l);
}

enum Do { PACK, ACCUM, UNPACK, FINALIZE, RECOMPUTE, UPDATE, UPDATE_PART, UPDATE_OTHER, OVERRIDE, SET_STATE, END, N_CALLS, REPORT = N_CALLS, CAPTURE, CAPTURED, REPLAY };
struct Act { int what; uint32_t arg; };            // CAPTURE: the next `arg` acts go into a new graph; REPLAY: graph number `arg`
const pt_scaler_cfg SCALER = {1024.0, 2.0, 0.5, 2, 0};

// The values that `acts` lead to (`seen`) and how many kernels end a step in it.
std::vector<double> play(const std::vector<Act>& acts, bool fp32, bool kernel_ends, uint64_t elems, size_t* ends = nullptr) {
  fake::ops.clear();
  fake::on_launch = on_launch;
  seen.clear();
  std::vector<std::vector<Launch>> graphs(1);
  const hipStream_t cap = fake::stream(0xc0);
  State s(2, elems, fp32, &SCALER);
  pt_pack_plan* q = s.plan();
  if (kernel_ends) {
    graph = &graphs[0];
    fake::capturing[0xc0] = true;
    (void)pt_step_end(s.ctx, cap);
    fake::capturing[0xc0] = false;
  }
  size_t left = 0;
  auto act = [&](const Act& a, hipStream_t st) {
    int rc = PT_OK;
    reads_scale = false;
    pt_hparams hp = HP;
    pt_step_report r{};
    switch (a.what) {
      case PACK:
        reads_scale = true;
        rc = fp32 ? s.accum(q, st) : s.pack(q, st);
        break;
      case ACCUM: if (fp32) rc = pt_chunk_accum_grads(s.ctx, q, (float* const*)s.g.data(), 0, 0, st); break;
      case UNPACK: rc = pt_chunk_unpack(s.ctx, q, s.p.data(), st); break;
      case FINALIZE: rc = s.finalize(1 + a.arg % 2, st); break;
      case RECOMPUTE: rc = pt_chunk_grad_sqnorm(s.ctx, s.g.data(), a.arg % 2, 1, 2 * (a.arg / 2 % 2), st); break;
      case UPDATE: rc = s.update(st); break;
      case UPDATE_PART: rc = s.update(a.arg % 2, 1, st); break;
      case UPDATE_OTHER:
        hp.lr = 1.0 + a.arg;
        rc = pt_chunk_adamw_step(s.ctx, &hp, 0, 2, s.g.data(), s.w.data(), s.m.data(), s.v.data(), s.p.data(), st);
        break;
      case OVERRIDE: rc = pt_step_override(s.ctx, 0.25f * a.arg, a.arg % 3 == 0, st); break;
      case SET_STATE: rc = pt_ctx_set_state(s.ctx, 10 + a.arg, 64.0, a.arg % 2, st); break;
      case END: rc = pt_step_end(s.ctx, st); break;
      case REPORT:
        rc = pt_step_report_read(s.ctx, &r, st);
        seen.insert(seen.end(), {3.0, r.loss_scale, r.grad_mult, double(r.found_inf), double(r.step), double(r.good_steps)});
    }
    if (rc != PT_OK) seen.insert(seen.end(), {4.0, double(rc)});
  };
  auto step = [&](bool inf) {
    inf_now = inf;
    for (const int what : {PACK, UNPACK, FINALIZE, UPDATE, END, REPORT}) act({what, 0}, nullptr);
  };
  step(false);                                     // the pointers that a graph may use are bound by eager calls
  for (size_t i = 0; i < acts.size(); ++i) {
    inf_now = acts[i].arg % 5 == 4;
    if (acts[i].what == CAPTURE) {
      graphs.emplace_back();
      graph = &graphs.back();
      left = acts[i].arg;
      fake::capturing[0xc0] = left != 0;
    } else if (acts[i].what == REPLAY) {
      if (acts[i].arg < graphs.size())
        for (const Launch& l : std::vector<Launch>(graphs[acts[i].arg])) run(l);
    } else if (left) {
      if (acts[i].what < N_CALLS) act(acts[i], cap);
      fake::capturing[0xc0] = --left != 0;
    } else act(acts[i], nullptr);
  }
  fake::capturing[0xc0] = false;
  for (int t = 0; t < 3; ++t) step(t == 1);
  if (ends) *ends = fake::launches("k_step_end").size();
  fake::on_launch = nullptr;
  return seen;
}

std::string text(const std::vector<Act>& acts) {
  static const char* names[] = {"pack", "accum", "unpack", "finalize", "recompute", "update", "update_part", "update_other", "override", "set_state",
                                "end", "report", "capture", "captured", "replay"};
  std::string t;
  for (const Act& a : acts) t += std::string(names[a.what]) + " " + std::to_string(a.arg) + "; ";
  return t;
}

// Chunks of so few elements that an update takes a norm alone along, its plan's sums not; of so many that it takes both.
constexpr uint64_t FEW = 64, MANY = 4096;

int same(const std::vector<Act>& acts, bool fp32 = false, uint64_t elems = FEW) {
  size_t ends = 0;
  const std::vector<double> apart = play(acts, fp32, true, elems, &ends);
  const size_t fused = fake::launches("k_adamw_fused").size();
  if (fused) { fprintf(stderr, "%zu fused updates in a captured context: %s\n", fused, text(acts).c_str()); return 1; }
  const std::vector<double> now = play(acts, fp32, false, elems);
  size_t calls = 2 + 3;                            // before and behind `acts`
  for (const Act& a : acts) calls += a.what == END;
  if (ends != calls) { fprintf(stderr, "%zu calls ended a step with %zu kernels: %s\n", calls, ends, text(acts).c_str()); return 1; }
  if (apart == now) return 0;
  fprintf(stderr, "differ (fp32 %d, %zu elements): %s\n", fp32, size_t(elems), text(acts).c_str());
  for (const auto* v : {&apart, &now}) {
    for (double x : *v) fprintf(stderr, "%g ", x);
    fprintf(stderr, "\n");
  }
  return 1;
}

// A step end captured alone, in a context whose packs, norms and updates are eager: every replay ends a step.
int step_end_in_a_graph() {
  std::vector<Act> acts = {{CAPTURE, 1}, {END, 0}};
  for (int t = 0; t < 4; ++t) for (const Act& a : {Act{PACK, 0}, Act{FINALIZE, 0}, Act{UPDATE, 0}, Act{REPLAY, 1}, Act{REPORT, 0}}) acts.push_back(a);
  const std::vector<double> v = play(acts, false, false, FEW);
  EXPECT(play(acts, false, false, MANY) == v);
  std::vector<double> t;
  for (size_t i = 0; i < v.size(); i += v[i] == 1.0 ? 4 : v[i] == 3.0 ? 6 : 2)
    if (v[i] == 1.0) t.push_back(v[i + 1]);
  EXPECT((t == std::vector<double>{1, 2, 3, 4, 5, 6, 7, 7}));    // the last but one is skipped
  return same(acts) || same(acts, false, MANY);
}

// Updates with hyper-parameters of their own for each of three groups of chunks, and a norm and an update a layer: from the second step on
// no more launches than with a step end of its own.
int steps_that_go_on_behind_an_update() {
  for (int layers = 0; layers < 2; ++layers) {
    State s(3, 4096);
    std::vector<pt_pack_plan*> q;
    for (uint32_t c = 0; c < 3; ++c) q.push_back(s.plan(c));
    for (int t = 0; t < 4; ++t) {
      const size_t at = fake::ops.size();
      if (!layers) {
        for (uint32_t c = 0; c < 3; ++c) OK(s.pack(q[c]));
        OK(s.finalize(PT_FINALIZE_STRICT));
      }
      for (uint32_t c = 0; c < 3; ++c) {
        pt_hparams hp = HP;
        hp.lr *= layers ? 1.0 : c + 1.0;
        if (layers) {
          OK(s.pack(q[c]));
          OK(s.finalize(PT_FINALIZE_CARRY));
        }
        OK(pt_chunk_adamw_step(s.ctx, &hp, c, 1, &s.g[c], &s.w[c], &s.m[c], &s.v[c], &s.p[c], nullptr));
      }
      OK(pt_step_end(s.ctx, nullptr));
      if (t == 0) continue;                        // the one that finds out
      EXPECT(fake::launches("k_reopen", at).empty());
      EXPECT(fake::launches("k_step_end", at).size() == 1);
    }
  }
  State s(3, 4096);                                // updates in parts with the same hyper-parameters go on ending early
  pt_pack_plan* q = s.plan();
  for (int t = 0; t < 3; ++t) {
    OK(s.pack(q));
    OK(s.finalize(PT_FINALIZE_STRICT));
    for (uint32_t c = 0; c < 3; ++c) OK(s.update(c, 1));
    const size_t at = fake::ops.size();
    OK(pt_step_end(s.ctx, nullptr));
    EXPECT(fake::ops.size() == at);
  }
  return 0;
}

// The norm without a context, of an arena that one launch takes: under capture it is two, whose counter every replay clears for itself.
int norm_without_a_context_captured() {
  void* arena = State::device(2 * 4096);
  double* out = (double*)State::device(16);
  int32_t* inf = (int32_t*)State::device(4);
  const hipStream_t s = fake::stream(0xc0);
  for (int n = 0; n < 40; ++n) {
    const bool capture = n % 3 == 1;
    const size_t at = fake::ops.size();
    fake::capturing[0xc0] = capture;
    OK(pt_chunk_grad_sqnorm_noalloc(arena, PT_BF16, 4096, 1, 1.0, out, inf, s));
    fake::capturing[0xc0] = false;
    EXPECT(fake::launches("k_sqnorm_arena", at).size() == 1 && fake::launches("k_scalars", at).size() == (capture ? 1u : 0u));
  }
  return 0;
}

// The same on two devices in turn, eight calls each: a counter is cleared by another call on its device before it is used again.
std::vector<uintptr_t> counters;                   // used, cleared
void note_counters(const fake::Op& op, void** args) {
  if (op.kernel == "k_sqnorm_arena") for (int k : {5, 6}) counters.push_back(*(uintptr_t*)args[k]);
}
int norm_counters_of_two_devices() {
  void* arena = State::device(2 * 4096);
  double* out = (double*)State::device(16);
  int32_t* inf = (int32_t*)State::device(4);
  fake::on_launch = note_counters;
  std::map<uintptr_t, bool> spoilt;
  for (int n = 0; n < 200; ++n) {
    fake::device = n / 8 % 2;
    counters.clear();
    OK(pt_chunk_grad_sqnorm_noalloc(arena, PT_BF16, 4096, 1, 1.0, out, inf, nullptr));
    EXPECT(counters.size() == 2 && counters[0] != counters[1]);
    if (spoilt.count(counters[0])) EXPECT(!spoilt[counters[0]]);
    spoilt[counters[0]] = true;
    spoilt[counters[1]] = false;
  }
  fake::on_launch = nullptr;
  fake::device = 0;
  return 0;
}

// Sums of less than 100 MB are added to with hints (what comes between two micro-batches takes the cache from them), the first 240 MB
// of larger ones without; packed words of any size are kept.
uint64_t kept = 0;                                 // elements, of the last launch
void note_kept(const fake::Op& op, void** args) {
  if (op.kernel == "k_accum" || op.kernel == "k_pack") kept = *(uint64_t*)args[8];
}
int kept_in_the_cache_by_size() {
  fake::on_launch = note_kept;
  for (int fp32 = 0; fp32 < 2; ++fp32)
    for (uint32_t C : {1u, 6143u, 6144u, 60000u}) {
      pt_ctx* ctx = nullptr;
      pt_pack_plan* q = nullptr;
      OK(pt_ctx_create(&ctx, PT_BF16, 4096, C, nullptr));
      OK(pt_ctx_set_option(ctx, "grad_fp32", fp32));
      const pt_segment seg = {State::device(2 * 4096), 0, 4096, 0, 0, 0};
      OK(pt_pack_plan_create(ctx, &seg, 1, &q));
      std::vector<void*> g(C, nullptr);
      g[0] = State::device(4 * 4096);
      OK(fp32 ? pt_chunk_accum_grads(ctx, q, (float* const*)g.data(), 0, 0, nullptr) : pt_chunk_pack_grads(ctx, q, g.data(), nullptr));
      EXPECT(kept == (!fp32 ? 240u << 19 : C < 6144 ? 0u : 240u << 18));
      OK(pt_pack_plan_destroy(q));
      OK(pt_ctx_destroy(ctx));
    }
  fake::on_launch = nullptr;
  return 0;
}

// Unpacked words are kept as far as the plan's first 240 MB go, wherever in the context they lie.
int unpack_kept_by_size() {
  constexpr uint64_t TILE = 1 << 16, FIT = 240u << 19;
  fake::on_launch = note_kept;
  for (const auto& [n, tiles] : {std::tuple<uint64_t, uint64_t>{3, 1}, {TILE + 1, 2}, {FIT, FIT / TILE}, {FIT + 1, FIT / TILE}, {1ull << 28, FIT / TILE}})
    for (uint32_t chunk = 0; chunk < 2; ++chunk) {
      pt_ctx* ctx = nullptr;
      pt_pack_plan* q = nullptr;
      OK(pt_ctx_create(&ctx, PT_BF16, 1 << 28, 2, nullptr));
      OK(pt_ctx_set_option(ctx, "pack_tile_elems", TILE));
      void* at[2] = {State::device(16), State::device(16)};
      const pt_segment seg = {State::device(16), 0, n, 0, chunk, 0};
      OK(pt_pack_plan_create(ctx, &seg, 1, &q));
      OK(pt_chunk_unpack(ctx, q, at, nullptr));
      EXPECT(kept == tiles);
      OK(pt_pack_plan_destroy(q));
      OK(pt_ctx_destroy(ctx));
    }
  fake::on_launch = nullptr;
  return 0;
}

// Every call alone, captured on a fresh context: what reads or changes what the end of a step changes makes later steps end in a
// kernel of their own; what does not, does not.
int captured_alone() {
  for (int fp32 = 0; fp32 < 2; ++fp32)
    for (int what = 0; what < N_CALLS; ++what) {
      const bool plain = what == UNPACK || what == ACCUM || what == FINALIZE;      // the last launches nothing
      const std::vector<Act> acts = {{PACK, 0}, {FINALIZE, 0}, {UPDATE, 0}, {END, 0}, {PACK, 0}, {FINALIZE, 0}, {CAPTURE, 1}, {what, 1}, {END, 0}};
      for (uint64_t elems : {FEW, MANY}) {
        size_t ends = 0;
        (void)play(acts, fp32, false, elems, &ends);
        EXPECT(ends == (what == END ? 5u : plain ? 1u : 4u));
        // with its plan's sums: before the capture, and behind it where it did not count
        EXPECT(fake::launches("k_adamw_fused").size() == (elems == FEW ? 0u : plain ? 5u : 2u));
        if (same(acts, fp32, elems)) return 1;
      }
    }
  return 0;
}

// Call sequences at random, captures and replays among them.
int sequences_at_random() {
  std::mt19937 r(7);
  for (int n = 0; n < 6000; ++n) {
    std::vector<Act> acts;
    const int len = 4 + r() % 28;
    for (int i = 0; i < len; ++i) {
      const uint32_t x = r() % 32;
      if (x < 10) acts.push_back({int(r() % N_CALLS), uint32_t(r() % 8)});
      else if (x < 22) for (const int what : {PACK, FINALIZE, UPDATE, END}) { if (r() % 8) acts.push_back({what, uint32_t(r() % 8)}); }
      else if (x < 25) acts.push_back({REPORT, 0});
      else if (x < 27 && n % 3) acts.push_back({CAPTURE, 1 + uint32_t(r() % 5)});
      else if (x < 31 && n % 3) acts.push_back({REPLAY, 1 + uint32_t(r() % 3)});
    }
    if (same(acts, n & 1, n / 2 % 2 ? MANY : FEW)) return 1;
  }
  return 0;
}

const std::map<std::string, int (*)()> checks = {
    {"step_end_in_a_graph", step_end_in_a_graph},
    {"captured_alone", captured_alone},
    {"kept_in_the_cache_by_size", kept_in_the_cache_by_size},
    {"unpack_kept_by_size", unpack_kept_by_size},
    {"norm_counters_of_two_devices", norm_counters_of_two_devices},
    {"norm_without_a_context_captured", norm_without_a_context_captured},
    {"steps_that_go_on_behind_an_update", steps_that_go_on_behind_an_update},
    {"sequences_at_random", sequences_at_random},
    {"step_ends_with_its_constants", step_ends_with_its_constants},
    {"captured_without_the_pack", captured_without_the_pack},
    {"put_off_at_most_once", put_off_at_most_once},
    {"finalize_on_a_stream_that_is_gone", finalize_on_a_stream_that_is_gone},
    {"failed_launch_in_place", failed_launch_in_place},
    {"overlapping_host_arrays", overlapping_host_arrays},
    {"host_update_beside_the_resident_one", host_update_beside_the_resident_one},
    {"norm_occupancy_by_size", norm_occupancy_by_size},
    {"unpack_occupancy_by_size", unpack_occupancy_by_size},
    {"accumulate_occupancy_by_size", accumulate_occupancy_by_size},
    {"launch_shape_options_and_back", launch_shape_options_and_back},
    {"plan_destroyed_and_its_reduction_fails", plan_destroyed_and_its_reduction_fails},
    {"side_streams_are_judged_by_their_own_steps", side_streams_are_judged_by_their_own_steps},
    {"recompute_and_norm_in_one_launch", recompute_and_norm_in_one_launch},
};

}  // namespace

int main(int argc, char** argv) {
  const auto it = argc == 2 ? checks.find(argv[1]) : checks.end();
  if (it == checks.end()) { fprintf(stderr, "no such check\n"); return 2; }
  const int rc = it->second();
  if (rc == 0) puts("held");
  return rc;
}
