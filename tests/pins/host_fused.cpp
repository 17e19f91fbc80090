// Which updates take the step's scalar work along in their own launch, and what they are called with, on a stand-in for the HIP runtime
// (fake_hip.h): no GPU, nothing runs.  Usage: host_fused <check>.  Exit code 0 = the check held.
#include "fake_hip.h"

#include <string>
#include <tuple>

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

struct State {
  uint64_t S;
  uint32_t C;
  pt_ctx* ctx = nullptr;
  pt_pack_plan* plan = nullptr;
  std::vector<void*> at;
  // the plan: `len` elements (0: all) of each chunk, or of the first and the last alone
  State(uint32_t n, uint64_t elems, uint64_t len = 0, bool ends = false) : S(elems), C(n) {
    void* q = nullptr;
    (void)hipMalloc(&q, 16);
    at.assign(C, q);                               // only looked at
    std::vector<pt_segment> segs;
    for (uint32_t c = 0; c < C; ++c) if (!ends || c == 0 || c + 1 == C) segs.push_back({q, 0, len ? len : S, 0, c, c});
    if (pt_ctx_create(&ctx, PT_BF16, S, C, nullptr) != PT_OK || pt_pack_plan_create(ctx, segs.data(), uint32_t(segs.size()), &plan) != PT_OK) exit(3);
  }
  ~State() { pt_pack_plan_destroy(plan); pt_ctx_destroy(ctx); }
  int pack() { return pt_chunk_pack_grads(ctx, plan, at.data(), nullptr); }
  int finalize(int how = PT_FINALIZE_STRICT) { return pt_chunk_grad_sqnorm(ctx, nullptr, 0, C, how, nullptr); }
  int update(uint32_t first, uint32_t n, double lr = 1e-4) {
    const pt_hparams hp = {lr, 0.9, 0.95, 1e-8, 0.1, 1.0};
    float* const* f = (float* const*)at.data();
    return pt_chunk_adamw_step(ctx, &hp, first, n, at.data(), f, f, f, at.data(), nullptr);
  }
};
size_t count(const char* kernel, size_t from) { return fake::launches(kernel, from).size(); }

// Up to 208 chunks, if a waiting plan's sums have workgroups to take them; a launch of the scalar kernel less then.
int by_size() {
  for (const auto& [C, S, fused] : {std::tuple{1u, 760ull, false}, {1u, 768ull, true}, {8u, 504ull, false}, {8u, 512ull, true}, {9u, 8ull, true},
                                    {1u, 1ull << 16, true}, {8u, 1ull << 13, true}, {64u, 1ull << 20, true}, {208u, 4096ull, true},
                                    {209u, 4096ull, false}}) {
    State s(C, S);
    for (int step = 0; step < 3; ++step) {
      OK(s.pack());
      OK(s.finalize());
      const size_t at = fake::ops.size();
      OK(s.update(0, C));
      EXPECT(count("k_adamw_fused", at) == (fused ? 1u : 0u) && count("k_adamw", at) == (fused ? 0u : 1u));
      EXPECT(count("k_scalars", at) == (fused ? 0u : 1u));
      const fake::Op run = fake::ops.back();
      const uint64_t tiles = (S / 4 + 7 + 63) / 64, all = C * tiles;      // 2816 run at once: so many take two
      if (fused) EXPECT(run.grid.y == 1 && run.grid.x == (all < 6144 ? all : all - 2816));
      else EXPECT(run.grid.y == C && run.grid.x == tiles);
      EXPECT(run.block.x == 64);
      OK(pt_step_end(s.ctx, nullptr));
      EXPECT(count("k_step_end", at) == 0);        // the step has ended with its constants
    }
  }
  return 0;
}

// Not where something else may need the constants or a launch of its own has to come first.
int not_otherwise() {
  enum { PART, OTHER_SHAPE, OTHER_THREADS, OTHER_GRID, NO_HINTS, CAPTURED, READ, GOES_ON, RECOMPUTE, OVERRIDE, AGAIN, STREAMED, N };
  for (int how = 0; how < N; ++how) {
    State s(2, 1 << 16);
    const hipStream_t cap = fake::stream(0xc0);
    pt_step_report rep;
    if (how == OTHER_SHAPE) OK(pt_ctx_set_option(s.ctx, "adamw_unroll", 4));
    if (how == OTHER_THREADS) OK(pt_ctx_set_option(s.ctx, "adamw_threads", 256));
    if (how == OTHER_GRID) OK(pt_ctx_set_option(s.ctx, "adamw_grid", 64));
    if (how == NO_HINTS) OK(pt_ctx_set_option(s.ctx, "adamw_nt", 0));
    if (how == CAPTURED) { fake::capturing[0xc0] = true; OK(pt_step_end(s.ctx, cap)); fake::capturing[0xc0] = false; }
    if (how == GOES_ON) {                          // a step with two sets of hyper-parameters
      OK(s.pack()); OK(s.finalize()); OK(s.update(0, 2)); OK(s.update(0, 2, 1.0)); OK(pt_step_end(s.ctx, nullptr));
    }
    OK(s.pack());
    if (how == RECOMPUTE) OK(pt_chunk_grad_sqnorm(s.ctx, s.at.data(), 0, 2, PT_FINALIZE_STRICT, nullptr));
    else if (how == OVERRIDE) OK(pt_step_override(s.ctx, 1.0f, 0, nullptr));
    else OK(s.finalize());
    if (how == READ) OK(pt_step_report_read(s.ctx, &rep, nullptr));
    if (how == AGAIN) OK(s.update(0, 2));
    if (how == STREAMED) {                         // has derived the constants
      void* h[5];
      for (void*& q : h) (void)hipHostMalloc(&q, 4 << 16, 0);
      const pt_hparams hp = {1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0};
      float* const* f = (float* const*)h;
      OK(pt_stream_reserve(s.ctx, 2));
      OK(pt_chunk_stream_step(s.ctx, &hp, 1, 1, h, f + 1, f + 2, f + 3, h + 4, nullptr));
    }
    const size_t at = fake::ops.size();
    OK(how == PART ? s.update(0, 1) : s.update(0, 2));
    EXPECT(count("k_adamw_fused", at) == 0 && count("k_adamw", at) == 1);
    if (how == AGAIN || how == STREAMED) EXPECT(count("k_scalars", at) == 0);
  }
  return 0;
}

// Nor in a context with host threads, whose update waits for an event that must not be behind the whole resident one.
int not_with_host_threads() {
  State s(3, 1 << 16);
  void* h[5];
  for (void*& q : h) (void)hipHostMalloc(&q, 4 << 16, 0);
  const pt_hparams hp = {1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0};
  float* const* f = (float* const*)h;
  for (int step = 0; step < 3; ++step) {
    OK(s.pack());
    OK(s.finalize());
    const size_t at = fake::ops.size();
    OK(s.update(0, step ? 3 : 2));                 // the first one leaves a chunk to the host; later ones take all and it comes again
    OK(pt_chunk_host_adamw_step(s.ctx, &hp, 2, 1, h, f + 1, f + 2, f + 3, h + 4, 2, nullptr));
    EXPECT(count("k_adamw_fused", at) == 0 && count("k_scalars", at) == 1 && count("k_adamw", at) == 1);
    size_t record = 0, update = 0;
    for (size_t i = at; i < fake::ops.size(); ++i) {
      if (fake::ops[i].what == "record" && !record) record = i;
      if (fake::ops[i].kernel == "k_adamw") update = i;
    }
    EXPECT(record && record < update);
    OK(pt_step_end(s.ctx, nullptr));
  }
  return 0;
}

// Sums that the update does not take: k_scalars takes them in front, with all the rest where they waited.
int sums_it_does_not_take() {
  struct Case { uint32_t C; uint64_t S, len; bool ends; uint32_t pack, update; bool fused; };
  for (const Case& c : {Case{1, 16384 << 13, 0, false, 0, 0, true},         // as many tiles as sums may wait of
                        Case{1, 16385 << 13, 0, false, 1, 0, true},
                        Case{7, 2049 << 13, 0, false, 0, 0, true},          // 21 units of 4096 partial sums, the most there is room for is 24
                        Case{8, 1 << 20, 0, true, 0, 0, true},              // the first and the last of eight chunks
                        Case{9, 1 << 20, 0, true, 0, 1, false},             // of nine: room for eight
                        Case{64, 1 << 20, 8, true, 0, 1, false},
                        Case{65, 1 << 20, 8, true, 1, 0, true},             // more chunks than lanes: taken by the pack
                        Case{1, 1ull << 33, 8, false, 0, 0, true},
                        Case{1, 1ull << 34, 8, false, 0, 1, false}}) {      // 2^26 tiles
    State s(c.C, c.S, c.len, c.ends);
    size_t at = fake::ops.size();
    OK(s.pack());
    EXPECT(count("k_scalars", at) == c.pack);
    OK(s.finalize(PT_FINALIZE_CARRY));
    at = fake::ops.size();
    OK(s.update(0, c.C));
    EXPECT(count("k_scalars", at) == c.update && count("k_adamw_fused", at) == (c.fused ? 1u : 0u) && count("k_adamw", at) == (c.fused ? 0u : 1u));
  }
  return 0;
}

// A launch that fails leaves the work where it was: the next update has it done.
int failed_launch() {
  State s(2, 1 << 16);
  OK(s.pack());
  OK(s.finalize());
  fake::fail_kernel = "k_adamw_fused";
  fake::fail_after = 0;
  EXPECT(s.update(0, 2) == PT_ERR_HIP);
  fake::fail_after = -1;
  size_t at = fake::ops.size();
  OK(s.update(0, 1));
  EXPECT(count("k_scalars", at) == 1 && fake::launches("k_scalars", at)[0].grid.y == 2);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc == 2 ? argv[1] : "";
  const int rc = what == "by_size" ? by_size() : what == "not_otherwise" ? not_otherwise() : what == "not_with_host_threads" ? not_with_host_threads()
                 : what == "sums_it_does_not_take" ? sums_it_does_not_take() : what == "failed_launch" ? failed_launch() : 2;
  if (rc == 0) puts("held");
  return rc;
}
