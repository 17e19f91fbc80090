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
  State(uint32_t n, uint64_t elems) : S(elems), C(n) {
    void* q = nullptr;
    (void)hipMalloc(&q, 16);
    at.assign(C, q);                               // only looked at
    std::vector<pt_segment> segs;
    for (uint32_t c = 0; c < C; ++c) segs.push_back({q, 0, S, 0, c, c});
    if (pt_ctx_create(&ctx, PT_BF16, S, C, nullptr) != PT_OK || pt_pack_plan_create(ctx, segs.data(), C, &plan) != PT_OK) exit(3);
  }
  ~State() { pt_pack_plan_destroy(plan); pt_ctx_destroy(ctx); }
  int pack() { return pt_chunk_pack_grads(ctx, plan, at.data(), nullptr); }
  int finalize() { return pt_chunk_grad_sqnorm(ctx, nullptr, 0, C, PT_FINALIZE_STRICT, nullptr); }
  int update(uint32_t first, uint32_t n, double lr = 1e-4) {
    const pt_hparams hp = {lr, 0.9, 0.95, 1e-8, 0.1, 1.0};
    float* const* f = (float* const*)at.data();
    return pt_chunk_adamw_step(ctx, &hp, first, n, at.data(), f, f, f, at.data(), nullptr);
  }
};
size_t count(const char* kernel, size_t from) { return fake::launches(kernel, from).size(); }

// Up to 208 chunks, if a waiting plan's sums have workgroups to take them; a launch of the scalar kernel less then.
int by_size() {
  for (const auto& [C, S, fused] : {std::tuple{1u, 760ull, false}, {1u, 768ull, true}, {8u, 504ull, false}, {8u, 512ull, true}, {9u, 8ull, true}, {1u, 1ull << 16, true},
                                    {8u, 1ull << 13, true}, {64u, 1ull << 20, true}, {208u, 4096ull, true}, {209u, 4096ull, false}}) {
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
  enum { PART, OTHER_SHAPE, NO_HINTS, CAPTURED, READ, GOES_ON, RECOMPUTE, OVERRIDE, AGAIN, N };
  for (int how = 0; how < N; ++how) {
    State s(2, 1 << 16);
    const hipStream_t cap = fake::stream(0xc0);
    pt_step_report rep;
    if (how == OTHER_SHAPE) OK(pt_ctx_set_option(s.ctx, "adamw_unroll", 4));
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
    const size_t at = fake::ops.size();
    OK(how == PART ? s.update(0, 1) : s.update(0, 2));
    EXPECT(count("k_adamw_fused", at) == 0 && count("k_adamw", at) == 1);
    if (how == AGAIN) EXPECT(count("k_scalars", at) == 0);
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
  const int rc = what == "by_size" ? by_size() : what == "not_otherwise" ? not_otherwise() : what == "failed_launch" ? failed_launch() : 2;
  if (rc == 0) puts("held");
  return rc;
}
