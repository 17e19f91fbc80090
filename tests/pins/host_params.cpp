// The host-side update's 16-bit parameters leave past the caches, a block at a time: every alignment of the array, lengths around a
// vector and a block, the gradient in the same array - against one pass over the elements, with what lies around them untouched.
// With plain stores too, which calls take whose state fits the caches.
// Exit code 0 = the same bits.
#include <cstdio>
#include <vector>

#include "pt_host_update.h"

int main() {
  using namespace pt_host;
  for (uint64_t chunks : {1, 3}) {                 // the line between the two
    Job job;
    job.n_chunks = uint32_t(chunks);
    job.S = (STREAM_ELEMS + chunks - 1) / chunks;
    job.prepare();
    if (!job.stream) return 2;
    job.S -= 8;
    job.prepare();
    if (job.stream) return 3;
  }
  const Consts k{0.9f, 0.95f, 0.1f, 0.05f, 0.99999f, 1e-3f, 3.2f, 1e-8f, 0.7f};
  std::vector<uint64_t> lengths;
  for (uint64_t n = 0; n <= 40; ++n) lengths.push_back(n);
  for (uint64_t b : {PARAM_BLOCK, 2 * PARAM_BLOCK})
    for (uint64_t n = b - 9; n <= b + 9; ++n) lengths.push_back(n);
  for (int how = 0; how < 4; ++how)
    for (int own_gradient = 0; own_gradient < 2; ++own_gradient)
      for (uint64_t off = 0; off < 40; ++off)
        for (uint64_t n : lengths) {
          const bool fp16 = how & 1, stream = how < 2;
          std::vector<uint16_t> g(n), mem(n + 128, 0xabcd);
          std::vector<float> w(n), m(n), v(n), w2, m2, v2;
          uint32_t r = uint32_t(n * 131 + off);
          for (uint64_t i = 0; i < n; ++i) {
            r = r * 1664525u + 1013904223u;
            g[i] = uint16_t(r >> 16) & 0xbbffu;
            w[i] = float(int(r >> 8 & 0xffff) - 32768) * 1e-6f; m[i] = w[i] * 0.01f; v[i] = w[i] * w[i];
          }
          w2 = w; m2 = m; v2 = v;
          uint16_t* p = reinterpret_cast<uint16_t*>((reinterpret_cast<uintptr_t>(mem.data()) + 63) & ~uintptr_t(63)) + off;
          const uint16_t* from = g.data();
          if (own_gradient) { std::copy(g.begin(), g.end(), p); from = p; }
          (fp16 ? update_fp16 : update_bf16)(k, from, w.data(), m.data(), v.data(), p, n, stream);
          for (uint64_t i = 0; i < n; ++i) {
            const float gg = (fp16 ? fp16_to_f32(g[i]) : bf16_to_f32(g[i])) * k.gm;
            const float mn = std::fmaf(k.b1, m2[i], k.omb1 * gg), t2 = k.omb2 * gg, vn = std::fmaf(k.b2, v2[i], t2 * gg);
            const float u = mn / std::fmaf(std::sqrt(vn), k.rsb2, k.eps), wn = std::fmaf(-k.step_size, u, w2[i] * k.decay);
            if (p[i] != (fp16 ? f32_to_fp16(wn) : f32_to_bf16(wn)) || w[i] != wn || m[i] != mn || v[i] != vn) {
              fprintf(stderr, "fp16 %d own %d offset %zu length %zu element %zu\n", fp16, own_gradient, size_t(off), size_t(n), size_t(i));
              return 1;
            }
          }
          for (uint16_t* q = mem.data(); q < mem.data() + mem.size(); ++q)
            if ((q < p || q >= p + n) && *q != 0xabcd) { fprintf(stderr, "offset %zu length %zu: written outside\n", size_t(off), size_t(n)); return 1; }
        }
  puts("held");
  return 0;
}
