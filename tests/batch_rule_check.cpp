// Host check of batch_rule.h: what the rule calls apart is apart place by place, on small layouts drawn over
// one buffer, and the layouts that programs use are called apart.  Built and run by tests/test_sched_host.py.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "batch_rule.h"

using namespace minf;

// places of batch element b, as 8-element units of a buffer
template <class F>
static void places(const BatchLayout &x, int64_t b, F f) {
  for (int64_t h = 0; h < x.heads; ++h)
    for (int64_t t = 0; t < x.tokens; ++t)
      for (int64_t d = 0; d < 128; d += 8) f((int64_t)x.base + b * x.sb + h * x.sh + t * x.st + d);
}
// no place that one element writes is read or written by another one
static bool truly_apart(const BatchLayout *in, const BatchLayout &o) {
  std::map<int64_t, int64_t> writer;
  for (int64_t b = 0; b < o.batch; ++b) {
    bool ok = true;
    places(o, b, [&](int64_t p) { ok = ok && writer.emplace(p, b).first->second == b; });
    if (!ok) return false;
  }
  for (int i = 0; i < 3; ++i)
    for (int64_t b = 0; b < o.batch; ++b) {
      bool ok = true;
      places(in[i], b, [&](int64_t p) {
        const auto w = writer.find(p);
        ok = ok && (w == writer.end() || w->second == b);
      });
      if (!ok) return false;
    }
  return true;
}

static int bad = 0, apart_seen = 0, other_seen = 0;
static void expect(const char *what, bool want, const BatchLayout &q, const BatchLayout &k, const BatchLayout &v,
                   const BatchLayout &o) {
  if (batch_apart(q, k, v, o) != want) {
    printf("FAIL %s: apart is %d\n", what, !want);
    bad = 1;
  }
}

int main() {
  const int64_t B = 3, H = 4, G = 2, N = 64, D = 128, far = 1 << 30;
  auto head = [&](uint64_t base, int64_t n) { return BatchLayout{base, n * N * D, N * D, D, B, n, N}; };
  auto token = [&](uint64_t base, int64_t n) { return BatchLayout{base, n * N * D, D, n * D, B, n, N}; };
  // slices of one fused buffer of F heads, from head h on
  auto fused_h = [&](int64_t F, int64_t h, int64_t n) { return BatchLayout{(uint64_t)(far + h * N * D), F * N * D, N * D, D, B, n, N}; };
  auto fused_t = [&](int64_t F, int64_t h, int64_t n) { return BatchLayout{(uint64_t)(far + h * D), F * N * D, D, F * D, B, n, N}; };
  const BatchLayout q = head(far, H), k = head(2 * far, G), v = head(3 * far, G);
  expect("head-major", true, q, k, v, head(0, H));
  expect("token-major", true, token(far, H), token(2 * far, G), token(3 * far, G), token(0, H));
  expect("batch inside the tokens", true, q, k, v, BatchLayout{0, H * D, D, B * H * D, B, H, N});
  expect("fused, output apart", true, fused_t(8, 0, 4), fused_t(8, 4, 2), fused_t(8, 6, 2), token(0, H));
  expect("fused token-major, in place", true, fused_t(8, 0, 4), fused_t(8, 4, 2), fused_t(8, 6, 2), fused_t(8, 0, 4));
  expect("fused head-major, in place", true, fused_h(8, 0, 4), fused_h(8, 4, 2), fused_h(8, 6, 2), fused_h(8, 0, 4));
  expect("fused with the output", true, fused_t(12, 0, 4), fused_t(12, 4, 2), fused_t(12, 6, 2), fused_t(12, 8, 4));
  expect("fused head-major with the output", true, fused_h(12, 8, 4), fused_h(12, 4, 2), fused_h(12, 6, 2), fused_h(12, 0, 4));
  expect("one set of keys", true, q, BatchLayout{2u << 30, 0, N * D, D, B, G, N}, v, head(0, H));
  expect("one output", false, q, k, v, BatchLayout{0, 0, N * D, D, B, H, N});
  expect("outputs one head apart", false, q, k, v, BatchLayout{0, N * D, N * D, D, B, H, N});
  expect("outputs one token apart", false, q, k, v, BatchLayout{0, D, N * D, D, B, H, N});
  expect("output over the keys of the element before", false, q, BatchLayout{0, H * N * D, N * D, D, B, G, N}, v,
         BatchLayout{(uint64_t)(H * N * D), H * N * D, N * D, D, B, H, N});
  expect("output over the queries of the element before", false, BatchLayout{0, H * N * D, N * D, D, B, H, N}, k, v,
         BatchLayout{(uint64_t)(H * N * D), H * N * D, N * D, D, B, H, N});
  expect("one element", true, q, k, v, BatchLayout{0, 0, N * D, D, 1, H, N});
  srand(7);
  for (int i = 0; i < 60000; ++i) {
    BatchLayout x[4];
    const int64_t batch = 2 + rand() % 2, heads = 1 + rand() % 3, tokens = 1 + rand() % 3;
    const int64_t unit[] = {0, 64, 128, 136, 256, 384, 512, 768, 1024, 1152, 1536, 2304, 4608};
    const int64_t sb = unit[rand() % 13], sh = unit[rand() % 13], st = unit[1 + rand() % 12];
    for (int t = 0; t < 4; ++t) {
      const bool same = rand() % 2;
      x[t] = BatchLayout{(uint64_t)(64 * (rand() % 80)), same ? sb : unit[rand() % 13], same ? sh : unit[rand() % 13],
                         same ? st : unit[1 + rand() % 12], batch, heads, tokens};
    }
    if (rand() % 4 == 0) x[0].base = x[3].base;
    const bool apart = batch_apart(x[0], x[1], x[2], x[3]);
    ++(apart ? apart_seen : other_seen);
    if (apart && !truly_apart(x, x[3])) {
      printf("FAIL drawn layout %d is not apart\n", i);
      bad = 1;
    }
  }
  if (apart_seen < 1000 || other_seen < 1000) { printf("FAIL draws %d %d\n", apart_seen, other_seen); bad = 1; }
  if (!bad) printf("ok layouts %d apart, %d not\n", apart_seen, other_seen);
  return bad;
}
