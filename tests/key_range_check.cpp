// Host check of the range passes of the register selection (key_range.h): the passes of
// reg_threshold with the counts taken by plain loops, on rows whose places without an element hold
// 0, against a sort.  Every selection must keep exactly its k largest keys.  Built and run by
// tests/test_sched_host.py.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#define MINF_HD
#include "key_range.h"

using namespace minf;

static unsigned order_key(float f) {
  unsigned u;
  memcpy(&u, &f, 4);
  return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}

static float bits(unsigned u) {
  float f;
  memcpy(&f, &u, 4);
  return f;
}

static int check(const char *name, const std::vector<float> &row, int places, int k) {
  std::vector<unsigned> u((size_t)places, 0u);
  for (size_t i = 0; i < row.size(); ++i) u[i] = std::max(order_key(row[i]), 1u);
  unsigned lo = 0xffffffffu, hi = 0u;
  for (unsigned e : u) { lo = std::min(lo, e - 1u); hi = std::max(hi, e); }
  KeyRange r{lo + 1u, hi};
  unsigned thr = 0;
  int eq = 0, krem = k, pass = 0;
  for (;; ++pass) {
    if (pass == 4) { printf("FAIL %s n %zu k %d: no end\n", name, row.size(), k); return 1; }
    const int shift = key_range_shift(r);
    std::vector<int> hist(REG_BINS, 0);
    for (unsigned e : u)
      if (key_range_has(r, e)) {
        const unsigned bin = (e - r.lo) >> shift;
        if (bin >= (unsigned)REG_BINS) { printf("FAIL %s n %zu k %d: bin %u\n", name, row.size(), k, bin); return 1; }
        ++hist[bin];
      }
    int bin = REG_BINS - 1;
    while (bin >= 0 && hist[bin] < krem) krem -= hist[bin--];
    if (bin < 0) { printf("FAIL %s n %zu k %d: no bin\n", name, row.size(), k); return 1; }
    r = key_range_bin(r, (unsigned)bin, shift);
    if (shift == 0) { thr = r.lo; eq = krem; break; }
    if (hist[bin] == krem) { thr = r.lo - 1u; eq = 0; break; }
  }
  std::vector<unsigned> sorted;
  for (size_t i = 0; i < row.size(); ++i) sorted.push_back(u[i]);
  std::sort(sorted.begin(), sorted.end(), [](unsigned a, unsigned b) { return a > b; });
  // kept: keys above thr, then eq of those equal to it
  int gt = 0, same = 0;
  for (unsigned e : u) { gt += e > thr; same += e == thr && e != 0u; }
  const bool ok = gt + eq == k && eq <= same && (gt == 0 || sorted[gt - 1] > thr) && sorted[k - 1] == (eq ? thr : sorted[gt - 1]);
  if (!ok) { printf("FAIL %s n %zu k %d: kept %d above and %d of %d equal\n", name, row.size(), k, gt, eq, same); return 1; }
  return 0;
}

int main() {
  int bad = 0, n_cases = 0;
  std::mt19937 g(7);
  std::uniform_real_distribution<float> uni(0.f, 1.f);
  const struct { int n, places; } sizes[] = {{64, 4096}, {4160, 8192}, {8192, 8192}, {8256, 12288}, {40960, 40960}};
  for (auto z : sizes)
    for (int k : {1, 2, 3, 30, 64}) {
      auto run = [&](const char *name, auto value) {
        std::vector<float> row((size_t)z.n);
        for (int i = 0; i < z.n; ++i) row[(size_t)i] = value(i);
        bad |= check(name, row, z.places, k);
        ++n_cases;
      };
      run("uniform", [&](int) { return uni(g); });
      run("positive", [&](int i) { return 0.01f + 1e-6f * (float)i; });
      run("equal", [&](int) { return 0.25f; });
      run("few values", [&](int i) { return (float)(i % 3); });
      run("both signs", [&](int) { return uni(g) - 0.5f; });
      run("infinities", [&](int i) { return i % 5 == 0 ? INFINITY : i % 5 == 1 ? -INFINITY : uni(g); });
      // NaN scores: the quiet NaN of the hardware and the payloads that bf16 inputs can carry; their
      // keys end at 2^32, where the range of a last bin must not come back around to 0
      for (unsigned nan : {0x7fc00000u, 0x7fff0000u, 0x7fffffffu, 0xffc00000u, 0xffff0000u, 0xffffffffu})
        for (int count : {1, 3, 64})
          run("nan", [&](int i) { return i < count ? bits(nan) : 0.01f + 1e-6f * (float)i; });
      run("all nan", [&](int i) { return bits(0x7fff0000u | (unsigned)(i & 0xffff)); });
      run("extremes", [&](int i) { return i % 2 ? bits(0x7fffffffu) : bits(0xffffffffu); });
    }
  if (!bad) printf("ok cases %d\n", n_cases);
  return bad;
}
