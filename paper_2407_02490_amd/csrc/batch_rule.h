// Whether the batch elements of an attention call may run at the same time (host only, plain C++; a test
// compares it with enumerated layouts).  Outputs that lie over each other, or over what another element
// reads, have to be written in batch order, one launch per element: the order that a caller sees then does
// not depend on which block ends first.  The rule only has to be right when it says "apart"; layouts that it
// cannot tell apart get one launch per element.
#ifndef MINF_BATCH_RULE_H_
#define MINF_BATCH_RULE_H_

#include <stdint.h>

namespace minf {

// [batch][heads][tokens][128] elements of 2 bytes from `base` (an address / 2) on; strides in elements, >= 0.
struct BatchLayout {
  uint64_t base;
  int64_t sb, sh, st;
  int64_t batch, heads, tokens;
  int64_t row_end() const { return (heads - 1) * sh + 128; }                    // of the heads of one token
  int64_t element_end() const { return (tokens - 1) * st + row_end(); }         // of one batch element
  int64_t end() const { return (batch - 1) * sb + element_end(); }
};

// No two places of the layout are the same: every stride steps over all that the smaller ones reach.
inline bool places_differ(const BatchLayout &o) {
  int64_t stride[3] = {o.sb, o.sh, o.st}, size[3] = {o.batch, o.heads, o.tokens}, reach = 128;
  for (int i = 0; i < 3; ++i) {
    int least = i;
    for (int j = i + 1; j < 3; ++j)
      if (stride[j] < stride[least]) least = j;
    const int64_t s = stride[least], n = size[least];
    stride[least] = stride[i]; size[least] = size[i];
    if (n == 1) continue;
    if (s < reach) return false;
    reach += (n - 1) * s;
  }
  return true;
}

// Places of o repeated every `period` elements never meet those of x: ends within the period.
inline bool periods_apart(const BatchLayout &o, const BatchLayout &x, int64_t period, int64_t o_end, int64_t x_end) {
  if (period <= 0 || o_end > period || x_end > period) return false;
  const uint64_t p = (uint64_t)period;
  const int64_t r = (int64_t)((o.base % p + p - x.base % p) % p);              // start of o behind a start of x
  return r >= x_end && r + o_end <= period;
}

// o and the input x: disjoint, as whole ranges, per batch element or per token (slices of one fused buffer).
inline bool input_apart(const BatchLayout &o, const BatchLayout &x) {
  if (o.base >= x.base + (uint64_t)x.end() || x.base >= o.base + (uint64_t)o.end()) return true;
  if (o.sb == x.sb && periods_apart(o, x, o.sb, o.element_end(), x.element_end())) return true;
  return o.sb == x.sb && o.st == x.st && o.st > 0 && o.sb % o.st == 0 &&
         periods_apart(o, x, o.st, o.row_end(), x.row_end());
}

// q, k, v, o: of the heads that the call reads or writes.  (o in the place of q: a block reads its own rows
// before it writes them.)
inline bool batch_apart(const BatchLayout &q, const BatchLayout &k, const BatchLayout &v, const BatchLayout &o) {
  if (o.batch == 1) return true;
  const bool in_place = o.base == q.base && o.sb == q.sb && o.sh == q.sh && o.st == q.st;
  return places_differ(o) && (in_place || input_apart(o, q)) && input_apart(o, k) && input_apart(o, v);
}

}  // namespace minf
#endif
