// Arithmetic of the range passes of the register selection (index_kernels.hip: reg_threshold).
// Plain integer code, also compiled for the host, where a test runs whole selections with it.
#ifndef MINF_KEY_RANGE_H_
#define MINF_KEY_RANGE_H_

#ifndef MINF_HD
#define MINF_HD __host__ __device__
#endif

namespace minf {

constexpr int REG_BINS = 2048;

// A pass looks at the order keys lo <= u <= hi (lo >= 1: the value 0 stands for "no element") in
// bins of 1 << shift keys; bin of u = (u - lo) >> shift < REG_BINS.
struct KeyRange {
  unsigned lo, hi;
};

MINF_HD inline int key_range_shift(const KeyRange &r) {
  const unsigned width = r.hi - r.lo;
  return width < (unsigned)REG_BINS ? 0 : 21 - __builtin_clz(width);
}

MINF_HD inline bool key_range_has(const KeyRange &r, unsigned u) { return u - r.lo <= r.hi - r.lo; }

// The range of one bin.  Its end is taken as a distance from its start, which cannot wrap: a last
// bin that reaches past 2^32 (keys of NaN scores lie there) would otherwise come back around to 0
// and count the places without an element.
MINF_HD inline KeyRange key_range_bin(const KeyRange &r, unsigned bin, int shift) {
  KeyRange b;
  b.lo = r.lo + (bin << shift);
  const unsigned width = r.hi - b.lo, bin_width = (1u << shift) - 1u;
  b.hi = b.lo + (width < bin_width ? width : bin_width);
  return b;
}

}  // namespace minf
#endif
