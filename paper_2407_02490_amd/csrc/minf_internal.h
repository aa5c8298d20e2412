// Internal declarations shared by the HIP translation units of libminf.
// Nothing here is part of the C ABI (see include/minf.h).
#ifndef MINF_INTERNAL_H_
#define MINF_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dispatch.h"
#include "minf.h"

namespace minf {

typedef __bf16 bf16_t;

// Per-call view of Q/K/V/O: the first of the launch's batch elements (device pointers, strides in
// elements; _sb: to the next batch element).  c_log2 = softmax_scale * log2(e): logits are scaled into the
// base-2 domain so that exp is a bare v_exp_f32.
struct QKV {
  const bf16_t *q, *k, *v;
  bf16_t *o;
  int64_t q_sb, q_sh, q_st, k_sb, k_sh, k_st, v_sb, v_sh, v_st, o_sb, o_sh, o_st;
  int32_t N, group, n_q;              // n_q: query heads of the layer (not of the call's list)
  float scale, c_log2;
};

// Head ids of one call, passed to kernels by value.
struct HeadList {
  int32_t n;
  int32_t h[MINF_MAX_HEADS];
};

// Mapping of hardware workgroup ids to work items (head slot, block).
// Consecutive hardware ids land on different XCDs (8 of them, each with its own
// 4 MB L2), and workgroups are handed to the XCDs in order, so an XCD whose
// workgroups run longer than the others' starves the rest of the chip
// (measured: per-XCD head ranges cost 44% idle time on heads of unequal
// weight).  Therefore every XCD gets the same mix at every moment: heads are
// taken in chunks; inside a chunk the blocks, heaviest (last) first, are cut
// into stripes of `stripe` consecutive blocks that are dealt to the XCDs in
// serpentine order; inside a stripe the order is (block, head).  A chunk is a
// run of consecutive list slots whose heads read the same K/V head (at most 8):
// the workgroups resident on one XCD at a time are then a few neighbouring blocks
// of one GQA group and share their K/V tiles in that XCD's L2, all XCDs work on
// the same K/V head at once, and the K/V heads in flight stay few enough for the
// memory-side cache (measured at 1M tokens: chunks that mix K/V heads cost 6% on
// Vertical-Slash and 11% on Block-Sparse attention).
// That is ORDER_BY_CHUNK.  Its price is the end of the launch: the heaviest blocks of the last chunk
// start last.  Where the caches hold the K/V heads anyway, the blocks of all heads are taken heaviest
// first: ORDER_APART gives every one of 2, 4 or 8 equal chunks its own XCDs (whose L2s then see one K/V
// head, or two), ORDER_TOGETHER goes through all heads at every block, for other lists.  OrderRule
// (dispatch.h) says where which pays.  No influence on the results.
enum { ORDER_BY_CHUNK = 0, ORDER_APART = 1, ORDER_TOGETHER = 2 };
struct Sched {
  int32_t n_heads, n_blk, stripe, ls;   // ls = stripes per XCD per chunk
  int32_t per_xcd;                      // workgroups per XCD (grid = 8 * per_xcd)
  int32_t order, apart;                 // ORDER_*; XCDs per chunk of ORDER_APART
  uint8_t cstart[MINF_MAX_HEADS];       // per list slot: first slot of its chunk
  uint8_t csize[MINF_MAX_HEADS];        // per list slot: size of its chunk
};
constexpr int SCHED_MAX_CHUNK = 8;
inline Sched make_sched(const HeadList &hl, int group, int n_blk, const OrderRule &rule = OrderRule{0, 0, 0}) {
  Sched s;
  s.n_heads = hl.n;
  s.n_blk = n_blk;
  int stripe = n_blk / 64;
  s.stripe = stripe < 1 ? 1 : (stripe > 32 ? 32 : stripe);
  const int n_stripes = (n_blk + s.stripe - 1) / s.stripe;
  s.ls = (n_stripes + 7) / 8;
  s.per_xcd = s.ls * s.stripe * hl.n;      // sum over chunks of ls * stripe * chunk size
  for (int i = 0; i < MINF_MAX_HEADS; ++i) s.cstart[i] = s.csize[i] = 0;
  s.order = ORDER_BY_CHUNK;
  s.apart = 0;
  int chunks = 0;
  bool equal = true, whole = rule.round > 0;
  for (int i = 0; i < hl.n;) {
    int j = i + 1;
    while (j < hl.n && j - i < SCHED_MAX_CHUNK && hl.h[j] / group == hl.h[i] / group) ++j;
    for (int t = i; t < j; ++t) {
      s.cstart[t] = (uint8_t)i;
      s.csize[t] = (uint8_t)(j - i);
    }
    ++chunks;
    equal = equal && j - i == s.csize[0];
    if (whole) {                        // the chunk's workgroups per XCD: whole rounds, or a last one nearly full
      const int rest = s.ls * s.stripe * (j - i) % rule.round;
      whole = rest == 0 || 4 * rest > 3 * rule.round;
    }
    i = j;
  }
  if (chunks < 2 || whole) return s;
  if (equal && 8 % chunks == 0) {
    if (!rule.apart || (rule.but & chunks)) return s;
    s.order = ORDER_APART;
    s.apart = 8 / chunks;
    s.per_xcd = (n_blk + s.apart - 1) / s.apart * s.csize[0];
  } else if (chunks <= rule.together) {
    s.order = ORDER_TOGETHER;
    s.per_xcd = (n_blk + 7) / 8 * hl.n;
  }
  return s;
}
// Work item of position hw (0 <= hw < 8 * per_xcd) of the launch order; false if that position
// holds none.  Plain integer arithmetic: also compiled for the host, where a test enumerates it.
__host__ __device__ inline bool decode_item(const Sched &s, int hw, int &slot, int &blk) {
  const int xcd = hw & 7;
  int seq = hw >> 3;
  if (s.order != ORDER_BY_CHUNK) {
    // `n` XCDs take the blocks of `heads` slots in serpentine order, the heaviest block of all heads first
    const bool apart = s.order == ORDER_APART;
    const int n = apart ? s.apart : 8, heads = apart ? s.csize[0] : s.n_heads;
    const int c = xcd / n, sub = xcd - c * n, r = seq / heads;
    slot = c * heads + seq - r * heads;
    const int rank = r * n + ((r & 1) ? n - 1 - sub : sub);
    blk = s.n_blk - 1 - rank;
    return rank < s.n_blk;
  }
  // every head contributes ls * stripe items per XCD, so the chunk follows from the head position
  const int per_head = s.ls * s.stripe;
  const int hpos = seq / per_head;
  const int c0 = s.cstart[hpos], csize = s.csize[hpos];
  seq -= c0 * per_head;
  const int per_stripe = s.stripe * csize;
  const int lstripe = seq / per_stripe;
  const int r = seq - lstripe * per_stripe;
  // stripes are dealt to the XCDs in serpentine order (0..7, 7..0, ...) so that work that
  // grows with the block index (dense causal) stays balanced across XCDs
  const int pos = (lstripe & 1) ? 7 - xcd : xcd;
  const int rank = (lstripe * 8 + pos) * s.stripe + r / csize;   // 0 = last block
  slot = c0 + r % csize;
  blk = s.n_blk - 1 - rank;
  return rank < s.n_blk;
}
// Two launches in one (Vertical-Slash and Block-Sparse heads of a layer): workgroup ids come in groups of
// 40 = 32 positions of the first launch order and 8 of the second, so that the two kinds are interleaved
// four to one and a position's low three bits stay the XCD of the hardware id.  kind 0: first, 1: second.
// Returns false if the id holds no item.  groups = max(ceil(8 a.per_xcd / 32), b.per_xcd), grid = 40 groups.
__host__ __device__ inline int mixed_groups(int a_per_xcd, int b_per_xcd) {
  const int ga = (8 * a_per_xcd + 31) / 32;
  return ga > b_per_xcd ? ga : b_per_xcd;
}
__host__ __device__ inline int mixed_groups(const Sched &a, const Sched &b) { return mixed_groups(a.per_xcd, b.per_xcd); }
__host__ __device__ inline void mixed_position(int w, int &kind, int &hw) {
  const int g = w / 40, r = w - 40 * g, xcd = r & 7, q = r >> 3;
  kind = q < 4 ? 0 : 1;
  hw = kind == 0 ? (4 * g + q) * 8 + xcd : g * 8 + xcd;
}
// Position hw of launch order WHICH.  The two orders of a mixed launch are kept apart by a comment that the
// compiler takes for an instruction: merged into one path on a reference to either, both structures (568
// bytes a lane) are copied to scratch memory first (4 + 4 heads of 1K tokens 27.6 -> 20.9 us without, 12 + 4 of
// 4K 146 -> 124, 26 + 6 of 8K 572 -> 555).
template <int WHICH>
__host__ __device__ inline bool decode_in_grid(const Sched &s, int hw, int &slot, int &blk) {
  const bool found = hw < 8 * s.per_xcd && decode_item(s, hw, slot, blk);
#ifdef __HIP_DEVICE_COMPILE__
  if (WHICH == 0) asm volatile("; order 0");
  else asm volatile("; order 1");
#endif
  return found;
}
__host__ __device__ inline bool decode_mixed(const Sched &a, const Sched &b, int w, int &kind, int &slot, int &blk) {
  int hw;
  mixed_position(w, kind, hw);
  return kind == 0 ? decode_in_grid<0>(a, hw, slot, blk) : decode_in_grid<1>(b, hw, slot, blk);
}
// The same with workgroups of four waves: an item of a kind is taken by the four waves together, or
// (each = true) every wave takes its own, four consecutive positions of the workgroup's XCD.
__host__ __device__ inline int wide_per_xcd(const Sched &s, bool each) { return each ? (s.per_xcd + 3) / 4 : s.per_xcd; }
__host__ __device__ inline bool decode_wide(const Sched &a, bool a_each, const Sched &b, bool b_each, int w, int wave,
                                            int &kind, int &slot, int &blk) {
  int hw;
  mixed_position(w, kind, hw);
  if (kind == 0 ? a_each : b_each) hw = ((4 * (hw >> 3) + wave) << 3) | (hw & 7);
  return kind == 0 ? decode_in_grid<0>(a, hw, slot, blk) : decode_in_grid<1>(b, hw, slot, blk);
}
// Returns false if this workgroup has no work item.
__device__ inline bool decode_wg(const Sched &s, int &slot, int &blk) {
  return decode_item(s, blockIdx.x, slot, blk);
}

// The batch elements of a call run in one launch: grid dimension y of the attention kernels, z of the index
// kernels.  A launch per element leaves the chip to drain, and the index kernels of short prompts do not
// fill it: two prompts of 40256 tokens, 16 heads, 3 % of 3.65 ms; pairs of short ones 188 -> 139 us and
// 147 -> 112.  The kernels are chosen as for one element, so an element has the same bits alone.  Index row
// of (batch element b, list slot s) in the index arrays and the workspace: b n + s, n listed heads.
// (Outputs that meet: batch_rule.h.)
constexpr int MAX_BATCH_LAUNCH = 16384;             // batch elements per launch (grid limit 65535)
__device__ inline QKV at_batch(QKV x, int b) {
  if (b != 0) {                                     // single prompts skip the four 64-bit products
    x.q += b * x.q_sb; x.k += b * x.k_sb; x.v += b * x.v_sb; x.o += b * x.o_sb;
  }
  return x;
}

// attention launches (attn_kernels.hip); nb: batch elements
hipError_t launch_ashape(const QKV &x, int nb, const HeadList &hl, int n_init, int n_local, hipStream_t st);
hipError_t launch_bs(const QKV &x, int nb, const HeadList &hl, const int32_t *blk_idx, const int32_t *blk_cnt,
                     const int32_t *order, int topk, hipStream_t st);
hipError_t launch_vs(const QKV &x, int nb, const HeadList &hl, const int32_t *v_idx, const int32_t *cover,
                     const uint32_t *cover_bits, const int32_t *counts, int nv, int ns,
                     int cover_words, hipStream_t st);

hipError_t launch_vs_bs(const QKV &x, int nb, const HeadList &hv, const int32_t *v_idx, const int32_t *cover,
                        const uint32_t *cover_bits, const int32_t *counts, int nv, int ns, int cover_words,
                        const HeadList &hb, const int32_t *blk_idx, const int32_t *blk_cnt, const int32_t *order,
                        int topk, hipStream_t st);

// index launches (index_kernels.hip)
size_t vs_index_ws_bytes(int N, int n_heads);
size_t bs_index_ws_bytes(int N, int n_heads, int topk);
// batch elements (1 .. batch) whose rows a workspace of at least the bytes above holds at a time
int vs_index_batch(int N, int n_heads, int nv, int ns, size_t ws_bytes, int batch);
int bs_index_batch(int N, const HeadList &hl, int group, int topk, size_t ws_bytes, int batch);
hipError_t launch_build_vs(const QKV &x, int nb, const HeadList &hl, int last_q, int nv, int ns,
                           int32_t *v_idx, int32_t *s_idx, int32_t *cover, uint32_t *cover_bits,
                           int32_t *counts, int cover_words, void *ws, hipStream_t st);
hipError_t launch_vs_lines(int N, int rows, int nv, int ns, const int32_t *s_idx, int32_t *cover,
                           uint32_t *cover_bits, int32_t *counts, int cover_words, hipStream_t st);
hipError_t launch_build_bs(const QKV &x, int nb, const HeadList &hl, int topk, int32_t *blk_idx,
                           int32_t *blk_cnt, int32_t *order, void *ws, hipStream_t st);

}  // namespace minf
#endif
