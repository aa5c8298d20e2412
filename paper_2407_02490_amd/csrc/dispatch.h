// Rules that choose the kernel of an attention call.  Plain integer functions of the layer's shape
// and the budgets, compiled for the host only (a test evaluates them at measured sizes).  They know
// neither the listed heads nor the layout: the kernels round differently, and a head has to come out
// with the same bits whether its layer's heads are listed in one call or over several.
//
// n_q: query heads of the layer; N: tokens.  A work item is a (query head, 64-row block).
#ifndef MINF_DISPATCH_H_
#define MINF_DISPATCH_H_

#include <stdint.h>

namespace minf {

// A split launch holds one workgroup per CU (160 KiB of LDS): the layer's items in rounds of 256.  A
// rest of less than 96 items does not count: these are the shortest ones, taken last (514 items of 16K
// tokens, top-37: 117 -> 107 us with the index).
inline int64_t split_rounds(int n_q, int N) {
  const int64_t r = ((int64_t)n_q * (N / 64) + 160) / 256;
  return r < 1 ? 1 : r;
}
// Beyond 1024 items one wave per item fills every SIMD.
inline bool split_fits(int n_q, int N) { return (int64_t)n_q * (N / 64) <= 1024; }

// Block-Sparse: four waves per block (bs_split_kernel) or one (bs_kernel).
// One wave per item ends with its longest list, 1.55 us per listed block.  A round of the split
// kernel costs its own start and merge, as long as about 15 listed blocks, and then 0.52 us per
// listed block of an average list (causality shortens the first ones).  With L the longest list and
// A the average, split iff rounds (15 + A) < 3 L + 8.  One wave -> four, us:
//   256 items, 8K tokens:  top-2 12.2 -> 13.2, 8: 21.1 -> 15.8, 100: 163 -> 55
//   512 items, 8K tokens:  8: 24.0 -> 30.1, 16: 37.4 -> 37.2, 24: 49.7 -> 44.0, 100: 164 -> 86
//   768 items, 8K tokens:  37: 71.6 -> 81.9, 64: 109 -> 105, 100: 164 -> 127
//   1024 items, 8K tokens: 8: 29.6 -> 55.9, 50: 101 -> 115, 80: 143 -> 140, 100: 176 -> 159
//   1024 items, 4K tokens: 37: 74.1 -> 88.6, 64: 111 -> 96; 16K tokens: 110: 202 -> 205
//   2048 items, 8K tokens: 50: 201 -> 225, 100: 330 -> 310; 2560 items: 100: 390 -> 391
inline bool bs_split_pays(int n_q, int N, int topk) {
  const int64_t r = split_rounds(n_q, N), NB = N / 64, L = topk < NB ? topk : NB;
  const int64_t total = L * NB - L * (L - 1) / 2;                     // A NB
  return split_fits(n_q, N) && r * (15 * NB + total) < (3 * L + 8) * NB;
}

// Vertical-Slash: four waves per block (vs_split_kernel).  As above, but the length of a block's walk
// is known on the device only; nv + 4 ns stands for it (a slash brings the keys of its tile that its
// neighbours' tiles do not hold).  One wave -> four, us, for (nv, ns):
//   256 items:  every budget and length, e.g. 4K tokens (30, 64) 33 -> 22, (1000, 6096) 101 -> 39
//   512 items:  (30, 64) 4K 31 -> 35, 16K 28 -> 36, 8K 44 -> 39; (30, 256) 4K 49 -> 38, 16K 57 -> 53,
//               1K 34 -> 37; (256, 512) 4K 55 -> 40, 1K 38 -> 39; (1000, 6096) 1K 40 -> 37;
//               16 heads of 1088 tokens, (1088, 200), 272 items: layer 83 -> 71
//   768 items:  2K (1000, 6096) 62 -> 63; 4K (256, 512) 60 -> 62, (30, 1024) 90 -> 78; 8K (256, 512) 91 -> 88,
//               (30, 256) 69 -> 72; 16K (256, 512) 93 -> 96, (500, 1500) 147 -> 114
//   1024 items: 2K (1000, 6096) 65 -> 75; 4K (256, 512) 63 -> 79, (30, 1024) 82 -> 89, (30, 2048) 110 -> 100;
//               8K (30, 256) 87 -> 96, (1000, 256) 107 -> 111, (30, 512) 120 -> 112, (1000, 6096) 204 -> 160
//   2048 items: 8K (30, 2048) 226 -> 238, (1000, 6096) 341 -> 311 (four blocks per workgroup: 299)
inline bool vs_split_pays(int n_q, int N, int nv, int ns) {
  const int64_t r = split_rounds(n_q, N);
  const int64_t walk = (int64_t)(nv < N ? nv : N) + 4 * (int64_t)(ns < N ? ns : N);
  if (!split_fits(n_q, N)) return false;
  if (r <= 1) return true;
  if (r == 2) return walk >= (N >= 1536 ? 1024 : 1536);
  if (N < 3072) return false;
  return walk >= (N >= 8192 ? 2048 : r == 3 ? 4096 : 6000);
}

// Vertical-Slash: four consecutive blocks per workgroup (vs_share_kernel) or one (vs_kernel), where no
// block is split.  The four share the common part of slash runs of at least 704 offsets, and long
// runs are there only where many slashes are kept for the length of the row.  Without them the
// workgroup only holds its CU until its longest block ends, and on the shortest rows whether its
// rounds come out even decides (32, 40 and 64 heads of 2560 tokens: 98 -> 81, 118 -> 132, 153 -> 154).
// One block -> four, 32 heads unless stated, us by number of slashes:
//   2K (64 heads)   512: 91 -> 111, 1500: 105 -> 129, all: 110 -> 133;  1K (128 heads) 512: 71 -> 147
//   3K   512: 79 -> 82, 1800: 122 -> 103, all: 126 -> 106;  24 heads 512: 70 -> 79, all: 100 -> 94
//        40 heads 512: 94 -> 112, 1800: 142 -> 148, all: 148 -> 152;  64 heads 512: 122 -> 134, all: 195 -> 178
//   3.5K 512: 97 -> 103, 1200: 165 -> 156, 1800: 158 -> 141;  40 heads 1200: 186 -> 190, 1800: 180 -> 179
//   4K   512: 100 -> 101, 1024: 157 -> 156, 1500: 197 -> 187, 6096: 193 -> 173;  6K  2500: 372 -> 356
//   8K   200: 380 -> 398, 1500: 406 -> 415, 3072: 464 -> 473, 3500: 564 -> 562, 4096: 601 -> 554, 6096: 593 -> 520
//   16K  512: 714 -> 727, 2048: 920 -> 946, 4096: 1500 -> 1499, 5000: 1755 -> 1658, 6096: 1888 -> 1707
//   32K  2048: 1995 -> 2040, 4096: 2733 -> 2811, 5000: 4491 -> 4504, 6096: 5326 -> 5136, 12288: 7272 -> 6585
//   64K  4096: 4862 -> 4949, 5000: 10480 -> 10613, 6096: 12996 -> 12943, 8192: 16247 -> 15764
//   128K (8 heads)  4096: 2337 -> 2371, 6096: 8122 -> 8186, 8192: 11181 -> 11111, 12288: 16454 -> 16261
// On very long rows with many runs four neighbours gain without common tiles.  8 heads (1M: 4), ms:
//   256K  5000: 12.58 -> 12.79, 6096: 15.49 -> 15.47;  384K  4600: 18.28 -> 17.99, 6096: 31.4 -> 28.9
//   512K  4096: 8.91 -> 9.23, 4600: 21.96 -> 22.33, 5000: 28.3 -> 27.7, 6096: 42.2 -> 37.6
//   1M    4096: 9.00 -> 9.32, 5000: 47.3 -> 41.9, 6096: 65.7 -> 61.7, 12288: 168.8 -> 134.3; 24 heads of the
//         mixed recipe, four seeds: 291 -> 260, 231 -> 224, 289 -> 260, 207 -> 211 (69.5 % of the L2 requests
//         hit instead of 66.2 %, 0.87 TB from the fabric instead of 1.00)
inline bool vs_share_pays(int N, int ns) {
  if (N < 3072) return false;
  if ((int64_t)(N >= 3584 && N <= 6144 ? 3 : 2) * ns >= N) return true;
  return (int64_t)40 * (ns - 4096) >= N || (N >= 393216 && ns >= 5000);
}

// A-shape and dense (n_local >= N): four waves per block (ashape_split_kernel) against four blocks
// per workgroup that share their tiles and need a quarter of the loads.  Us, shared -> split:
//   512 items:  4K tokens (1024, 4096) 98 -> 52, (128, 1024) 58 -> 40, (0, 128) 33 -> 25, dense 99 -> 53
//   768 items:  8K tokens (1024, 4096) 134 -> 123, (0, 128) 34 -> 36, dense 177 -> 131
//   1024 items: 8K tokens (1024, 4096) 139 -> 144, (128, 1024) 62 -> 73, dense 184 -> 162;
//               dense of 4K 103 -> 99, 16K 345 -> 289, 2K 71 -> 74
//   2048 items: 8K tokens dense 307 -> 311
inline bool ashape_split_pays(int n_q, int N, int n_local) {
  const int64_t items = (int64_t)n_q * (N / 64);
  return items <= 512 || (n_local >= N && N >= 4096 && items <= 1024);
}

// Block-Sparse index of rows of up to 2048 blocks: a workgroup per 16 rows that keeps their logits in LDS
// (bs_rows_kernel, one workgroup per CU at a time), or the candidate lists of bs_topk_kernel; same bits.
// groups: workgroups of the first, over heads and batch elements.  The lists cost little where few entries
// are kept (they are cut less often), the rows cost the same for every budget.  Index build, lists -> rows, us:
//   top-1    1024 blocks, 24 heads (1536 groups) 226 -> 214, 32 (2048) 261 -> 275; 2048 blocks, 12 heads (1536)
//            354 -> 311, 16 (2048) 386 -> 400, 24 (3072) 401 -> 576; 29 heads of 1036 blocks (1885) 235 -> 281
//   top-37   24 heads of 1024 244 -> 215, 32 279 -> 274, 12 of 2048 368 -> 308, 29 of 1036 253 -> 276
//   top-64   32 heads of 1024 302 -> 276, 16 of 2048 433 -> 397, 29 of 1036 283 -> 273, 24 of 2048 455 -> 578
//   top-100  32 heads of 1024 371 -> 280, 16 of 2048 538 -> 402; 24 of 2048 (3072) 557 -> 581, 32 674 -> 761
// Of 4851 points of 700 to 2100 groups the rows lose 9 % at most (top-1) where the rule takes them, 25 % with 2048 for
// every budget; past 2048 groups they would still gain at top-80 and more.
inline bool bs_rows_pay(int64_t groups, int topk) { return groups <= (topk < 64 ? 1536 : 2048); }

// Order of a launch's work items (minf_internal.h: ORDER_*).  apart: chunks that are equal and 2, 4 or 8 get XCDs
// of their own, except for the numbers of chunks in the mask `but`; together: the largest number of other chunks
// that are mixed; round: workgroups an XCD holds, if a chunk that fills whole rounds of them by itself loses by
// either (0: it does not).
// Chunk after chunk -> apart, us (query heads / K/V heads, tokens):
//   dense   8/8 4K 72 -> 52, 8K 191 -> 163, 16K 673 -> 456, 32K 2295 -> 1746; 4/4 32K 1234 -> 884; 16/4 8K 301 -> 238;
//           32/8 4K 171 -> 133, 8K 514 -> 467, 20K 2779 -> 2712; 8/2 8K..32K, 16/4 16K, 4/4 64K the same;
//           whole rounds of four-wave blocks (or nearly): 16/4 4K 96.7 -> 98.6; VS 16/4 3200 tokens, layer 104 -> 109
//   A-shape 32/8 4K 172 -> 133, 8K 458 -> 420, 32K 2215 -> 2162, 64K 4864 -> 4548, 128K 9750 -> 9398; 8/4 11K 249 -> 188;
//           16/4 64K 2331 -> 2263; worst 6/2 16K 260 -> 265
//   BS      32/8 4K 198 -> 147, 8K 578 -> 540, 16K 1417 -> 1391, 32K 3140 -> 3091; 8/8 20K 578 -> 469, 32K 924 -> 832;
//           8/2 16K 391 -> 386, 32K 814 -> 815, 64K 1710 -> 1797; 4/4 64K 959 -> 990
//   VS, four blocks per workgroup: 32/8 4K 182 -> 135, 8K 517 -> 467; 16/8 13K 676 -> 581; 8/8 16K 599 -> 452, 20K 733 -> 678;
//           16/8 26K 1871 -> 1970; 8/8 64K 3430 -> 3818; whole rounds: 16/4 16K 869 -> 867, 32K 2768 -> 2949
//   VS, others: 8/8 4K 72 -> 54, 8K 189 -> 164; 4/4 8K 111 -> 87; (500, 1500) 16/4 8K 320 -> 257, 32/8 8K 518 -> 500,
//           16K 1194 -> 1256; 8/8 32K 731 -> 783; (30, 64) 32/8 2816 tokens 64.6 -> 53.8, 3136 the same, 4800 71.7 -> 80.0,
//           6784 103 -> 118, 7488 106 -> 130, 16/4 6208 45.9 -> 53.9, but 8/8 6464 48.8 -> 40.5; (30, 128) 32/8 4800
//           109 -> 111, 6784 172 -> 170, 16/4 6208 82.7 -> 77.6; (256, 512) 32/8 4800 197 -> 174, 6784 291 -> 266
//   VS, four waves per block where the walk does not grow over the whole row, two chunks, three and more rounds of items,
//         4/2 heads: (256, 512) 8640 56.5 -> 61.2, 9600 65.3 -> 62.5, 13440 75.6 -> 88.3, 16000 88.6 -> 84.9; (3000, 200) 11840
//         90.2 -> 100, 15680 116 -> 108; (500, 1500) 12160 143 -> 136, 13760 135 -> 151; longer walks (100, 1800) 12480
//         162 -> 161, 13120 182 -> 170, 13760 163 -> 171, (30, 2048) 13120 181 -> 170; two rounds of items gain 0 to 3 %
//         four chunks of short walks, three rounds: (256, 512) 8/4 4160 46.0 -> 48.9, 4480 51.0 -> 54.3, 4/4 8320 49.7 -> 56.2,
//         9600 55.8 -> 59.6, 11.2K 58.7 -> 63.4, 11.5K 67.1 -> 62.3, 12.5K the same; of longer ones (3000, 200) 4/4 9280
//         86.2 -> 78.7, (30, 2048) 8640 104 -> 94.1
// Chunk after chunk -> together, 12 heads of 3 K/V heads unless stated:
//   dense 4K 84 -> 77, 8K 217 -> 207, 16K 768 -> 698; A-shape 4K 85 -> 77, 8K..64K within 1 %
//   BS    4K 88 -> 81, 8K 243 -> 212, 16K 591 -> 567, 32K 1226 -> 1372; 8 chunks of 16K 413 -> 529; beyond 8K only for
//         long lists: top-16  11K 72.2 -> 75.5, 10/5 9K 71.7 -> 77.0, 6/3 16K 72.6 -> 82.9;  top-37  15K 227 -> 232,
//         5/5 9K 68.0 -> 73.4, 6/3 16K 145 -> 164;  top-64  10/5 9K 206 -> 186, 3/3 12K 94.8 -> 87.7, 6/3 16K 238 -> 261;
//         top-100  11K 303 -> 262, 15K 512 -> 464, 10/5 9K 249 -> 205, 6/3 16K 345 -> 338, worst 3/3 16K 151 -> 157
//         (some lists of a few blocks gain there too: top-8 11K 57.6 -> 50.8)
//   VS, four blocks per workgroup: 8K 217 -> 205, 16K 735 -> 681, 32K 2213 -> 2134; others: 4K 91 -> 89,
//         (500, 1500) 8K 220 -> 236; four-wave blocks of 7 chunks 8K 318 -> 328 (mixed layer)
//   VS, four waves per block, where the walk does not grow over the whole row: (500, 1500) 7/7 3712 67.8 -> 56.3,
//         6/3 4608 62.6 -> 54.5, 7/7 4992 81.4 -> 88.1, 6/6 6912 96.1 -> 111, 5/5 8K 100 -> 110; (256, 256) 5/5 4032
//         53.5 -> 42.7, 6848 63.5 -> 73.9, 3/3 11K 62.3 -> 72.0; where it does: (1000, 6096) 7/7 4992 82.1 -> 75.5,
//         5/5 6144 84.9 -> 69.5, 8K 121 -> 116, 3/3 9344 108 -> 84.5, 6/3 9920 184 -> 192, 3/3 12160 146 -> 159, two
//         prompts of 15744 407 -> 451; (3000, 200) 3/3 9344 79.4 -> 67.4
struct OrderRule {
  int apart, together, round, but = 0;
};
constexpr int XCD_CUS = 32;                        // workgroups of 128 KiB and more that an XCD holds
inline OrderRule split_order(int N) {              // four waves per block, any kind; three K/V heads of 16K fit the L2s
  return OrderRule{N <= 16384, 49152 / N, XCD_CUS};
}
inline OrderRule vs_order(int n_q, int N, int nv, int ns, bool split, bool share) {
  const int64_t walk = nv + 4 * (int64_t)ns;
  OrderRule r = split   ? split_order(N)
                : share ? OrderRule{N <= 20480, N <= 32768 ? 64 : 0, XCD_CUS}
                        : OrderRule{N <= 8192, N <= 4096 ? 64 : 0, 0};
  // blocks of short walks weigh all the same
  if (!split && !share && N > 3072 && (int64_t)n_q * (N / 64) > 1024 && walk < 512) r.apart = 0;
  const bool flat = 16 * (int64_t)(nv > ns ? nv : ns) < 5 * (int64_t)N;        // no walk grows over the whole row
  if (split && (N > 12032 || (N > 4608 && flat))) r.together = 0;
  if (split && flat && (int64_t)n_q * (N / 64) > 512) {
    if (N > 8192 && N <= 14336 && walk < 7168) r.but |= 2;
    if (N > 4096 && N <= 11264 && walk < 3072) r.but |= 4;
  }
  return r;
}
inline OrderRule bs_order(int N, int topk, bool split) {
  OrderRule r = split ? split_order(N) : OrderRule{N <= 32768, N <= 16384 ? 49152 / N : 0, 0};
  if (N > 8192 && (topk < 64 || (topk < 100 && N > 14336))) r.together = 0;
  return r;
}
inline OrderRule ashape_order(int N) { return OrderRule{N <= 131072, N <= 65536 ? 64 : 0, 0}; }

}  // namespace minf
#endif
