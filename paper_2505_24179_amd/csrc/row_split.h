// Which attention calls run with two waves per row (NT = 1 of attn_rows_kernel), which sparse ones of the others take their
// shorter rows from queues, and how many heads a wave of the Selection-Pass takes.  Host only, plain C++.
//
// A SIMD holds one wave of either form, so 1024 waves run at a time.  Up to 512 rows every half row has a place from the
// start, and the longest row, which is the call, takes about two thirds of the time.  With more rows the rest waits for
// places: what a row costs besides its blocks (start, Q in, O out) is then paid one after the other, twice as often as
// with whole rows, and the operand loads, twice as many per FLOP, begin to count.  So the limit goes by the longest row.
// Attention call, us, one wave per row -> two (group of 4 where the rows allow it; rows of one batch, all alike; operands with a
// sink and a query's own key as its largest, masks that keep as much as the Selection-Pass does):
//                        rows  512              768              1024             1280             1536             2048
//   sparse bf16,      1 block 14.5 -> 13.8     15.9 -> 18.9     18.5 -> 20.8     26.6 -> 26.6     28.1 -> 27.9     33 -> 34.3
//                     2      17.8 -> 15.6     19.8 -> 21.8     22.1 -> 23.9     28.3 -> 30.1     31.5 -> 33.2     37.3 -> 39.5
//                     4      20.9 -> 17.9     23.6 -> 22.9     26.4 -> 26.2     30.4 -> 32.6     32.8 -> 34.7     39 -> 43.4
//                     8      27.6 -> 21.5     29.9 -> 25.5     33.3 -> 29.9     35.1 -> 37.8     38.5 -> 39.7     44.2 -> 48.9
//                    16      39.4 -> 27.3     43.9 -> 32.6     44.6 -> 36.5     50.6 -> 48.9     47.9 -> 50.4     56.4 -> 62.9
//                    32      56.7 -> 38       65 -> 43.7       63.4 -> 48.1     69.9 -> 62.9     71.7 -> 70.3     78.8 -> 85.2
//                    64      90.4 -> 58.2     98 -> 66         102 -> 73.7      100 -> 90.8      104 -> 103       117 -> 131
//                   128      127 -> 78.4      131 -> 91.3      134 -> 97        141 -> 136       142 -> 142       152 -> 177
//   32-key blocks,    4 block 21.2 -> 17.4     23.6 -> 23.3     26.4 -> 26.5     30.5 -> 32.7     33 -> 35         39.1 -> 44
//                     8      27.3 -> 21.2     29.8 -> 26       32.8 -> 29.6     34.6 -> 37.5     38.3 -> 39.7     43.9 -> 48.7
//                    16      36.8 -> 25.8     42.7 -> 32.5     42.1 -> 36.2     47.3 -> 47.5     45.8 -> 49       53.2 -> 61.1
//                    32      53.3 -> 35.8     61 -> 40.8       58.9 -> 45.6     63.3 -> 61.1     65.3 -> 67       71.4 -> 82.4
//                    64      67.8 -> 45.2     73.2 -> 51.2     78 -> 59.5       77.6 -> 73.9     81.1 -> 83.2     92.8 -> 106
//                   128      100 -> 62        96.5 -> 67.7     98 -> 73.7       106 -> 99        102 -> 103       113 -> 129
//   sparse int8,      8 block 35.6 -> 29.2     39.9 -> 35.7     42.1 -> 40.1     45.1 -> 48.3     50.5 -> 52.3     59.7 -> 64.9
//                    16      45.2 -> 34.3     53.1 -> 42.5     53.5 -> 46.3     57.9 -> 57.8     58.1 -> 60.8     70.4 -> 76.5
//                    32      64.9 -> 46.1     70.1 -> 51.5     69.4 -> 55.7     74.9 -> 70.4     80.1 -> 77.8     86.5 -> 95.4
//                    64      91.4 -> 61.9     101 -> 69.3      105 -> 76.7      104 -> 94.6      105 -> 105       118 -> 132
//                   128      124 -> 80.4      134 -> 92        132 -> 96.6      138 -> 126       144 -> 137       150 -> 170
//   sparse FP8,       1 block 25.9 -> 23.8     30.8 -> 31.8     34.4 -> 34.7     47 -> 42.3       49.8 -> 45.5     56.8 -> 55.5
//                     2      29.4 -> 24.8     34.8 -> 33       34.8 -> 36.1     46.4 -> 43.8     50 -> 46.4       57.1 -> 57.2
//                     8      36.1 -> 27.6     42.5 -> 36.1     41.7 -> 39.8     51 -> 48.7       55 -> 52.1       63.3 -> 64
//                    16      45.7 -> 32.4     52.5 -> 40.5     51.2 -> 44.8     56.1 -> 54.4     60.2 -> 59       70.9 -> 72.4
//                    32      62.3 -> 42       67.5 -> 46.4     66.5 -> 52.4     69 -> 65.2       69.6 -> 70.8     83.7 -> 87.8
//                    64      87.4 -> 55.5     93.6 -> 60.5     90.8 -> 68.4     94 -> 84.5       93.6 -> 92.7     109 -> 116
//                   128      114 -> 74        119 -> 75.8      115 -> 84.3      120 -> 109       131 -> 118       133 -> 146
//   dense bf16,       1 block 14.8 -> 12       15.5 -> 17.1     17.7 -> 19.1     26 -> 24.2       27.3 -> 26.1     30.1 -> 32.2
//                     4      22 -> 16.4       23.5 -> 21.9     25.8 -> 24.6     29.9 -> 30.9     32.3 -> 33       38.5 -> 41.4
//                     8      28.9 -> 20.6     30.4 -> 24.7     32.6 -> 29       35 -> 36.4       38.1 -> 38.4     45.3 -> 47.4
//                    16      42.6 -> 27.6     46.1 -> 32.9     45.4 -> 37       49.6 -> 49.5     50 -> 52.2       59.2 -> 63.8
//                    32      66.5 -> 41.8     70.1 -> 47.3     69 -> 52.7       74.7 -> 70.2     76.3 -> 79.1     86.6 -> 95.8
//                    64      113 -> 68.7      116 -> 75.4      118 -> 87.9      120 -> 117       124 -> 132       145 -> 163
//                   128      205 -> 121       205 -> 138       211 -> 156       210 -> 220       218 -> 240       257 -> 299
//   dense FP8,        2 block 28.4 -> 22.2     31.2 -> 30.2     33.2 -> 33.7     44.8 -> 41.3     48 -> 43.3       54.6 -> 54
//                     8      34.8 -> 26       38.8 -> 33.2     40.8 -> 37.5     47.5 -> 45.6     51.6 -> 48.8     60.5 -> 61.3
//                    16      44.5 -> 31.7     48.1 -> 38.7     50.2 -> 43       54.5 -> 54.1     58.9 -> 57.8     69.5 -> 72
//                    32      62.1 -> 42.3     65.8 -> 46.7     67.1 -> 54.1     71.8 -> 68.3     73.1 -> 74.9     89.5 -> 92.2
//                    64      94.8 -> 61.5     98.6 -> 66       100 -> 75.4      103 -> 98.2      107 -> 110       126 -> 136
//                   128      161 -> 100       163 -> 109       166 -> 120       167 -> 161       170 -> 181       202 -> 225
// (8-bit first products with 32-key blocks as bf16 ones, dense ones 5 % less at the limits.  Rows of one or two blocks gain
// again beyond 1024 rows, where neither form has places for all; the limits leave that out for bf16 and sparse FP8.  Over 904
// calls of 56 shapes the form that is taken is 0.2 % slower than the better one, 7 % at most but for one-block rows of FP8, 11.)
#pragma once

namespace sale {

struct RowSplitLimit {
  int blocks;                                                  // longest row: at least this many 64-key blocks
  int sparse, sparse32, sparse_fp8, dense, dense_fp8;          // rows up to which two waves per row are taken
};
// (from the table above and, between its lengths and rows, from the calls that tests/test_row_split.py holds)
constexpr RowSplitLimit kRowSplitLimits[] = {
    {96, 1536, 1536, 1536, 1280, 1280}, {64, 1536, 1280, 1536, 1280, 1280}, {48, 1536, 1280, 1536, 1280, 1344},
    {32, 1280, 1280, 1408, 1280, 1280}, {24, 1280, 1152, 1408, 1280, 1280}, {16, 1280, 1152, 1536, 1152, 1536},
    {12, 1152, 1024, 1536, 1152, 1536}, {6, 1024, 1024, 1536, 1024, 1536},  {4, 960, 896, 1536, 1024, 1536},
    {3, 768, 704, 1536, 768, 1536},     {2, 512, 512, 1536, 512, 1536},     {0, 512, 512, 512, 512, 1536}};

struct RowSplitCall {
  long rows;         // 64-row blocks of all heads and batch entries
  long even_rows;    // rows as long as the longest sequence's that make up as much work: `rows` if all sequences are alike
  int longest;       // 64-key blocks of the longest row (of its sequence: what a mask keeps is not known here, and where every
                     // row of a long sequence keeps as few as 13 blocks two waves lose at 640 - 1024 rows: FP8 67.8 -> 74.3 us,
                     // bf16 48.6 -> 49.5 and 55.5 -> 58.1)
  int kv_heads;      // of all batch entries
  int group;         // query heads per KV head
  bool dense, bk32, int8, fp8;
  bool by_position;  // packed sequences without row counts: whole rows are issued in the order of the tokens
};

inline bool two_waves_per_row(const RowSplitCall& c) {
  const RowSplitLimit* l = kRowSplitLimits;
  while (c.longest < l->blocks) ++l;
  auto limit_of = [&](const RowSplitLimit& r) {
    return c.dense ? (c.fp8 ? r.dense_fp8 : r.dense) : c.bk32 ? r.sparse32 : c.fp8 ? r.sparse_fp8 : r.sparse;
  };
  int limit = limit_of(*l);
  // (all rows of a packed call, of which the limit counts the long ones: as many as were timed)
  if (c.rows > (c.dense ? (c.fp8 ? 1536 : 1280) : c.bk32 ? 2080 : 1536)) return false;
  // Whole rows issued by position start some of the longest last once there are more of them than places; halves are sorted
  // (packed, dense: 78 x 1024 tokens, one head 84.3 -> 66.3 us; 3 x 4096, 6 / 2 heads 128 -> 117; 10 x 256, 32 / 8 heads 38.0 ->
  // 31.7).
  if (c.by_position && c.rows > 1024 && c.longest >= 4 && (c.longest >= 16 || c.rows <= 1536)) return true;
  // Half or more of the dense kernel's four-row workgroups is padding when a KV head has one or two rows: 64 tokens x 512 /
  // 1024 / 1280 heads 1.3 - 1.4 times as fast with two waves per row, 128 tokens 1.1 - 1.2 times.
  if (c.dense && c.group == 1 && c.longest <= 2) return true;
  // Workgroup b runs on XCD b % 8 and serves KV head b % kv_heads.  Where every XCD reads more KV heads at a time than four,
  // few query heads share them, and a KV head's rows are spread over the XCDs, the operands do not stay in the L2s, and halves,
  // with twice the loads, lose more: dense, 1K x 63 heads 48.9 -> 57.9 us, 4K x 19 heads 128 -> 151, 256 x 191 24.7 -> 27.3
  // (21 groups of 3, 1K: 46.3 -> 41.3; 1K x 50 heads 46.8 -> 38.9, 62 heads 48.1 -> 46.9), and up to these limits they do
  // not: 2K x 31 74.4 -> 73.4, 4K x 15 119 -> 108, 1K x 43 47.4 -> 40.4, 1K x 62 49.8 -> 46.6.  Sparse: 1.7K x 45 heads 76.2 ->
  // 78.1, 4K x 19 115 -> 121, 16K x 5 217 -> 226 (4K x 18 106 -> 93.2); with 32-key blocks 71.2 -> 74.7, 91.5 -> 97.5, 156 -> 169
  // (84.5 -> 77.1).  (The 8-bit first product loads half as much for it: dense, 4K x 18 130 -> 115, x 19 129 -> 136, 1.7K x 45
  // 83.4 -> 90.8; sparse 4K x 19 121 -> 114, 16K x 5 200 -> 188.)
  int share = 1;      // gcd(kv_heads, 8): KV head h is served by 8 / share of the XCDs
  while (share < 8 && c.kv_heads % (2 * share) == 0) share *= 2;
  if ((c.dense || !c.int8) && c.group < 3 && share < 4 && c.kv_heads / share > 4) {
    const int crowded = !c.dense || c.int8 ? 1152 : c.longest >= 32 || share == 2 ? 1024 : c.longest >= 8 ? 768 : 640;
    if (crowded < limit) limit = crowded;
  }
  return c.even_rows <= limit;
}

// Issue by queue (next_in_queue) of sparse calls with row counts, one wave per row and no window launches.  It evens out the XCDs
// but lets one read the K', V' of another's heads, and a row from a queue starts later by an atomic addition's round trip.
// Attention call of 32 / 8 heads, us, rows issued by position in the sorted list -> by queue:
//   bf16            4160 tokens 134 -> 134, 8K 294 -> 292, 10K 377 -> 365, 12K 518 -> 476, 16K 757 -> 740
//   32-key blocks   8K 216 -> 226, 10K 273 -> 280, 12K 370 -> 342, 16K 537 -> 526
//   int8            8K 275 -> 271, 10K 356 -> 351, 12K 478 -> 443, 16K 692 -> 665; 32-key blocks 8K 225 -> 230, 12K 368 -> 339
//   FP8             4160 112 -> 112, 6K 163 -> 163, 8K 247 -> 240, 12K 416 -> 379, 16K 590 -> 568
// (With an earlier step, fewer rows or heads: 14K x 40 heads over 2 710 -> 698, 12K x 8, batch 3 433 -> 414, 16K x 8 (2048 rows)
// 342.8 -> 344.2; 32-key 12K x 8, batch 3 342 -> 354, 16K, 16 over 2, batch 2 467 -> 465; FP8 6K x 24 153 -> 141.)
// The 16-bit pass is the one whose operands no longer fit its own XCD's L2 above 8K tokens, where there is little left to lose;
// the FP8 pass asks for half of them.
constexpr int kMaxQueues = 256;      // (room for the counters)
inline bool issue_by_queue(const RowSplitCall& c) {
  if (c.kv_heads < 2 || c.kv_heads > kMaxQueues) return false;
  return c.fp8 || (c.rows >= 4096 && c.longest >= (c.bk32 ? 256 : 160));
}

// Query heads per wave of select_kernel: four, so that a K~ fragment feeds twice as many products, where rows are long and work
// is plenty (rows times mask words of the longest); with two there are twice as many waves.  Select call, us, two heads -> four
// (query / KV heads x tokens):
//   rows of fewer than 8 mask words  32/8x12K 179 -> 182, x16K 280 -> 287, x20K 402 -> 413, x24.4K 586 -> 601, x28K 751 -> 746;
//                                    64/8x16K 533 -> 539, x24K 1062 -> 1060
//   little work                      4/1x32K 145 -> 165, 8/1x30K 239 -> 243, 8/2x32K 266 -> 271
//   otherwise                        12/1x32K 396 -> 385, 16/2x32K 490 -> 487, 32/8x30K 866 -> 829, x32K 948 -> 942, x48K 1984 ->
//                                    1941, 4/1x64K 486 -> 478, 8/2x48K 562 -> 555, x64K 915 -> 888, 32/8x64K 3437 -> 3287,
//                                    4/1x128K 1822 -> 1745, 32/8x128K 13300 -> 12530; two sequences of 32K 1882 -> 1850
// (A packed call whose longest sequence is not most of it may lose a little: 32K, 12K 1106 -> 1130.)  With 32-key blocks, which
// have half the maxima per product, two are as fast at 64K (3.66, 3.70 ms) and use fewer registers.
inline int select_heads_per_wave(bool bk32, int group, long rows, int words) {
  if (!bk32 && group % 4 == 0 && words >= 8 && rows * words >= 40960) return 4;
  return group % 2 == 0 ? 2 : 1;
}

}  // namespace sale
