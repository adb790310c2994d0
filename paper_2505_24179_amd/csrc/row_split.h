// Which attention calls run with two waves per row (NT = 1 of attn_rows_kernel), which sparse ones of the others take their
// shorter rows from queues, and how many heads a wave of the Selection-Pass takes.  Host only, plain C++.
//
// A SIMD holds one wave of either form, so 1024 waves run at a time.  Up to 512 rows every half row has a place from the
// start, and the longest row, which is the call, takes about two thirds of the time.  With more rows the rest waits for
// places: what a row costs besides its blocks (start, Q in, O out) is then paid one after the other, twice as often as
// with whole rows, and the operand loads, twice as many per FLOP, begin to count.  So the limit goes by the longest row.
// Attention call, us, one wave per row -> two (group of 4 where the rows allow it; rows of one batch, all alike):
//                        rows  512              768              1024             1280             1536             2048
//   sparse bf16,     1 block  14.7 -> 12.8     16.7 -> 19       19.5 -> 21.1     27.5 -> 27.5     29.6 -> 29.8     34.3 -> 35.6
//                    4        18.2 -> 15.1     21.7 -> 22       24.7 -> 24.8     30 -> 31.6       33.4 -> 33.6     38.9 -> 43.2
//                    8        19.8 -> 16.1     22.8 -> 24.4     26 -> 27.8       32.6 -> 35.4     35.9 -> 37.1     44.8 -> 46.7
//                   16        29.4 -> 22.3     35 -> 29.6       35.7 -> 33.6     40.2 -> 43.1     42 -> 45.8       49.2 -> 57.9
//                   32        48.7 -> 36       53.7 -> 42.1     53.1 -> 46.4     58.9 -> 60.4     64.5 -> 66.2     72.4 -> 85.6
//                   64        81.2 -> 57       83.7 -> 63.9     90.1 -> 70.6     95.9 -> 84.4     100 -> 93.8      103 -> 118
//                  128        154 -> 101       -                164 -> 113       -                177 -> 130       184 -> 162
//   32-key blocks,   8 blocks 20 -> 16.5       22.4 -> 23.8     25.5 -> 26       31.8 -> 33.5     34.8 -> 35.2     39.2 -> 43.5
//                   16        28.2 -> 21.7     34.3 -> 29.5     34.4 -> 32.8     39.7 -> 43.4     39.6 -> 44.6     48.1 -> 56.7
//                   32        46.2 -> 34       50.9 -> 38.9     50.3 -> 42.9     61.2 -> 54.7     63.4 -> 61       65.1 -> 75.2
//                   64        82 -> 55.6       84.2 -> 60.2     89.2 -> 63.7     91.3 -> 68.8     94.3 -> 75.5     97.1 -> 94.1
//                  128        155 -> 96.8      -                163 -> 106       -                170 -> 116       176 -> 120
//   sparse int8,    16 blocks 41.4 -> 34.5     47.8 -> 43       50.2 -> 47.6     56.3 -> 58.9     58.6 -> 61.8     68.4 -> 75.2
//                   64        86.5 -> 64.1     89.5 -> 70.8     94.3 -> 76.7     102 -> 91.4      106 -> 101       112 -> 122
//   sparse FP8,      1 block  36.1 -> 33       42.3 -> 42.4     47.1 -> 45.8     59.7 -> 54       61 -> 55.9       67.7 -> 65
//                    8        41.6 -> 35.6     48.2 -> 46.9     52 -> 50.9       60.6 -> 59.8     64.4 -> 62       73.6 -> 73.6
//                   16        52.2 -> 41.8     59.2 -> 51.1     61.6 -> 56.2     65.9 -> 65.6     69.4 -> 69.2     80 -> 81.3
//                   32        68.7 -> 51.7     74.2 -> 57.9     76.6 -> 65       80.5 -> 76.6     81.9 -> 82.3     94.9 -> 98.4
//                   64        98.6 -> 69.8     102 -> 73.3      105 -> 81.5      108 -> 91.4      110 -> 101       119 -> 123
//   dense bf16,      1 block  15.4 -> 12.2     15.9 -> 17.3     18.1 -> 19.9     29 -> 25.1       29.3 -> 27.9     32.7 -> 32.7
//                    4        19.5 -> 14.9     21.7 -> 21.1     24 -> 24         30.5 -> 30.2     31.8 -> 32.3     38.1 -> 41.2
//                    8        23.7 -> 17.6     26.1 -> 23.5     28.5 -> 27.1     33.3 -> 35       36.2 -> 37.1     41.6 -> 46.1
//                   16        33.3 -> 24.1     37.8 -> 31.4     37.7 -> 34.5     42.3 -> 47.9     44.5 -> 49.7     52.6 -> 61
//                   32        54.4 -> 39.2     57.1 -> 45.8     57.6 -> 49.3     62.6 -> 68.6     65.6 -> 77.3     75.9 -> 91.6
//                   64        92.5 -> 65.3     92.9 -> 74.2     101 -> 84.3      105 -> 114       110 -> 130       127 -> 155
//                  128        168 -> 116       -                180 -> 151       -                201 -> 240       232 -> 286
//   dense FP8,      16 blocks 50.8 -> 39.8     59.1 -> 48.9     59.9 -> 54.1     63.1 -> 64.4     67.5 -> 67.7     76.6 -> 80.4
//                   64        99.4 -> 69.8     103 -> 74.9      107 -> 84.9      108 -> 104       111 -> 115       127 -> 138
// (Dense int8 as dense bf16, 5 % less at the limits.  Rows of 128 blocks and more would gain beyond the limits, which end where
// the form was first measured and tested: sparse, 2048 rows 184 -> 162 us in bf16, 178 -> 153 in FP8.)
#pragma once

namespace sale {

struct RowSplitLimit {
  int blocks;                                                  // longest row: at least this many 64-key blocks
  int sparse, sparse32, sparse_fp8, dense, dense_fp8;          // rows up to which two waves per row are taken
};
// (from the table above; between its lengths and rows the figures of the calls that tests/test_row_split.py holds)
constexpr RowSplitLimit kRowSplitLimits[] = {
    {200, 1536, 2080, 1280, 1280, 1152}, {64, 1536, 2080, 1280, 1152, 1152}, {48, 1408, 1920, 1280, 1152, 1152},
    {32, 1152, 1792, 1280, 1152, 1152},  {24, 1088, 1408, 1280, 1088, 1152}, {16, 1024, 1088, 1280, 1024, 1152},
    {12, 832, 832, 1024, 1024, 1152},    {8, 640, 576, 960, 1024, 1152},     {4, 704, 640, 960, 960, 1152},
    {2, 512, 512, 960, 512, 1152},       {0, 512, 512, 512, 512, 512}};

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
  const int most = limit_of(kRowSplitLimits[0]);
  int limit = limit_of(*l);
  if (c.rows > most) return false;
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
  // not: 2K x 31 74.4 -> 73.4, 4K x 15 120 -> 108, 1K x 43 45.8 -> 40.7.  Sparse: 2.1K x 45 heads 92.9 -> 108, 1.7K x 45
  // 71.0 -> 74.7 (6K x 15 heads 175 -> 121).  (The 8-bit first product loads half as much for it and does not lose:
  // 1K x 63 67.3 -> 67.7, 33 KV heads of 2K 91.7 -> 87.8.)
  int share = 1;      // gcd(kv_heads, 8): KV head h is served by 8 / share of the XCDs
  while (share < 8 && c.kv_heads % (2 * share) == 0) share *= 2;
  if (!c.int8 && !c.bk32 && c.group < 3 && share < 4 && c.kv_heads / share > 4) {
    const int crowded =
        !c.dense ? (c.longest >= 48 ? limit : 1280) : c.longest >= 32 ? 1024 : share == 2 ? 896 : c.longest >= 8 ? 768 : 640;
    if (crowded < limit) limit = crowded;
  }
  return c.even_rows <= limit;
}

// Issue by queue (next_in_queue) of sparse calls with row counts, one wave per row and no window launches.  It evens out the XCDs
// but lets one read the K', V' of another's heads, and a row from a queue starts later by an atomic addition's round trip.
// Attention call, us, rows issued by position in the sorted list -> by queue:
//   bf16            4160 x 32 heads 111 -> 112, 8K 264 -> 265, 10K 356 -> 347, 12K 522 -> 461, 16K 750 -> 689; 12K x 8, batch 3
//                   433 -> 414; 14K x 40 heads over 2 KV heads 710 -> 698; 16K x 8 (2048 rows) 342.8 -> 344.2
//   32-key blocks   8K 201 -> 213, 10K 262 -> 271, 12K 379 -> 343, 12K x 8, batch 3 342 -> 354; 16K 538 -> 519, 16 over 2, batch 2
//                   467 -> 465
//   int8            8K 266 -> 260, 10K 346 -> 336, 12K 470 -> 435, 16K 666 -> 624
//   FP8             4160 127 -> 114, 6K x 24 heads 153 -> 141, 8K 260 -> 248, 12K 447 -> 390, 16K 630 -> 570
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
