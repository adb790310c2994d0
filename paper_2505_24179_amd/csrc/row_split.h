// Which attention calls run with two waves per row (NT = 1 of attn_rows_kernel).  Host only, plain C++.
//
// A SIMD holds one wave of either form, so 1024 waves run at a time.  Up to 512 rows every half row has a place from the
// start, and the longest row, which is the call, takes about two thirds of the time.  With more rows the rest waits for
// places: what a row costs besides its blocks (start, Q in, O out) is then paid one after the other, twice as often as
// with whole rows, and the operand loads, twice as many per FLOP, begin to count.  So the limit goes by the longest row.
// Attention call, us, one wave per row -> two (group of 4 where the rows allow it; rows of one batch, all alike):
//                        rows  512             768             1024            1280            1536            2048
//   sparse bf16,    1 block    12.5 -> 11.3    14.8 -> 16.7    17.2 -> 18.3    24.3 -> 23.1    25.8 -> 25.7    30.7 -> 30.7
//                   4 blocks   18.0 -> 14.9    21.3 -> 20.0    23.7 -> 23.2    26.9 -> 29.0    30.0 -> 30.8    35.6 -> 39.2
//                   8          21.0 -> 16.3    24.1 -> 22.9    26.8 -> 26.5    29.6 -> 32.8    33.8 -> 35.0    42.7 -> 43.4
//                  16          35.4 -> 24.8    41.2 -> 30.4    41.3 -> 34.1    46.0 -> 43.2    44.8 -> 45.7    53.0 -> 57.4
//                  32          58.1 -> 40.6    63.1 -> 45.8    62.1 -> 48.7    68.2 -> 62.1    72.0 -> 70.8    77.9 -> 88.0
//                  64          98.7 -> 66.1     103 -> 71.1     108 -> 74.5     111 -> 89.0     115 -> 98.1     121 -> 128
//   32-key blocks,  8          21.9 -> 16.6    25.2 -> 22.6    28.0 -> 25.1    31.7 -> 30.7    35.2 -> 32.8    39.8 -> 40.3
//                  16          35.4 -> 24.3    40.8 -> 29.6    40.8 -> 33.1    45.3 -> 42.0    43.7 -> 42.8    50.8 -> 53.3
//                  32          56.5 -> 38.9    60.0 -> 42.1    59.3 -> 43.5    73.2 -> 53.8    75.4 -> 61.0    74.4 -> 75.5
//                  64           103 -> 67.6     105 -> 70.6     108 -> 72.2     109 -> 73.8     113 -> 76.2     116 -> 98.7
//   sparse int8,   16          47.3 -> 36.3    53.6 -> 43.0    55.5 -> 48.4    60.5 -> 57.6    60.4 -> 61.1    70.9 -> 74.4
//                  64           107 -> 74.6     110 -> 77.2     114 -> 81.4     118 -> 95.3     123 -> 104      128 -> 133
//   sparse FP8,     8          39.8 -> 36.4    45.9 -> 46.7    49.6 -> 51.7    55.3 -> 58.9    59.6 -> 61.9    67.6 -> 72.1
//                  16          52.3 -> 45.9    59.9 -> 52.9    62.2 -> 58.8    65.7 -> 67.7    66.5 -> 72.4    76.4 -> 85.9
//                  32          74.2 -> 61.8    79.4 -> 67.1    82.1 -> 73.4    86.4 -> 85.8    88.0 -> 94.3    97.6 -> 114
//   dense bf16,     4          17.8 -> 14.3    20.6 -> 19.7    22.7 -> 22.6    26.6 -> 28.7    28.6 -> 30.6    34.5 -> 38.4
//                   8          25.6 -> 19.1    27.8 -> 22.6    29.8 -> 26.5    30.2 -> 33.2    33.6 -> 36.4    40.3 -> 44.3
//                  16          38.7 -> 26.5    43.2 -> 32.3    43.1 -> 35.3    47.4 -> 47.6    45.9 -> 50.2    54.4 -> 60.1
//                  64           111 -> 73.9     113 -> 81.5     118 -> 90.9     121 -> 120      127 -> 138      144 -> 167
//   dense FP8,     16          54.1 -> 46.1    59.3 -> 52.9    62.7 -> 58.7    66.5 -> 70.3    67.1 -> 75.3    77.8 -> 89.2
//                  64           121 -> 95.2     124 -> 99.6     127 -> 109      130 -> 135      133 -> 153      149 -> 185
// (Dense int8 as dense bf16, at 16 blocks and 1280 rows 63.2 -> 61.9.  The limits end where the form was measured and tested
// first: sparse rows of 64 blocks and more would gain further, 2048 rows of 128 blocks 214 -> 178 us in bf16, 216 -> 199 in FP8.)
#pragma once

namespace sale {

struct RowSplitLimit {
  int blocks;                                                  // longest row: at least this many 64-key blocks
  int sparse, sparse32, sparse_fp8, dense, dense_fp8;          // rows up to which two waves per row are taken
};
// (the last rows at which nine of ten calls of that kind and length were no slower, of 16500 drawn ones with 1 to 64 heads)
constexpr RowSplitLimit kRowSplitLimits[] = {
    {48, 1536, 2080, 1280, 1280, 1024}, {40, 1536, 1920, 1280, 1280, 1024}, {32, 1536, 1792, 1280, 1280, 1024},
    {24, 1408, 1664, 1152, 1280, 1024}, {16, 1280, 1536, 1152, 1280, 1024}, {12, 1216, 1408, 1024, 1024, 1024},
    {8, 960, 1152, 704, 1024, 1024},    {5, 832, 832, 704, 832, 896},       {4, 768, 768, 640, 704, 768},
    {3, 576, 704, 512, 512, 512},       {0, 512, 512, 512, 512, 512}};

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

}  // namespace sale
