// Computation-Pass (Sec. 3.1, Eq. 1 with the block mask of Eq. 2) and the dense
// causal kernel of the same design (every causally visible block kept).
//
// Design for gfx950
// -----------------
// * One wave = one unit (query head, 64-row query block) walking its OWN mask
//   row; in calls of few rows the two halves of a unit go to two waves
//   (row_split.h).  The masks of the query heads that share a KV head differ block by
//   block, so staging a tile once for several heads only pays when their bits
//   coincide; instead each wave streams the operands of exactly the blocks its
//   row keeps straight from global memory into MFMA operand registers: no LDS
//   staging, no barriers, a skipped block costs nothing.
// * To make those loads full 1 KB coalesced transactions (and to get V
//   transposed for free) a pre-pass copies K and V once into "fragment order"
//   (layouts at rearrange_kv_kernel).
// * Each wave computes the TRANSPOSED score tile S^T = K Q^T (keys x queries)
//   with v_mfma_f32_16x16x32_bf16: a lane then owns 4 keys of one query column
//   per tile, and the accumulators of two 16-key tiles are, register for
//   register, the B operand of the second product O^T = V^T P^T (up to a
//   permutation of the contraction index that the V copy applies as well), so P
//   never leaves registers.
// * The 16x16x32 shape, because the long calls run at the card's power limit:
//   contracting 32 instead of 16 deep it reads and writes its accumulators half
//   as often per FLOP.  Random operands, matrix stream with exponentials beside
//   it, per SIMD: 48.2 MFLOP x 32768 / us with 32x32x16, 52.9 with 16x16x32; the
//   8-bit product alone 54.8 and 64.7.  (Dense, 32K x 32 heads, in a kernel that
//   took no running maximum: 6.82 -> 6.26 ms.)
// * Softmax in fp32 with exp2 and the scale folded in, against the running
//   maximum of the row; O accumulates in fp32.  The finished bf16 tile is
//   transposed through LDS (each wave its own 17 KB, no barrier) so that it
//   leaves as whole 256-byte rows.
// * Scheduling.  Few rows, dense and sparse: a workgroup is one unit, its two
//   waves take 32 queries each.  Otherwise, dense: a workgroup is 4 successive
//   units of one KV head (with 4 query heads per KV head the same query block:
//   they read the same blocks in step, so three of four loads hit L1).  Longest
//   rows first, workgroups round-robin over KV heads (blockIdx % n_kv_heads: one
//   KV head per XCD / L2 when there are 8).
//   Sparse: row lengths are heavy-tailed (a query block with one weak row keeps
//   everything) and differ between heads, so every unit is its own 64-thread
//   workgroup.  Short sequences: one sweep per row, rows issued by decreasing
//   kept-block count (a counting sort of row_counts), the shorter half from
//   queues where that pays (next_in_queue).  Longer ones: the long
//   rows are swept window by window (a window of K', V' fits an XCD's L2) with
//   their accumulators parked in the workspace in between, every window launch
//   is balanced over the XCDs by a table that moves rows of over-loaded heads to
//   the lanes of under-loaded ones, and the short rows ride at the tail of the
//   window launches (details at launch_sparse_rows and balance_kernel).
#include <type_traits>

#include "pass8.h"
#include "row_split.h"
#include "sale_common.h"

namespace sale {

// Counting sort of the units of each KV head by kept-block count (without row_counts: by the length of the row),
// descending: order[kvh][rank] = unit id (block * group + head-in-group).  One workgroup per KV head.
// slot_of (optional): rows keeping more than long_count blocks draw a parking slot from *slot_counter (cleared by
// the K' / V' copy that precedes this kernel) as long as there are slots; every other row gets -1.
constexpr int kOrderBins = kMaskWordsMax * 64 + 2;
__device__ __forceinline__ void order_units(const Geo& g, int kvh, int* bin, const int32_t* __restrict__ row_counts,
                                            int32_t* __restrict__ order, int32_t* __restrict__ slot_of, int long_count,
                                            int n_slots, int* __restrict__ slot_counter) {
  const int units = g.n_qb * g.group;
  const int max_count = min(g.n_kb, g.words * 64);      // (a row keeps at most the key blocks of its own sequence)
  const int nbins = max_count + 1;
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) bin[b] = 0;
  __syncthreads();
  auto count_of = [&](int id) {
    const int i = id / g.group;
    const int c = row_counts ? row_counts[(size_t)(kvh * g.group + id % g.group) * g.n_qb + i] : seq_pos(g, i).il + 1;
    return min(max(c, 0), max_count);
  };
  for (int id = threadIdx.x; id < units; id += blockDim.x) atomicAdd(&bin[count_of(id)], 1);
  __syncthreads();
  if (threadIdx.x < 64) {          // start offset of every bin, largest count first: lane l has a 64th of the bins
    const int per = (nbins + 63) / 64, hi = nbins - 1 - (int)threadIdx.x * per, lo = max(hi - per + 1, 0);
    int sum = 0;
    for (int b = hi; b >= lo; --b) sum += bin[b];
    int run = sum;
    for (int d = 1; d < 64; d *= 2) { const int o = __shfl_up(run, d, 64); if ((int)threadIdx.x >= d) run += o; }
    run -= sum;
    for (int b = hi; b >= lo; --b) { const int n = bin[b]; bin[b] = run; run += n; }
  }
  __syncthreads();
  for (int id = threadIdx.x; id < units; id += blockDim.x) {
    const int cnt = count_of(id);
    order[(size_t)kvh * units + atomicAdd(&bin[cnt], 1)] = id;
    if (slot_of) {
      int slot = -1;
      if (cnt > long_count && n_slots > 0) {
        slot = atomicAdd(slot_counter, 1);
        if (slot >= n_slots) slot = -1;
      }
      slot_of[(size_t)(kvh * g.group + id % g.group) * g.n_qb + id / g.group] = slot;
    }
  }
}

__global__ __launch_bounds__(1024) void order_units_kernel(Geo g, const int32_t* __restrict__ row_counts,
                                                           int32_t* __restrict__ order, int32_t* __restrict__ slot_of,
                                                           int long_count, int n_slots, int* __restrict__ slot_counter) {
  __shared__ int bin[kOrderBins];
  order_units(g, blockIdx.x, bin, row_counts, order, slot_of, long_count, n_slots, slot_counter);
}

// The same sort as the first workgroups (one per KV head) of the launch of rearrange_kv_kernel, for calls without window
// launches, whose sort needs no slot counter: one launch less
// (attention call: one head of 2K tokens 21.2 -> 18.9 us, 4K x 32 heads 136.3 -> 134.0, 16K 820 -> 815).
constexpr int kQueueStride = 32;      // ints from one queue's counter to the next (see next_in_queue)
struct OrderJob {
  int heads;                      // 0: nothing to sort
  int* taken;                     // cleared: the heads' queues (see next_in_queue)
  const int32_t* row_counts;      // nullptr: rows by their length
  int32_t* order;
};

// Fragment order: what one load instruction of the attention kernel reads is 1 KB in a row.
//   K' [kv head][block j][kt 0..3][s 0..3][lane 0..63]   : 8 channels 32s + 8(lane/16).. of key row 16kt + lane%16
//   V' [kv head][block j][half 0..1][dt 0..7][lane 0..63] : channel 16dt + lane%16 of the 8 keys
//                                                           32half + 16(e/4) + 4(lane/16) + e%4,  e = 0..7
// (the key order inside V' is the order in which the S^T accumulator registers
// hand P^T to the second product).
// K, V: which copies are made.  The 8-bit first product does not read K' and the FP8 second product not V': without the
// copies nobody reads the attention call with int8 takes 1496 instead of 1512 us at 25K, with FP8 7446 instead of 7544
// us at 64K.  (As template parameters: a run-time test kept the loads of V from being in flight with those of K, 28.0
// instead of 27.5 us in the dense call of 1K tokens.)
// Without the copy of K the first pass over the 8-bit operands follows in the same launch, from workgroup `tiles` on.
struct Then8 { int tiles; Pass8 pass; };
struct NoPass8 {};
template <bool K, bool V>
__global__ __launch_bounds__(256) void rearrange_kv_kernel(Geo g, OrderJob job, std::conditional_t<K, NoPass8, Then8> then,
                                                           const uint16_t* __restrict__ k,
                                                           const uint16_t* __restrict__ v,
                                                           u32x4* __restrict__ kp, u32x4* __restrict__ vp,
                                                           int* __restrict__ slot_counter) {
  __shared__ union { uint16_t sv[64 * (kHeadDim + 2)]; int bin[kOrderBins]; double pass[128]; } lds;
  if ((int)blockIdx.x < job.heads) {
    if (job.taken && threadIdx.x == 0) job.taken[kQueueStride * blockIdx.x] = 0;
    order_units(g, blockIdx.x, lds.bin, job.row_counts, job.order, nullptr, 0, 0, nullptr);
    return;
  }
  uint16_t* const sv = lds.sv;
  const int block = (int)blockIdx.x - job.heads, seq = g.seq;
  if constexpr (!K)
    if (block >= then.tiles) { then.pass.run(g, block - then.tiles, lds.pass); return; }
  const Strided &lk = g.sk, &lv = g.sv;
  const int tid = threadIdx.x;
  if (slot_counter && block == 0 && tid == 0) *slot_counter = 0;      // (for order_units_kernel, next on the stream)
  const size_t tile = block;                           // flattened (kv head, block j): rows tile*64 .. +63
  const int tiles_per_head = seq / 64;
  const uint16_t* kt = k + row_off(lk, (int)(tile / tiles_per_head), (int)(tile % tiles_per_head) * 64);
  const uint16_t* vt = v + row_off(lv, (int)(tile / tiles_per_head), (int)(tile % tiles_per_head) * 64);
#pragma unroll
  for (int r = 0; r < (V ? 4 : 0); ++r) {
    const int chunk = tid + 256 * r;                   // V tile -> LDS, rows padded by one bank
    const int row = chunk >> 4, col = (chunk & 15) * 8;
    const u32x4 w = *(const u32x4*)(vt + (size_t)row * lv.st + col);
    uint32_t* d = (uint32_t*)&sv[row * (kHeadDim + 2) + col];
    d[0] = w[0]; d[1] = w[1]; d[2] = w[2]; d[3] = w[3];
  }
#pragma unroll
  for (int r = 0; r < (K ? 4 : 0); ++r) {
    const int oc = tid + 256 * r;
    const int lane = oc & 63, s = (oc >> 6) & 3, kt16 = oc >> 8;
    kp[tile * 1024 + oc] = *(const u32x4*)(kt + (size_t)(16 * kt16 + (lane & 15)) * lk.st + 32 * s + 8 * (lane >> 4));
  }
  if constexpr (!V) return;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int oc = tid + 256 * r;
    const int lane = oc & 63, dt = (oc >> 6) & 7, half = oc >> 9;
    const int d = 16 * dt + (lane & 15), grp = lane >> 4;
    uint32_t w[4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      const int e = 2 * e2;
      const int key = 32 * half + 16 * (e >> 2) + 4 * grp + (e & 3);
      w[e2] = (uint32_t)sv[key * (kHeadDim + 2) + d] | ((uint32_t)sv[(key + 1) * (kHeadDim + 2) + d] << 16);
    }
    u32x4 out;
    out[0] = w[0]; out[1] = w[1]; out[2] = w[2]; out[3] = w[3];
    vp[tile * 1024 + oc] = out;
  }
}

// Which rows a launch handles and which part of them.  win_word < 0: the whole row in one go.
// win_word >= 0: only the key blocks of that 64-block mask word; a row then resumes from the state
// (fp32 O^T accumulators, running max and sum, exactly the register contents) that the launch of the
// previous word parked in its slot of the workspace, and parks it again unless this word holds its diagonal block.
// slot_of (window launches): the parking slot of every row block, or -1 for the rows that are swept whole: the
// short ones, and the long ones that found no slot in the caller's workspace.
// Workgroups from number tail_from on (tail_from >= 0) form the tail of a window launch: they take the
// rows without a slot, whole, rank tail_phase + k * tail_stride of each KV head's
// sorted list, so that every window launch ends with its share of short rows and its last long rows do
// not leave the chip idle.
struct RowFilter {
  const int32_t* slot_of;
  int win_word;    // first mask word of the window, or < 0
  int win_words;   // words per window
  int tail_from, tail_stride, tail_phase;
  int* taken;           // issue by queue (below): rows taken from each KV head's queue; nullptr: rows as they come
  int queue_from;       // first rank in the queues
};

// order: optional [kv head][rank] -> unit id within the KV head (block * group + head-in-group).
// BK32: the mask has one bit per 32 keys (b_k = 32) instead of one per 64.  The kernel always works on
// pairs of 32-key half-tiles; with b_k = 64 a pair is the two halves of one block, with b_k = 32 it is any
// two kept half-tiles of the row (the operand copies K', V' are addressable by half-tile).
// QK8: the first product runs on the 8-bit operands of the quantized Computation-Pass (Sec. 3.4 "Integration
// with SageAttention") with v_mfma_i32_16x16x64_i8 (PV8: 32x32x32): half the K bytes and half the MFMA time of that product.
struct Qk8 {
  const int8_t* q8;       // [q head][N][128]
  const u32x4* k8p;       // fragment order, 8 KB per 64 keys
  const float* q_scale;   // [q head][N / 64]
  const float* k_scale;   // [kv head][N / 64]
  const float* k_mean;    // [kv head][128]: the mean key taken out of K before quantization
  const u32x4* v8p;       // FP8 V in fragment order, 8 KB per 64 keys (PV8 only)
  const float* v_scale;   // [kv head][128] (PV8 only)
};
// PV8 (with QK8, 64-key blocks): the second product in FP8 with v_mfma_f32_32x32x64_f8f6f4 - a quarter of the V
// bytes and half the MFMA time of that product; see the PV8 section of the kernel.
constexpr float kIntOffset = 12582912.0f;            // 1.5 * 2^23, bit pattern 0x4B400000 (see qk_mfma)

// The matrix stream of one phase of the pipeline (see the kernel): nq MFMAs of the first product (kind 0), whose scores the
// second half of the phase then looks at, np of the second (kind 1), and the row sums (kind 2).
struct PhaseStep { int kind, n; };
constexpr PhaseStep phase_step(int i, int nq, int np) {
  return i < nq ? PhaseStep{0, i} : i < nq + np ? PhaseStep{1, i - nq} : PhaseStep{2, i - nq - np};
}
// The same for a step of the FP8 pass: np MFMAs of the second product (kind 1), 64 cycles each, nt of the row sums (kind 2)
// and nq of the first product (kind 0), 32 cycles each.  fp8_upto: how many of `ops` vector instructions are issued by the end
// of step i, in proportion to time: from the third MFMA on (the last scores are still on their way) until the first product
// turns to the second query tile, whose old scores are then used up (with both sets of scores the step spills).
constexpr PhaseStep fp8_step(int i, int nq, int np, int nt) {
  const int per = np / nt + 1;      // products and sum of one query tile
  return i >= np + nt ? PhaseStep{0, i - np - nt} : i % per == per - 1 ? PhaseStep{2, i / per} : PhaseStep{1, i - i / per};
}
constexpr int fp8_upto(int i, int nq, int np, int nt, int ops) {
  const int lead = 4, span = nt == 2 ? nq / 2 : nq, total = 2 * np + nt + span - lead;      // (in 32 cycles)
  int done = -lead;
  for (int k = 0; k <= i; ++k) done += fp8_step(k, nq, np, nt).kind == 1 ? 2 : 1;
  return done <= 0 ? 0 : done >= total ? ops : (ops * done + total - 1) / total;
}

// Issue by queue (calls without window launches; see issue_by_queue for which).  Workgroups go to the XCDs round-robin, so with
// lane = KV head every XCD has the rows of its own heads, and these keep different numbers of blocks: at 16K tokens x 32 heads
// the XCDs had finished after 690 .. 887 us.  The longer half of a head's sorted rows is issued as before; the rows of rank
// queue_from .. are a queue, from which a workgroup takes the next row of its own head (whose K', V' its XCD's L2 holds) or,
// when there is none left, of the head with the most rows left.  The grid has more workgroups than rows, so that an XCD that
// is done early has some left; those that find nothing only read the counters.  A counter has 128 bytes of its own: next to
// each other the additions of all XCDs went one by one, and the call took 20 % longer.
// Attention call, without -> with: 16K x 32 heads bf16 757 -> 740 us, int8 692 -> 665, FP8 590 -> 568; 12K 518 -> 476, 478 -> 443,
// 416 -> 379.
__device__ __forceinline__ int next_in_queue(const RowFilter& flt, int n_kvh, int units, int lane, bool own, int& kvh) {
  const int n = units - flt.queue_from;
  for (;; own = true) {      // (a queue found empty stays empty: at most once per head)
    if (own) {
      int r = 0;
      if (lane == 0) r = atomicAdd(&flt.taken[kQueueStride * kvh], 1);
      r = __builtin_amdgcn_readfirstlane(r);
      if (r < n) return flt.queue_from + r;
    }
    int least = n, at = 0;
    for (int h = lane; h < n_kvh; h += 64) {
      const int t = __hip_atomic_load(&flt.taken[kQueueStride * h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (t < least) { least = t; at = h; }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const int l = __shfl_xor(least, off, 64), a = __shfl_xor(at, off, 64);
      if (l < least || (l == least && a < at)) { least = l; at = a; }
    }
    least = __builtin_amdgcn_readfirstlane(least);
    if (least >= n) return units;
    kvh = __builtin_amdgcn_readfirstlane(at);
  }
}

// NT: 32-query tiles per wave.  NT = 2: one wave per row (or WAVES rows per workgroup).  NT = 1 (WAVES = 1, no window
// launches): the two waves of a workgroup take 32 queries each of ONE row: half the MFMAs and half the softmax per wave
// and key block, the same operand loads (the second wave of a row hits in L1).  Both forms run one wave per SIMD: 268 - 304
// registers (bf16 304, int8 268, FP8 270) against 393 - 449, where two waves would need 256 or less.  So a row gains because
// its work is on two SIMDs, not because one wave covers the other's latency.  A query's arithmetic is the same in both, bit
// for bit.
template <int WAVES, bool BK32, bool QK8, bool PV8 = false, int NT = 2>
__global__ __launch_bounds__(WAVES * (2 / NT) * 64) void attn_rows_kernel(Geo g, const uint16_t* __restrict__ q,
                                                               const bf16x8* __restrict__ kp,
                                                               const bf16x8* __restrict__ vp, Qk8 q8o,
                                                               const uint64_t* __restrict__ mask,
                                                               const int32_t* __restrict__ order,
                                                               const int32_t* __restrict__ assign,
                                                               uint16_t* __restrict__ o, float* __restrict__ o32,
                                                               float* __restrict__ lse,
                                                               RowFilter flt, f32x4* __restrict__ st_o,
                                                               float* __restrict__ st_ml) {
  static_assert(NT == 2 || WAVES == 1, "the two halves of a row share a workgroup of their own");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);      // (wave-uniform by construction: the unit and its addresses are scalars)
  const int wave = NT == 1 ? 0 : wave_id;
  const int q0 = NT == 1 ? wave_id * 32 : 0;      // first query of this wave inside the row block
  constexpr int NQ = 2 * NT;                      // 16-query tiles of this wave
  const int c = lane & 31, h = lane >> 5;         // column and row group of a lane in a 32x32 tile (PV8)
  const int n16 = lane & 15, g16 = lane >> 4;     // ... in a 16x16 tile
  const int units = g.n_qb * g.group;
  Unit u;
  const bool tail = WAVES == 1 && flt.tail_from >= 0 && (int)blockIdx.x >= flt.tail_from;
  {
    const int b = tail ? (int)blockIdx.x - flt.tail_from : (int)blockIdx.x;
    u.kvh = b % g.n_kvh;
    int rank = tail ? (b / g.n_kvh) * flt.tail_stride + flt.tail_phase : (b / g.n_kvh) * WAVES + wave;
    if (WAVES == 1 && NT == 2 && flt.taken && rank >= flt.queue_from) {
      rank = __builtin_amdgcn_readfirstlane(next_in_queue(flt, g.n_kvh, units, lane, rank < units, u.kvh));
      u.kvh = __builtin_amdgcn_readfirstlane(u.kvh);
    }
    u.valid = rank < units;
    int id = !u.valid ? 0 : (order ? order[(size_t)u.kvh * units + rank] : units - 1 - rank);
    if (assign && !tail) {
      // balanced issue: slot `rank` of lane blockIdx % n_kvh holds a unit of ANY KV head (or nothing)
      const int entry = u.valid ? assign[(size_t)u.kvh * units + rank] : -1;
      u.valid = entry >= 0;
      u.kvh = u.valid ? entry / units : 0;
      id = u.valid ? entry % units : 0;
    }
    u.i = id / g.group;
    u.qh = u.kvh * g.group + id % g.group;
  }
  if (!u.valid) return;
  const size_t unit_flat = (size_t)u.qh * g.n_qb + u.i;
  const int slot = flt.slot_of ? flt.slot_of[unit_flat] : -1;
  if (tail && slot >= 0) return;      // (rows with a slot are swept window by window through the tables)

  // ---- this wave's list of kept blocks: the set bits of its mask row, below the diagonal ----
  const uint64_t* mrow = mask ? mask + ((size_t)u.qh * g.n_qb + u.i) * g.words : nullptr;
  const SeqPos sp = seq_pos(g, u.i);                // (variable-length batches: block indices inside the row's sequence)
  const int il = sp.il;
  const int j_last = BK32 ? 2 * il + 1 : il;        // last causally visible mask bit of the row
  const int last_word = j_last >> 6;
  const int win_word = tail ? -1 : flt.win_word;
  if (win_word > last_word) return;
  const int word_lo = win_word >= 0 ? win_word : 0;
  const int word_hi = win_word >= 0 ? min(win_word + flt.win_words - 1, last_word) : last_word;
  const bool park = win_word >= 0 && word_hi < last_word;
  auto row_word = [&](int wc) -> uint64_t {
    const int lo = wc * 64;
    const uint64_t causal = j_last >= lo + 63 ? ~0ull : ((2ull << (j_last - lo)) - 1ull);
    return mrow ? (mrow[wc] & causal) : causal;
  };
  // A row takes part only in the windows where it keeps a block (and in its last one): it resumes iff an
  // earlier window held one of its blocks.
  bool resume = false;
  if (win_word > 0) {
    const uint64_t nonzero = __builtin_amdgcn_ballot_w64(lane < word_lo && row_word(lane) != 0ull);
    resume = nonzero != 0ull;
  }

  constexpr int kRowPad = kHeadDim + 8;      // bf16 elements per LDS row of the staged output
  __shared__ __attribute__((aligned(16))) uint16_t o_lds[WAVES * 64 * kRowPad];

  // ---- operands -----------------------------------------------------------------------
  // Q fragments (B operand of S^T = K Q^T), resident for the whole row: query n16 of tile qt, channels 32 s + 8 g16 ..
  // (8-bit: 64 s + 16 g16 ..).
  bf16x8 qf[QK8 ? 1 : NQ][QK8 ? 1 : 4];
  i32x4 qf8[QK8 ? (PV8 ? NT : NQ) : 1][QK8 ? (PV8 ? 4 : 2) : 1];
  if constexpr (PV8) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int8_t* row = q8o.q8 + ((size_t)u.qh * g.seq + u.i * 64 + q0 + 32 * nt + c) * kHeadDim + 16 * h;
#pragma unroll
      for (int s = 0; s < 4; ++s) qf8[nt][s] = *(const i32x4*)(row + 32 * s);
    }
  } else {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      if constexpr (QK8) {
        const int8_t* row = q8o.q8 + ((size_t)u.qh * g.seq + u.i * 64 + q0 + 16 * qt + n16) * kHeadDim + 16 * g16;
#pragma unroll
        for (int s = 0; s < 2; ++s) qf8[qt][s] = *(const i32x4*)(row + 64 * s);
      } else {
        const uint16_t* row = q + row_off(g.sq, u.qh, u.i * 64 + q0 + 16 * qt + n16) + 8 * g16;
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[qt][s] = *(const bf16x8*)(row + 32 * s);
      }
    }
  }
  const float cs = 0.08838834764831845f * 1.4426950408889634f;   // log2(e) / sqrt(d)
  // Logits are handled in log2 units: x = (raw product) * cl[slot], cl = log2(e) / sqrt(d), times the
  // scales of the 8-bit operands of the slot's key block when QK8.
  float sq_cs = cs;
  const int first_tile = __builtin_amdgcn_readfirstlane((int)((size_t)u.kvh * g.seq / 64) + (u.i - il));
  const int tiles = __builtin_amdgcn_readfirstlane(il) + 1;      // (64-key tiles up to the diagonal)
  const int lane16 = lane * 16;
  __amdgpu_buffer_rsrc_t k8t;
  const float* ks8 = nullptr;
  if constexpr (QK8) {
    sq_cs = q8o.q_scale[unit_flat] * cs;
    k8t = operand_buffer(q8o.k8p + (size_t)first_tile * 512, tiles * 8192);      // 512 16-byte chunks per 64 keys
    ks8 = q8o.k_scale + first_tile;
  }
  // (the sequence's first key tile: u.i - il 64-row blocks into the KV head)
  const __amdgpu_buffer_rsrc_t kt = operand_buffer(kp + (size_t)first_tile * 1024, tiles * 16384);     // 1024 16-byte chunks per 64 keys
  const __amdgpu_buffer_rsrc_t vt = PV8 ? operand_buffer(q8o.v8p + (size_t)first_tile * 512, tiles * 8192)
                                        : operand_buffer(vp + (size_t)first_tile * 1024, tiles * 16384);
  f32x16 oacc[PV8 ? 4 : 1][PV8 ? NT : 1];      // PV8: O^T in 32x32 tiles
  f32x4 o16[PV8 ? 1 : 8][PV8 ? 1 : NQ];        // otherwise: O^T in 16x16 tiles, channels 16 dt + 4 g16 .. of query n16 of tile qt
  float m_run[NQ], l_run[NQ];      // m_run in log2 units (PV8: [nt])
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) { m_run[qt] = PV8 ? -INFINITY : -1e30f; l_run[qt] = 0.0f; }
  if constexpr (PV8) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][nt][r] = 0.0f;
  } else {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
        for (int r = 0; r < 4; ++r) o16[dt][qt][r] = 0.0f;
  }

  if constexpr (NT == 2) if (resume) {
    const f32x4* so = st_o + (size_t)slot * 2048 + lane;       // 32 chunks of [lane] 16 bytes
    const float* sml = st_ml + (size_t)slot * 256;             // PV8: [m nt0, m nt1, l nt0, l nt1][lane]; otherwise [m, l][query]
    if constexpr (PV8) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            const f32x4 w = so[((dt * 2 + nt) * 4 + qd) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) oacc[dt][nt][4 * qd + e] = w[e];
          }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) { m_run[nt] = sml[64 * nt + lane]; l_run[nt] = sml[128 + 64 * nt + lane]; }
    } else {
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) o16[dt][qt] = so[(dt * NQ + qt) * 64];
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) { m_run[qt] = sml[16 * qt + n16]; l_run[qt] = sml[128 + 16 * qt + n16]; }
    }
  }
  // ---- the row's kept blocks, in ascending order, as a list in LDS (this wave's part of the output staging area) ----
  // BK32: with an odd number of kept half-tiles the first one comes twice, the first time emptied, so that there are whole
  // pairs and the half-tiles of the diagonal block, the largest indices of a row, fall into the last one.
  uint16_t* const list = o_lds + (wave * 64 + q0) * kRowPad;
  static_assert(32 * NT * kRowPad >= kMaskWordsMax * 64 + 16, "the list of the longest row fits the staging area");
  constexpr bool kListed = WAVES == 1;          // (the four-row workgroups are the dense kernel's: every block)
  int n_pairs = 0;
  bool lone = false;
  auto build_list = [&](int lo, int hi) {
    const uint64_t mine = lane >= lo && lane <= hi ? row_word(lane) : 0ull;
    lone = BK32 && (__popcll(__builtin_amdgcn_ballot_w64((__popcll(mine) & 1) != 0)) & 1) != 0;
    int n = lone ? 1 : 0, first = -1, last = 0;
    for (uint64_t any = __builtin_amdgcn_ballot_w64(mine != 0ull); any != 0ull; any &= any - 1) {
      const int w = __builtin_ctzll(any);
      const uint64_t word = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, w) |
                            (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), w) << 32;
      const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(word >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)word, 0));
      if ((word >> lane) & 1) list[n + before] = (uint16_t)(w * 64 + lane);
      if (first < 0) first = w * 64 + __builtin_ctzll(word);
      last = w * 64 + 63 - __builtin_clzll(word);
      n += __popcll(word);
    }
    if (lone && lane == 0) list[0] = (uint16_t)first;
    if (lane < 8) list[n + lane] = (uint16_t)last;      // (the loads run up to two pairs ahead, the list is read three ahead)
    n_pairs = BK32 ? n >> 1 : n;
    wave_exchange();
  };
  auto entry = [&](int n) __attribute__((always_inline)) -> uint32_t {      // of pair n
    if constexpr (!kListed) return (uint32_t)min(n, tiles - 1);
    else if constexpr (BK32) return (uint32_t)list[2 * n] | (uint32_t)list[2 * n + 1] << 16;      // (one load)
    else return list[n];
  };
  if constexpr (PV8) {
    // ---- fully quantized pass: 8-bit first product, FP8 second product ---------------------------------
    // S^T = K8 Q8^T (16 MFMAs per 64-key block), causal mask on the diagonal block, ONE row maximum over the block's 64 keys,
    // rescale, P8 = fp8(448 * exp2(x - m)) packed straight into the B operand of the FP8 MFMA (a lane's 16 + 16 accumulator
    // values of the two half-tiles are its 32 contraction elements; the V8' copy is in the same key order),
    // O^T += V8^T P8^T (8 MFMAs, K = 64).  The row sums are MFMAs with ones in 16 rows of the A operand per query tile:
    // numerator and denominator are then sums of the SAME rounded probabilities.
    // The definition takes a running maximum block by block, so a step cannot do without it; but the products of its
    // neighbours run meanwhile: step t is  O += V8(t - 1) P8(t - 1), the row sums, S(t + 1) = K8(t + 1) Q8  on the matrix unit,
    // beside the maximum and the exponentials of S(t) on the vector unit, laid side by side as in `phase` below; operands are
    // requested again, for the next step, by the MFMA that has read them.  A row maximum that grew is applied to O at the end
    // of the step, before P8(t) is multiplied.  (One block after the other a step was its 1152 MFMA cycles plus about 2000 of
    // vector instructions.)
    static_assert(QK8 && !BK32, "the FP8 second product comes with the 8-bit first product on 64-key blocks");
    const float kLog2Top = 8.807354922057604f;      // log2(448)
    constexpr int kQ8 = 8 * NT, kP8 = 4 * NT, kTileOps = 106, kOps = kTileOps * NT;
    i32x4 k8[2][4];
    u32x4 v8[4][2];
    i32x16 S[2][NT];         // [half-tile][query tile]: the integer accumulators, as in the QK8 pass below
    // Row sums: the B operand of the 32x32x64 product, read as that of a 16x16x128 one, holds in lane l keys of query l % 32 as
    // column l % 16, contraction group l / 16.  A operand for query tile nt: row i is 1 (E4M3: 0x38) in the groups of parity
    // i / 4 % 2 if i / 8 == nt.  Lane (c, h) then gets, in all four registers, the sum of query c of tile h over both lane halves.
    i32x8 P8[NT], rows_of[NT];
    f32x4 lacc;
#pragma unroll
    for (int r = 0; r < 4; ++r) lacc[r] = h == 0 ? l_run[0] : l_run[NT - 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int w = 0; w < 8; ++w) rows_of[nt][w] = (n16 >> 2 & 1) == (g16 & 1) && n16 >> 3 == nt ? 0x38383838 : 0;
      asm("" : "+a"(rows_of[nt]));
    }
    i32x16 magic;
#pragma unroll
    for (int r = 0; r < 16; ++r) magic[r] = 0x4B400000;
    auto qk8 = [&](int n) __attribute__((always_inline)) {      // MFMA n of S = K8 Q8^T
      const int nt = n / 8, s = n / 2 % 4, mt = n % 2;
      S[mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(k8[mt][s], qf8[nt][s], s == 0 ? magic : S[mt][nt], 0, 0, 0);
    };
    auto pv8 = [&](int n) __attribute__((always_inline)) {      // MFMA n of O^T += V8^T P8^T
      const int dt = n % 4, nt = n / 4;      // (a query tile at a time: the registers of its probabilities are the next step's)
      i32x8 va;
#pragma unroll
      for (int w = 0; w < 4; ++w) { va[w] = (int)v8[dt][0][w]; va[4 + w] = (int)v8[dt][1][w]; }
      oacc[dt][nt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, P8[nt], oacc[dt][nt], 0, 0, 0, 0, 0, 0);
    };
    auto sum8 = [&](int nt) __attribute__((always_inline)) {
      lacc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(rows_of[nt], P8[nt], lacc, 0, 0, 0, 0, 0, 0);
    };
    auto load_k8 = [&](int j, int mt, int s) __attribute__((always_inline)) { k8[mt][s] = load_chunk<i32x4>(k8t, lane16, j * 8192, mt * 4 + s); };
    auto load_v8 = [&](int j, int dt, int jj) __attribute__((always_inline)) { v8[dt][jj] = load_chunk<u32x4>(vt, lane16, j * 8192, dt * 2 + jj); };
    auto hide8 = [&]() __attribute__((always_inline)) {           // the diagonal block: keys after the query
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int seen = q0 + 32 * nt + c - 4 * h;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (32 * mt + 8 * (r >> 2) + (r & 3) > seen) S[mt][nt][r] = (int)0xFF800000;
      }
    };
    float m_new[NT];
    // One step: k_scale of the block whose scores are in S; blocks to request K8 and V8 of.  Returns whether
    // some row's maximum grew: O, the sums and m_run are then to be rescaled before the next step.
    auto step8 = [&](float k_scale, int k_next, int v_next) __attribute__((always_inline)) -> bool {
#pragma clang fp contract(off)      // (every copy of the step rounds alike)
      const float cj = k_scale * sq_cs;              // raw integer product -> logit in log2 units
      const float off = kIntOffset * cj;             // what the accumulators' offset amounts to in logit units
      float most[NT], mx[NT], mb[NT], over[NT], up[NT], E[NT][32];
      f32x16 F[NT][2];
      int top[NT][2];
      i32x8 P_new[NT];
      i32x16 now[2][NT];      // the scores of this step (the first product writes S meanwhile)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) now[mt][nt] = S[mt][nt];
      // The VALU stream, per query tile: 16 maxima in two chains (of integers: with the offset all scores are positive floats
      // of one exponent, hidden ones negative), the row maximum, then five instructions per two scores as in `phase`.
      // The base mb has the size of the accumulators' offset, so it is rounded in steps of about cj: with large scales
      // (outliers in K) the largest probability would come out above 464, which is NaN in FP8, and a query's NaN would reach
      // the sums of the queries that share its column there (0 x NaN).  A base that lets it is moved up to where it does not.
      auto valu = [&](int n) __attribute__((always_inline)) {
#pragma clang fp contract(off)
        const int nt = n / kTileOps, o = n % kTileOps;
        if (o < 16) {
          auto max3 = [](int a, int b, int w) { return max(max(a, b), w); };
          const int mt = o % 2, i = o / 2;
          if (i == 0) top[nt][mt] = max3(now[mt][nt][0], now[mt][nt][1], now[mt][nt][2]);
          else if (i < 7) top[nt][mt] = max3(top[nt][mt], now[mt][nt][2 * i + 1], now[mt][nt][2 * i + 2]);
          else if (mt == 0) top[nt][0] = max3(top[nt][0], now[0][nt][15], now[1][nt][15]);
          else top[nt][0] = max(top[nt][0], top[nt][1]);
        } else if (o == 16) {
          most[nt] = max_with_other_half(int_bits_as_float(top[nt][0]));
          mx[nt] = __builtin_fmaf(most[nt], cj, -off);
        } else if (o == 17) {
          m_new[nt] = fmaxf(m_run[nt], mx[nt]);
          mb[nt] = m_new[nt] - kLog2Top + off;       // exp2(x - m) * 448, x = (S - offset) * cj
        } else if (o == 18) {
          over[nt] = __builtin_fmaf(most[nt], cj, -mb[nt]);
        } else if (o == 19) {
          up[nt] = __builtin_fmaf(mb[nt], 1.0f + 0x1p-23f, over[nt] - kLog2Top);      // (at least mb + (over - log2 448), however it is rounded)
        } else if (o == 20) {
          mb[nt] = over[nt] > 8.85f ? up[nt] : mb[nt];      // (2^8.85 = 461)
        } else {
          const int q = o - 21, e0 = 2 * (q / 5), k = q % 5;
          const int e = k == 0 ? e0 : k == 1 ? e0 - 1 : k == 2 ? e0 + 1 : k == 3 ? e0 : e0 - 2;
          if (e < 0 || e >= 32) return;
          if (k == 0 && e % 16 == 0) F[nt][e / 16] = int_bits_as_floats(now[e / 16][nt]);
          if (k == 0 || k == 2) E[nt][e] = __builtin_fmaf(F[nt][e / 16][e % 16], cj, -mb[nt]);
          else if (k == 1 || k == 3) E[nt][e] = __builtin_amdgcn_exp2f(E[nt][e]);
          else P_new[nt][e / 4] = e % 4 == 0 ? __builtin_amdgcn_cvt_pk_fp8_f32(E[nt][e], E[nt][e + 1], any_int(), false)
                                             : __builtin_amdgcn_cvt_pk_fp8_f32(E[nt][e], E[nt][e + 1], P_new[nt][e / 4], true);
        }
      };
      static_for<kQ8 + kP8 + NT>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        constexpr PhaseStep st = fp8_step(i, kQ8, kP8, NT);
        if constexpr (st.kind == 1) {
          pv8(st.n);
          if constexpr (st.n >= 4 * (NT - 1)) { load_v8(v_next, st.n % 4, 0); load_v8(v_next, st.n % 4, 1); }
        } else if constexpr (st.kind == 2) {
          sum8(st.n);
        } else {
          qk8(st.n);
          if constexpr (st.n >= 8 * (NT - 1)) load_k8(k_next, st.n % 2, st.n / 2 % 4);
        }
        constexpr int from = i == 0 ? 0 : fp8_upto(i - 1, kQ8, kP8, NT, kOps), to = fp8_upto(i, kQ8, kP8, NT, kOps);
        static_for<to - from>([&](auto vc) __attribute__((always_inline)) { valu(from + decltype(vc)::value); });
        __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) P8[nt] = P_new[nt];
      return __builtin_expect_with_probability(__builtin_amdgcn_ballot_w64(mx[0] > m_run[0] || mx[NT - 1] > m_run[NT - 1]) != 0ull, 0, 0.999);
    };
    auto rescale8 = [&]() __attribute__((always_inline)) {
      float alpha[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        alpha[nt] = __builtin_amdgcn_exp2f(m_run[nt] - m_new[nt]);
        m_run[nt] = m_new[nt];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[dt][nt][r] *= alpha[nt];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) lacc[r] *= h == 0 ? alpha[0] : alpha[NT - 1];
    };
    auto block_of = [&](uint32_t raw) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane((int)raw); };

    if constexpr (kListed) build_list(word_lo, word_hi); else n_pairs = tiles;
    asm("" : "+v"(n_pairs));      // (in a vector register for the register allocator's sake: see the other passes)
    if (n_pairs > 0) {
      int j0 = block_of(entry(0)), j1 = block_of(entry(1));      // blocks of this step and the next
      uint32_t ahead = entry(2);
      float s0 = ks8[j0], s1 = ks8[j1];
#pragma unroll
      for (int n = 0; n < 8; ++n) load_k8(j0, n / 4, n % 4);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int w = 0; w < 8; ++w) P8[nt][w] = 0;      // (the first step multiplies by zero)
#pragma unroll
      for (int n = 0; n < 8; ++n) v8[n / 2][n % 2] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int n = 0; n < kQ8; ++n) qk8(n);
#pragma unroll
      for (int n = 0; n < 8; ++n) load_k8(j1, n / 4, n % 4);
      // (an inner loop that a grown maximum leaves: with the rescaling inside it the compiler moves O^T about in every step)
      for (int n = 1; n < n_pairs;) {
        bool grew = false;
        while (n < n_pairs && !grew) {
          const int j2 = block_of(ahead);
          const float s2 = ks8[j2];
          ahead = entry(n + 2);
          grew = step8(s0, j2, block_of((uint32_t)j0));
          j0 = j1; j1 = j2; s0 = s1; s1 = s2;
          ++n;
        }
        if (grew) rescale8();
      }
      j0 = block_of((uint32_t)j0);
      if (j0 == tiles - 1) hide8();
      if (step8(s0, j0, j0)) rescale8();
#pragma unroll
      for (int n = 0; n < kP8; ++n) pv8(n);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) sum8(nt);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) l_run[nt] = __shfl(lacc[0], c + 32 * nt, 64);      // (the sum of query c of tile nt, in both halves)
  } else {
  // ---- one sweep over the row's kept half-tiles ----------------------------------------------------------
  // A software pipeline over half-tiles (32 keys x all queries of the wave), two of them (a pair) per iteration.  Phase t
  //   S(t + 1) = K(t + 1) Q^T       MFMA
  //   O += V(t - 1)^T P(t - 1)^T    MFMA, and the row sums of P(t - 1)
  //   P(t) = exp2(S(t) - maximum)   VALU, and the largest of the scores S(t + 1)
  //   loads of K(t + 3), V(t + 1) into the registers that the two products have just read
  // has no branch and no dependency between its three streams, so that they are laid side by side by hand: micro-group i is
  // one MFMA, its share of the VALU stream and of the loads, closed by a scheduling barrier.  (A wave alone on its SIMD
  // issues one vector instruction inside the 16 cycles of an MFMA for free, two for 4 cycles more; a phase asks for 1.5.)
  // Between two phases one test: has some row of S(t + 1) grown beyond its maximum?  Then the maximum is raised before
  // P(t + 1) is made, and O and the row sums, which P(t) has yet to enter at the old one, are scaled after the next phase, both
  // for the 16-query tiles with such a row alone.  (A rise costs about 600 cycles, half of it the branches, which a wave alone
  // on its SIMD waits for.  The sinks and local keys of attention make them rare after the first blocks; on random operands
  // without either, 8K x 32 / 8 heads, dense, they are a fifth of the call: 529 us, 541 with all tiles treated at once, 414
  // if none were seen; 556 with the kernel before.)
  // (Before, a step found the maxima across lanes in every block, in front of its exponentials, summed with dot products and
  // walked its mask bits in vector registers: 290 vector instructions besides the MFMAs instead of 207, and branches that cut
  // the schedule in pieces.  Without a running maximum it is 168, but then the largest probability of a row is rounded like
  // the others instead of being 1, and the errors against 64 bits grow by 1 % in O, by 30 % in lse.)
  // Attention call, before -> after, and without the maximum: dense 32K 7.60 -> 6.77 ms (6.27), sparse 4K 133 -> 124 us (113),
  // 16K 823 -> 720 (679), 32K 2.45 -> 2.27 ms (2.15), 128K 38.3 -> 35.4 (33.9), 64K with 32-key blocks 7.73 -> 7.11 (6.91);
  // int8 at 25K 1.49 -> 1.27 (1.18); dense 1K 27.4 -> 27.7 us (24.8).
  f32x4 S[2][2][NQ];                // [slot][16-key tile][query tile]: keys 4 g16 .. of query n16
  i32x4 A[2][NQ];                   // QK8: the integer accumulators of the first product (see qk_mfma)
  bf16x8 P[2][NQ];                  // keys 4 g16 .. of both 16-key tiles: the B operand of the second product as it is
  f32x4 lacc[NQ];                   // row sums: every register of lane (n16, g16) holds the sum over all keys of query n16
  bf16x8 kf[QK8 ? 1 : 2][QK8 ? 1 : 8], vf[2][8];      // operands of slot mt: K chunk 4 kt + s, V chunk dt
  i32x4 kf8[QK8 ? 2 : 1][QK8 ? 4 : 1];                // K chunk 2 kt + s
  bf16x8 ones;                      // A operand of the row sums
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  asm("" : "+a"(ones));      // (operands that stay go to accumulation registers: the
  // results of both products and what the vector unit makes take nearly all of the 256 ordinary ones, and a spill in front
  // of the sweep makes its waits for the operand loads those of the reload)
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
    for (int ks = 0; ks < (QK8 ? 2 : 4); ++ks) {
      if constexpr (QK8) asm("" : "+a"(qf8[qt][ks])); else asm("" : "+a"(qf[qt][ks]));
    }
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
    for (int r = 0; r < 4; ++r) lacc[qt][r] = l_run[qt];
  const i32x4 magic = {0x4B400000, 0x4B400000, 0x4B400000, 0x4B400000};
  constexpr int kSteps = QK8 ? 2 : 4;                                                   // contraction steps of the first product
  constexpr int kQk = 2 * kSteps * NQ, kPv = 8 * NQ, kElems = 8 * NQ;                   // MFMAs of the two products and scores per lane of a phase

  // MFMA n of S[y] = K(slot y) Q^T: a K fragment serves all query tiles in a row
  auto qk_mfma = [&](int y, int n) __attribute__((always_inline)) {
    const int kt = n / (kSteps * NQ), ks = n / NQ % kSteps, qt = n % NQ;
    if constexpr (QK8) {
      // The integer accumulators start at the bit pattern of kIntOffset = 1.5 * 2^23: an integer x with |x| < 2^22
      // added to it (the sums are below 127 * 127 * 128 < 2^21) gives the bit pattern of the FLOAT kIntOffset + x,
      // so the sums are read as floats without a conversion each; the offset leaves with the scaling FMAs.
      A[kt][qt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf8[y][kSteps * kt + ks], qf8[qt][ks], ks == 0 ? magic : A[kt][qt], 0, 0, 0);
    } else {
      const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
      S[y][kt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[y][kSteps * kt + ks], qf[qt][ks], ks == 0 ? z : S[y][kt][qt], 0, 0, 0);
    }
  };
  // MFMA n of O^T += V^T(slot y) P^T(slot y)
  auto pv_mfma = [&](int y, int n) __attribute__((always_inline)) {
    const int dt = n / NQ, qt = n % NQ;
    o16[dt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[y][dt], P[y][qt], o16[dt][qt], 0, 0, 0);
  };
  // Row sums of the ROUNDED probabilities, on the matrix unit (v_dot2c_f32_bf16, one per two probabilities, held up the MFMAs
  // next to it by 18 cycles each).  (One accumulator for all query tiles, four rows of it each, is 12 registers less, but 0 x NaN
  // would carry a query's NaN to the others.)
  auto sum_mfma = [&](int y, int qt) __attribute__((always_inline)) {
    lacc[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, P[y][qt], lacc[qt], 0, 0, 0);
  };
  auto load_k1 = [&](int t, int y, int n) __attribute__((always_inline)) {      // chunk n of a half-tile's K operands
    if constexpr (QK8) kf8[y][n] = load_chunk<i32x4>(k8t, lane16, t * 4096, n);
    else kf[y][n] = load_chunk<bf16x8>(kt, lane16, t * 8192, n);
  };
  auto load_v1 = [&](int t, int y, int n) __attribute__((always_inline)) { vf[y][n] = load_chunk<bf16x8>(vt, lane16, t * 8192, n); };
  auto load_k = [&](int hb, int y) __attribute__((always_inline)) {
    const int t = __builtin_amdgcn_readfirstlane(hb);
#pragma unroll
    for (int n = 0; n < 2 * kSteps; ++n) load_k1(t, y, n);
  };
  auto load_v = [&](int hb, int y) __attribute__((always_inline)) {
    const int t = __builtin_amdgcn_readfirstlane(hb);
#pragma unroll
    for (int n = 0; n < 8; ++n) load_v1(t, y, n);
  };
  auto finish = [&](int y, int kt, int qt) __attribute__((always_inline)) { if constexpr (QK8) S[y][kt][qt] = int_bits_as_floats(A[kt][qt]); };      // (no instruction)
  // keys after the query: koff = first key of the half-tile minus first query row of the block (a huge koff empties it)
  auto hide = [&](int x, int koff) __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const int seen = q0 + 16 * qt + n16 - 4 * g16 - koff;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * kt + r > seen) S[x][kt][qt][r] = -INFINITY;
    }
  };
  // Reference of the exponents, m_run: the running maximum of each query, half-tile by half-tile (a query that has seen no key
  // yet: a number below all logits).
  auto factor = [&](float k_scale) __attribute__((always_inline)) { return QK8 ? k_scale * sq_cs : cs; };      // score -> logit in log2 units
  auto logit = [&](float v, float ch) __attribute__((always_inline)) { return QK8 ? __builtin_fmaf(v, ch, -kIntOffset * ch) : v * ch; };
  float seen[NQ];      // (not QK8) m_run as a score
  float alpha[NQ];     // what the last rise takes O and the row sums of a query tile by, ...
  uint32_t due = 0;    // ... and the tiles (one bit each) where that is still to be done
  // (v_maximum3_f32: for v_max3_f32 the compiler first quiets every product that enters.  A NaN makes its query's results NaN anyway.)
  auto max3 = [](float a, float b, float w) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), w); };
  // top[qt]: the largest score that a lane holds of query tile qt
  auto tops_of = [&](int x, float (&top)[NQ]) __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const f32x4 e = S[x][0][qt], f = S[x][1][qt];
      top[qt] = __builtin_elementwise_maximum(max3(max3(max3(e[0], e[1], e[2]), e[3], f[0]), f[1], f[2]), f[3]);
    }
  };
  // The tiles with a query that rises above its maximum.  (Ballots: scalars, and so are the branches on them.)
  struct Rose { uint64_t in[NQ], any; };
  auto look = [&](const float (&top)[NQ], float ch) __attribute__((always_inline)) -> Rose {
    Rose r;
    r.any = 0;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      r.in[qt] = QK8 ? __builtin_amdgcn_ballot_w64(logit(top[qt], ch) > m_run[qt]) : __builtin_amdgcn_ballot_w64(top[qt] > seen[qt]);
      r.any |= r.in[qt];
    }
    return r;
  };
  auto raise = [&](const Rose& rose, const float (&top)[NQ], float ch) __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      if (rose.in[qt] == 0) continue;
      const float v = max_over_rows(top[qt]), m_new = __builtin_elementwise_maximum(m_run[qt], logit(v, ch));
      if constexpr (!QK8) seen[qt] = __builtin_elementwise_maximum(seen[qt], v);
      alpha[qt] = __builtin_amdgcn_exp2f(m_run[qt] - m_new);
      m_run[qt] = m_new;
      due |= 1u << qt;
    }
  };
  auto rescale = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      if ((due >> qt & 1) == 0) continue;
      lacc[qt] *= alpha[qt];
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) o16[dt][qt] *= alpha[qt];
    }
    due = 0;
  };

  struct Pair { int a, b; float ka, kb; };      // half-tiles of the two slots; QK8: the K scales of their blocks
  // One phase.  x: slot whose probabilities are made; y = 1 - x: slot of the two products and of the loads.  more: the scores
  // made here are complete (no key of theirs is to be hidden), so that their maximum counts.
  auto phase = [&](auto xc, float k_scale, int k_next, int v_next, float k_scale_next, bool more) __attribute__((always_inline)) {
    constexpr int x = decltype(xc)::value, y = 1 - x;
    constexpr int groups = kQk + kPv + NQ, exps = (kElems / 2 + 1) * 5, slots = exps + 4 * NQ;
    const float ch = factor(k_scale), ch_next = factor(k_scale_next);
    float mb[NQ], E[kElems], top[NQ];
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) mb[qt] = QK8 ? __builtin_fmaf(kIntOffset, ch, m_run[qt]) : m_run[qt];      // (QK8: the accumulators' offset)
    // The VALU stream, five instructions per two scores (score e: query tile e / 8, 16-key tile e / 4 % 2, register e % 4):
    // scale e, exp2 e - 1, scale e + 1, exp2 e, pack e - 2 and e - 1; then four per query tile for the maxima of the next scores
    auto valu = [&](int n) __attribute__((always_inline)) {
      if (n < exps) {
        const int e0 = 2 * (n / 5), o = n % 5;
        const int e = o == 0 ? e0 : o == 1 ? e0 - 1 : o == 2 ? e0 + 1 : o == 3 ? e0 : e0 - 2;
        if (e < 0 || e >= kElems) return;
        if (o == 0 || o == 2) E[e] = __builtin_fmaf(S[x][e / 4 % 2][e / 8][e % 4], ch, -mb[e / 8]);
        else if (o == 1 || o == 3) E[e] = __builtin_amdgcn_exp2f(E[e]);
        else { P[x][e / 8][e % 8] = (__bf16)E[e]; P[x][e / 8][e % 8 + 1] = (__bf16)E[e + 1]; }
      } else {
        const int qt = (n - exps) % NQ, o = (n - exps) / NQ;
        const f32x4 &e = S[y][0][qt], &f = S[y][1][qt];
        if (o == 0) { finish(y, 0, qt); top[qt] = max3(e[0], e[1], e[2]); }
        else if (o == 1) { finish(y, 1, qt); top[qt] = max3(top[qt], e[3], f[0]); }
        else if (o == 2) top[qt] = max3(top[qt], f[1], f[2]);
        else top[qt] = __builtin_elementwise_maximum(top[qt], f[3]);
      }
    };
    static_for<groups>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      constexpr PhaseStep st = phase_step(i, kQk, kPv);
      if constexpr (st.kind == 0) {
        qk_mfma(y, st.n);
        if constexpr (st.n % NQ == NQ - 1) load_k1(k_next, y, st.n / NQ);
      } else if constexpr (st.kind == 1) {
        pv_mfma(y, st.n);
        if constexpr (st.n % NQ == NQ - 1) load_v1(v_next, y, st.n / NQ);
      } else {
        sum_mfma(y, st.n);
      }
      constexpr int from = i * slots / groups, to = (i + 1) * slots / groups;
      static_for<to - from>([&](auto vc) __attribute__((always_inline)) { valu(from + decltype(vc)::value); });
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) asm volatile("" ::"v"(P[x][qt]));      // (the compiler would move their making past the branch, away from the MFMAs)
    Rose rose = look(top, ch_next);
    if (__builtin_expect_with_probability(due != 0 || (more && rose.any != 0), 0, 0.99)) {
      rescale();
      if (more) raise(rose, top, ch_next);
    }
  };
  const auto slot0 = std::integral_constant<int, 0>{};
  const auto slot1 = std::integral_constant<int, 1>{};

  auto pair_of = [&](uint32_t raw) __attribute__((always_inline)) -> Pair {
    const uint32_t w = kListed ? (uint32_t)__builtin_amdgcn_readfirstlane((int)raw) : raw;
    Pair p;
    p.a = BK32 ? (int)(w & 0xFFFFu) : 2 * (int)w;
    p.b = BK32 ? (int)(w >> 16) : p.a + 1;
    p.ka = p.kb = 1.0f;
    if constexpr (QK8) { p.ka = ks8[p.a >> 1]; p.kb = BK32 ? ks8[p.b >> 1] : p.ka; }
    return p;
  };

  if constexpr (kListed) build_list(word_lo, word_hi); else n_pairs = tiles;
  const int pairs = n_pairs;
  asm("" : "+v"(n_pairs));      // (a vector register on purpose: with scalar loop conditions the register allocator copies O^T between the loop's exits and spills)
  if (n_pairs > 0) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) seen[qt] = (m_run[qt] - 0x1p-20f * __builtin_fabsf(m_run[qt])) * (1.0f / cs);      // (of a resumed row: not above it)
    Pair c0 = pair_of(entry(0)), c1 = pair_of(entry(1));
    uint32_t ahead = entry(2);
    load_k(c0.a, 0);
    load_k(c0.b, 1);
    load_v(c0.a, 0);
#pragma unroll
    for (int n = 0; n < kQk; ++n) qk_mfma(0, n);
    load_k(c1.a, 0);
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) { finish(0, 0, qt); finish(0, 1, qt); }
    if (n_pairs == 1) hide(0, (c0.a - 2 * il) * 32);
    float top[NQ];
    auto look_at = [&](int x, float ch) __attribute__((always_inline)) { tops_of(x, top); raise(look(top, ch), top, ch); };
    look_at(0, factor(c0.ka));
    if (!resume) due = 0;      // (O is zero)
    if (BK32 && lone) hide(0, 1 << 24);
    // (nothing to multiply by yet: the first phase adds zeros)
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int e = 0; e < 8; ++e) vf[1][dt][e] = (__bf16)0.0f;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
      for (int e = 0; e < 8; ++e) P[1][qt][e] = (__bf16)0.0f;
    for (int n = 1; n < n_pairs; ++n) {
      const Pair c2 = pair_of(ahead);
      ahead = entry(n + 2);
      phase(slot0, c0.ka, c1.b, c0.b, c0.kb, true);
      phase(slot1, c0.kb, c2.a, c1.a, c1.ka, n + 1 < pairs);
      c0 = c1; c1 = c2;
    }
    // the last pair: the diagonal block, if it is kept
    c0.a = __builtin_amdgcn_readfirstlane(c0.a);      // (scalars to the compiler again, so that the loads stay single instructions)
    c0.b = __builtin_amdgcn_readfirstlane(c0.b);
    if (n_pairs > 1) {
      hide(0, (c0.a - 2 * il) * 32);
      look_at(0, factor(c0.ka));
    }
    phase(slot0, c0.ka, c0.b, c0.b, c0.kb, false);
    hide(1, (c0.b - 2 * il) * 32);
    look_at(1, factor(c0.kb));
    phase(slot1, c0.kb, c0.b, c0.b, c0.ka, false);
#pragma unroll
    for (int n = 0; n < kPv; ++n) pv_mfma(1, n);
#pragma unroll
    for (int n = 0; n < NQ; ++n) sum_mfma(1, n);
  }
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) l_run[qt] = lacc[qt][0];
  }

  if constexpr (NT == 2) if (park) {
    f32x4* so = st_o + (size_t)slot * 2048 + lane;
    float* sml = st_ml + (size_t)slot * 256;
    if constexpr (PV8) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            f32x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = oacc[dt][nt][4 * qd + e];
            so[((dt * 2 + nt) * 4 + qd) * 64] = w;
          }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) { sml[64 * nt + lane] = m_run[nt]; sml[128 + 64 * nt + lane] = l_run[nt]; }
    } else {
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) so[(dt * NQ + qt) * 64] = o16[dt][qt];
      if (g16 == 0) {
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) { sml[16 * qt + n16] = m_run[qt]; sml[128 + 16 * qt + n16] = l_run[qt]; }
      }
    }
    return;
  }
  // Output.  A lane holds, per tile, four consecutive channels of one query row: stored from there a
  // store instruction touches 16 or 32 rows.  The bf16 tile goes through LDS instead (rows padded by
  // four banks) and leaves as whole 256-byte rows, 4 rows per instruction.
  uint16_t* const tile = o_lds + (wave * 64 + q0) * kRowPad;
  // channels ch .. ch + 3 of query r of this wave
  auto put4 = [&](int r, int ch, f32x4 w) __attribute__((always_inline)) {
    if (o32) {     // calibration reads the output before it is rounded to bf16
      *(f32x4*)(o32 + ((size_t)u.qh * g.seq + u.i * 64 + q0 + r) * kHeadDim + ch) = w;
    } else {
      bf16x4 b;
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = (__bf16)w[e];
      *(bf16x4*)(tile + r * kRowPad + ch) = b;
    }
  };
  auto put_lse = [&](int r, float m, float l_tot) __attribute__((always_inline)) {
    const size_t row = (size_t)u.qh * g.seq + u.i * 64 + q0 + r;
    // (PV8: the sum is that of 448 p)
    // (the FMA is spelled out so that every instance of the kernel rounds alike)
    float v = l_tot > 0.0f ? __builtin_fmaf(m, 0.6931471805599453f, __logf(PV8 ? l_tot * (1.0f / 448.0f) : l_tot)) : -INFINITY;
    if constexpr (QK8) {
      // The 8-bit logits are those of K minus its mean key, i.e. Eq. 1's logits of this row minus q_r . mean /
      // sqrt(d) (which the softmax cancels in O); lse is reported for Eq. 1's S, so the shift goes back in.
      const uint16_t* qr = q + row_off(g.sq, u.qh, u.i * 64 + q0 + r);
      const float* mean = q8o.k_mean + (size_t)u.kvh * kHeadDim;
      float dot = 0.0f;
      for (int ch = 0; ch < kHeadDim; ++ch) dot = __builtin_fmaf(bf16_bits_to_float(qr[ch]), mean[ch], dot);
      v += dot * 0.08838834764831845f;
    }
    lse[row] = v;
  };
  if constexpr (PV8) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const float inv = l_run[nt] > 0.0f ? 1.0f / l_run[nt] : 0.0f;
      // O = v_scale[channel] * (sum P8 V8) / (sum P8)
      const float* vs = q8o.v_scale + (size_t)u.kvh * kHeadDim + 4 * h;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x4 sc = *(const f32x4*)(vs + 32 * dt + 8 * q4);
          f32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = oacc[dt][nt][4 * q4 + e] * sc[e] * inv;
          put4(32 * nt + c, 4 * h + 32 * dt + 8 * q4, w);
        }
      if (lse && h == 0) put_lse(32 * nt + c, m_run[nt], l_run[nt]);
    }
  } else {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const float inv = l_run[qt] > 0.0f ? 1.0f / l_run[qt] : 0.0f;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) put4(16 * qt + n16, 16 * dt + 4 * g16, o16[dt][qt] * inv);
      if (lse && g16 == 0) put_lse(16 * qt + n16, m_run[qt], l_run[qt]);
    }
  }
  if (!o32) {
    // (each wave reads back only its own tile: no barrier, LDS operations of a wave complete in order)
    wave_exchange();
    uint16_t* const out = o + row_off(g.so, u.qh, u.i * 64 + q0);
#pragma unroll
    for (int it = 0; it < 8 * NT; ++it) {
      const int r = 4 * it + (lane >> 4), ch = 8 * (lane & 15);
      *(u32x4*)(out + (size_t)r * g.so.st + ch) = *(const u32x4*)(tile + r * kRowPad + ch);
    }
  }
}

// All three in units of 64 keys (scaled by 64 / b_k for a mask with one bit per b_k keys).
// Workgroups go to the XCDs round-robin, so "lane" blockIdx % n_kvh of a launch always runs on the same XCDs.
// With lane = KV head an XCD's L2 serves one head's K', V', but the heads of a layer keep very different
// numbers of blocks (1.6x between the lightest and the heaviest at 128K here) and the light XCDs would idle.
// For every window launch (one workgroup of this kernel each) a table moves a representative sample (every
// so-many-th of the sorted list) of the units of every over-loaded head to the lanes of the under-loaded
// ones, in proportion to the work they lack in THAT window:
//   assign[window][lane][slot] = kvh * units + unit id, or -1.
// A unit takes part in a window if its row has a parking slot (a long row) and keeps a block there, or if the
// window holds its diagonal block (where the row is finished whatever it keeps).
// Falls back to lane = KV head when there are too many lanes or a lane would overflow.
constexpr int kMaxLanes = 256;
struct LaneLoad { unsigned long long work; int n_in; int pad; };      // per (window, KV head)
constexpr size_t kLaneLoadBytes = (size_t)(kMaskWordsMax / 2) * kMaxLanes * sizeof(LaneLoad);      // 128 KB
static_assert(kLaneLoadBytes >= kMaxQueues * kQueueStride * sizeof(int), "without window launches the loads' place holds the queues' counters");

// Shared by the two kernels below: the units of ONE head in ONE window, 1024 threads, thread t looks at the
// ranks t * per .. of the head's sorted list.
struct WindowScan {
  const Geo& g;
  const uint64_t* mask;
  const int32_t* slot_of;
  const int32_t* order;
  int w0, w1, bits_per_q, units;
  // blocks the unit at rank r of head h keeps in this window (-1: it does not take part)
  __device__ int in_window(int h, int r, int& id) const {
    id = order[(size_t)h * units + r];
    const int i = id / g.group, qh = h * g.group + id % g.group;
    if (slot_of[(size_t)qh * g.n_qb + i] < 0) return -1;      // swept whole, in a tail
    const int j_last = (seq_pos(g, i).il + 1) * bits_per_q - 1, last_word = j_last >> 6;
    if (w0 > last_word) return -1;
    const uint64_t* mrow = mask + ((size_t)qh * g.n_qb + i) * g.words;
    int c = 0;
    for (int wc = w0; wc < min(w1, last_word + 1); ++wc) {
      const int lo = wc * 64;
      const uint64_t causal = j_last >= lo + 63 ? ~0ull : ((2ull << (j_last - lo)) - 1ull);
      c += __popcll(mrow[wc] & causal);
    }
    return (c > 0 || w1 > last_word) ? c : -1;
  }
};

// exclusive prefix over a 1024-thread workgroup of a per-thread count; total in `sum`
__device__ __forceinline__ int block_scan_1024(int v, int* wave_sum, int& sum) {
  const int lane_id = threadIdx.x & 63, wave_id = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(inc, off, 64);
    if (lane_id >= off) inc += o;
  }
  __syncthreads();
  if (lane_id == 63) wave_sum[wave_id] = inc;
  __syncthreads();
  int base = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int x = wave_sum[w];
    if (w < wave_id) base += x;
    all += x;
  }
  sum = all;
  return base + inc - v;
}

// Workgroup (window, head): number of participating units and their work in the window; clears the head's
// own lane of the window's table.
__global__ __launch_bounds__(1024) void window_load_kernel(Geo g, const uint64_t* __restrict__ mask,
                                                           const int32_t* __restrict__ slot_of,
                                                           const int32_t* __restrict__ order, int win_words,
                                                           int bits_per_q, LaneLoad* __restrict__ load,
                                                           int32_t* __restrict__ assign_all) {
  __shared__ int wave_sum[16];
  __shared__ unsigned long long work;
  const int units = g.n_qb * g.group, lanes = g.n_kvh;
  const int win = blockIdx.x / lanes, h = blockIdx.x % lanes;
  const int tid = threadIdx.x, per = (units + 1023) / 1024;
  const WindowScan ws = {g, mask, slot_of, order, win * win_words, (win + 1) * win_words, bits_per_q, units};
  int32_t* mine = assign_all + ((size_t)win * lanes + h) * units;
  for (int e = tid; e < units; e += 1024) mine[e] = -1;
  if (tid == 0) work = 0;
  int n_mine = 0;
  unsigned long long w_mine = 0;
  for (int r = tid * per; r < min((tid + 1) * per, units); ++r) {
    int id;
    const int c = ws.in_window(h, r, id);
    if (c >= 0) { ++n_mine; w_mine += (unsigned long long)c; }
  }
  int n_tot;
  block_scan_1024(n_mine, wave_sum, n_tot);      // (its barriers also publish work = 0)
  if (w_mine) atomicAdd(&work, w_mine);
  __syncthreads();
  if (tid == 0 && h < kMaxLanes) { load[win * kMaxLanes + h].work = work; load[win * kMaxLanes + h].n_in = n_tot; }
}

// Workgroup (window, head): places the head's participating units in the window's table.
__global__ __launch_bounds__(1024) void balance_kernel(Geo g, const uint64_t* __restrict__ mask,
                                                       const int32_t* __restrict__ slot_of,
                                                       const int32_t* __restrict__ order, int win_words,
                                                       int bits_per_q, const LaneLoad* __restrict__ load,
                                                       int32_t* __restrict__ assign_all) {
  __shared__ int n_shed_h, shed_off_h, n_in_h, recv_lo[kMaxLanes + 1];
  __shared__ int wave_sum[16];
  const int units = g.n_qb * g.group, lanes = g.n_kvh;
  const int win = blockIdx.x / lanes, h = blockIdx.x % lanes;
  const int tid = threadIdx.x, per = (units + 1023) / 1024;
  const WindowScan ws = {g, mask, slot_of, order, win * win_words, (win + 1) * win_words, bits_per_q, units};
  int32_t* assign = assign_all + (size_t)win * lanes * units;
  const bool balance = lanes <= kMaxLanes && lanes > 1;
  if (tid == 0) {
    n_shed_h = 0; shed_off_h = 0; n_in_h = 1;
    for (int l = 0; l <= min(lanes, kMaxLanes); ++l) recv_lo[l] = 0;
    if (balance) {
      const LaneLoad* ld = load + win * kMaxLanes;
      unsigned long long sum = 0;
      for (int l = 0; l < lanes; ++l) sum += ld[l].work;
      const double target = (double)sum / lanes;
      double lack_total = 0.0;
      int shed_total = 0, my_shed = 0, my_off = 0;
      for (int l = 0; l < lanes; ++l) {
        const double w = (double)ld[l].work;
        const int ns = w > target ? (int)((double)ld[l].n_in * (w - target) / w) : 0;
        if (l == h) { my_shed = ns; my_off = shed_total; }
        shed_total += ns;
        if (w < target) lack_total += target - w;
      }
      // the shed units, numbered (offset of their head) + k, go to the lanes that lack work, in proportion
      double lack_run = 0.0;
      bool ok = lack_total > 0.0;
      for (int l = 0; l < lanes && ok; ++l) {
        recv_lo[l] = (int)((double)shed_total * (lack_run / lack_total));
        const double w = (double)ld[l].work;
        if (w < target) lack_run += target - w;
      }
      recv_lo[lanes] = shed_total;
      for (int l = 0; l < lanes && ok; ++l) {
        const double w = (double)ld[l].work;
        const int ns = w > target ? (int)((double)ld[l].n_in * (w - target) / w) : 0;
        ok = ld[l].n_in - ns + recv_lo[l + 1] - recv_lo[l] <= units;
      }
      if (ok) { n_shed_h = my_shed; shed_off_h = my_off; n_in_h = max(ld[h].n_in, 1); }
      else for (int l = 0; l <= lanes; ++l) recv_lo[l] = 0;
    }
  }
  int n_mine = 0;
  for (int rr = tid * per; rr < min((tid + 1) * per, units); ++rr) {
    int id;
    if (ws.in_window(h, rr, id) >= 0) ++n_mine;
  }
  int n_tot;
  int r = block_scan_1024(n_mine, wave_sum, n_tot);      // (its barriers also publish thread 0's parameters)
  // r counts the participating units of the head in sorted order (longest rows first)
  for (int rr = tid * per; rr < min((tid + 1) * per, units); ++rr) {
    int id;
    if (ws.in_window(h, rr, id) < 0) continue;
    int lane = h, pos = r;
    if (balance) {
      const long long ns = n_shed_h, n = n_in_h;
      const int before = (int)((long long)r * ns / n), upto = (int)((long long)(r + 1) * ns / n);
      if (upto > before) {                      // this unit is shed: global shed number p
        const int p = shed_off_h + before;
        int l = 0;
        while (l + 1 < lanes && recv_lo[l + 1] <= p) ++l;
        lane = l;
        // Received units go first in their new lane: all lanes then read the shedding head's window at the
        // start of a launch, together (interleaving them with the lane's own units was 6 % slower).
        pos = p - recv_lo[l];
      } else {
        pos = (recv_lo[h + 1] - recv_lo[h]) + (r - before);
      }
    }
    assign[(size_t)lane * units + pos] = h * units + id;
    ++r;
  }
}

constexpr int kLongRow = 192;        // rows keeping more than this (12K tokens) are swept window by window
// Window width in mask words of 64 x 64 keys.  bf16: 8K tokens, 4 MB of K', V' per KV head.  The 8-bit passes read three
// quarters or half as much per block and shorter steps pay more for every further window: 16K tokens.  Attention call, 8K / 12K /
// 16K / 32K tokens: FP8 64K 6.28 / 6.15 / 5.99 / 6.36 ms, 128K 23.8 / 23.2 / 23.3 / 24.9; int8 25K 1.35 / 1.31 / 1.27 / 1.30, 64K
// 7.78 / 7.75 / 7.78 / 8.23, 128K 29.9 / 30.0 / 31.1 / 32.5, 64K with 32-key blocks 6.19 / 6.13 / 6.14 / 6.46; bf16 32K 2.31 /
// 2.30 / 2.28 / 2.43, 64K 9.21 / 9.26 / 9.32 / 10.6, 128K 35.8 / 37.0 / 37.6 / 44.5, 64K with 32-key blocks 7.20 / 7.25 / 7.29 / 7.96.
constexpr int kWindowWords = 2, kWindowWords8 = 4;
constexpr int kWindowMinWords = 4;   // sequences of up to 16K tokens use one sweep per row

namespace {

// Window launches: long sequences.  Without a single parking slot in the workspace every row is swept whole.
bool use_windows(const Geo& g, const int32_t* row_counts, int n_slots) {
  return row_counts && g.words > kWindowMinWords * (g.bk == 32 ? 2 : 1) && n_slots > 0;
}

template <bool QK8, bool PV8>
int launch_dense_rows(const Geo& g, const uint16_t* q, const bf16x8* kp, const bf16x8* vp, Qk8 q8o, const int32_t* order,
                      uint16_t* o, float* o32, float* lse, bool halves, hipStream_t st) {
  const int units = g.n_qb * g.group;
  const RowFilter all = {nullptr, -1, 0, -1, 0, 0};
#define SALE_DENSE_ARGS g, q, kp, vp, q8o, nullptr, order, nullptr, o, o32, lse, all, nullptr, nullptr
  if (halves)
    attn_rows_kernel<1, false, QK8, PV8, 1><<<dim3((unsigned)(units * g.n_kvh)), dim3(128), 0, st>>>(SALE_DENSE_ARGS);
  else
    attn_rows_kernel<4, false, QK8, PV8><<<dim3((unsigned)(((units + 3) / 4) * g.n_kvh)), dim3(256), 0, st>>>(SALE_DENSE_ARGS);
#undef SALE_DENSE_ARGS
  return hipGetLastError() == hipSuccess ? SALE_OK : SALE_ERR_HIP;
}

template <bool BK32, bool QK8, bool PV8 = false>
int launch_sparse_rows(const Geo& g, const uint16_t* q, const bf16x8* kp, const bf16x8* vp, Qk8 q8o, const uint64_t* mask,
                       const int32_t* row_counts, int32_t* order /* nullptr: as they come */, int32_t* assign, LaneLoad* load, int32_t* slot_of,
                       int* slot_counter, int n_slots, uint16_t* o, float* o32, float* lse, f32x4* st_o, float* st_ml,
                       bool windows, bool halves, bool queues, hipStream_t st) {
  const int units = g.n_qb * g.group;
  const int f = BK32 ? 2 : 1;          // mask bits per 64 keys
  const dim3 grid((unsigned)(units * g.n_kvh));
  const RowFilter all = {nullptr, -1, 0, -1, 0, 0};
  if (windows) {      // (otherwise the rows were sorted beside the copies)
    order_units_kernel<<<dim3((unsigned)g.n_kvh), dim3(1024), 0, st>>>(g, row_counts, order, slot_of, kLongRow * f, n_slots,
                                                                       slot_counter);
    if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  }
  if (halves) {
    attn_rows_kernel<1, BK32, QK8, PV8, 1><<<grid, dim3(128), 0, st>>>(g, q, kp, vp, q8o, mask, order, nullptr,
                                                                       o, o32, lse, all, nullptr, nullptr);
    return hipGetLastError() == hipSuccess ? SALE_OK : SALE_ERR_HIP;
  }
  if (!windows) {
    RowFilter flt = all;
    dim3 issue = grid;
    if (queues) {      // (what an XCD may take beyond its own heads' rows: an eighth of them)
      flt.taken = (int*)load;
      flt.queue_from = units / 2;
      issue.x += (unsigned)(units / 8 * g.n_kvh);
    }
    attn_rows_kernel<1, BK32, QK8, PV8><<<issue, dim3(64), 0, st>>>(g, q, kp, vp, q8o, mask, order, nullptr,
                                                             o, o32, lse, flt, nullptr, nullptr);
    return hipGetLastError() == hipSuccess ? SALE_OK : SALE_ERR_HIP;
  }

  // Long rows carry most of the work and keep scattered blocks over the whole sequence: swept
  // independently they miss L2 on most loads.  They are processed one window (kWindowWords: in bf16 4 MB of K', V'
  // per KV head, the size of an XCD's L2) at a time, all rows together, so that the window is served by
  // the L2 of the XCD that owns the KV head; their accumulators wait in the workspace in between.
  // Measured at 128K tokens (L2 fills / time of the call): one sweep per row 218 GB / 50.7 ms; windows of
  // 16K tokens 121 GB / 37.5 ms; 8K tokens 57 GB / 37.4 ms; 4K tokens 50 GB / 39.1 ms (the parked state
  // then costs more than the window saves).  At 32K tokens windows (with the balancing below) and one sweep
  // per row are within 2 % of each other; shorter sequences use one sweep.
  // Short rows keep little besides the sink, the local band and the heavy columns everyone shares.
  // They are dealt over the window launches: launch number n ends with ranks n, n + launches, ... of every
  // KV head's sorted list (the tail of the grid), which fill the chip while its last long rows finish.
  const int step = (QK8 ? kWindowWords8 : kWindowWords) * f, launches = (g.words + step - 1) / step;
  const int tail_wgs = ((units + launches - 1) / launches) * g.n_kvh;
  window_load_kernel<<<dim3((unsigned)(launches * g.n_kvh)), dim3(1024), 0, st>>>(g, mask, slot_of, order, step, f, load,
                                                                                 assign);
  if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  balance_kernel<<<dim3((unsigned)(launches * g.n_kvh)), dim3(1024), 0, st>>>(g, mask, slot_of, order, step, f, load, assign);
  if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  for (int n = 0; n < launches; ++n) {
    // (the table holds the rows with a parking slot; the tail takes the others)
    const RowFilter flt = {slot_of, n * step, step, (int)grid.x, launches, n};
    attn_rows_kernel<1, BK32, QK8, PV8><<<dim3(grid.x + (unsigned)tail_wgs), dim3(64), 0, st>>>(
        g, q, kp, vp, q8o, mask, order, assign + (size_t)n * grid.x, o, o32, lse, flt, st_o, st_ml);
    if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  }
  return SALE_OK;
}

}  // namespace

// Workspace of the attention calls.  Fixed part: K' | V' | (sparse: unit order | parking slot per row block | balanced
// issue tables, room for 32 window launches | per-window head loads | slot counter) | 8-bit operand copies | FP8 copy
// of V | per-block sequence table; then (sparse) the parking slots, 33 KB each: as many as the caller's workspace holds,
// or (dense, packed sequences) the unit order, if it has room for it.
namespace {
struct AttnWs {
  u32x4 *kp, *vp;      // (room for both in every call; the 8-bit first product leaves K', the FP8 second one V' unused)
  int32_t *order, *slot_of, *assign;
  LaneLoad* load;
  int* slot_counter;
  uint8_t *ops8, *ops_fp8;
  int32_t* seq_table;
  uint8_t* parked;
  size_t fixed_bytes;
};
AttnWs carve_attn_ws(const sale_params_t* p, bool sparse, void* base) {
  const size_t tile_bytes = (size_t)p->batch * p->n_kv_heads * p->seq_len * kHeadDim * sizeof(uint16_t);
  const size_t n_units = (size_t)p->batch * p->n_q_heads * (p->seq_len / kBlockQ);
  AttnWs w = {};
  size_t off = 0;
  auto take = [&](size_t bytes) { uint8_t* ptr = (uint8_t*)base + off; off += (bytes + 63) & ~(size_t)63; return ptr; };
  w.kp = (u32x4*)take(tile_bytes);
  w.vp = (u32x4*)take(tile_bytes);
  if (sparse) {
    w.order = (int32_t*)take(n_units * sizeof(int32_t));
    w.slot_of = (int32_t*)take(n_units * sizeof(int32_t));
    w.assign = (int32_t*)take(n_units * (kMaskWordsMax / 2) * sizeof(int32_t));
    w.load = (LaneLoad*)take(kLaneLoadBytes);
    w.slot_counter = (int*)take(sizeof(int));
  }
  if (p->flags & SALE_FLAG_ATTN_INT8_QK) w.ops8 = take(int8_operand_bytes(p));
  if (p->flags & SALE_FLAG_ATTN_FP8_PV) w.ops_fp8 = take(fp8_operand_bytes(p));
  if (p->n_seqs > 0) w.seq_table = (int32_t*)take(seq_table_bytes(p));
  w.parked = (uint8_t*)base + off;
  w.fixed_bytes = off;
  return w;
}
}  // namespace

size_t attn_fixed_bytes(const sale_params_t* p, bool sparse) { return carve_attn_ws(p, sparse, nullptr).fixed_bytes; }

// What the issue of a call's rows goes by.
namespace {
struct BatchShape {
  int longest;             // 64-row blocks of the longest sequence
  long even_rows;          // rows that make up as much work in sequences of that length
  bool long_rows_wait;     // issued by position, 512 rows start before those of some sequence of 3/4 of that length or more
};
BatchShape batch_shape(const sale_params_t* p) {
  BatchShape s = {longest_sequence(p) / kBlockQ, (long)p->batch * p->n_q_heads * (p->seq_len / kBlockQ), false};
  if (p->n_seqs <= 0) return s;
  long long work = 0;
  for (int i = p->n_seqs - 1; i >= 0; --i) {
    const long long n = (p->cu_seqlens[i + 1] - p->cu_seqlens[i]) / kBlockQ;
    work += n * (n + 1);
    if (4 * n >= 3 * s.longest) s.long_rows_wait = (long)p->n_q_heads * ((p->seq_len - p->cu_seqlens[i + 1]) / kBlockQ) >= 512;
  }
  s.even_rows = (long)(p->n_q_heads * work / (s.longest + 1));
  return s;
}
}  // namespace

size_t dense_order_bytes(const sale_params_t* p) {
  return p->n_seqs > 0 ? (size_t)p->n_q_heads * (p->seq_len / kBlockQ) * sizeof(int32_t) : 0;
}

// o: bf16 output, or (o32 != nullptr) fp32 output instead.  mask == nullptr: dense causal attention
// (independent of b_k).  ws_bytes >= attn_fixed_bytes (checked by the callers); what lies beyond holds parking slots.
int launch_attn_rows(const sale_params_t* p, const void* q, const void* k, const void* v, const uint64_t* mask,
                     const int32_t* row_counts, void* o, float* o32, float* lse, void* ws, size_t ws_bytes, hipStream_t st) {
  Geo g = make_geo(p);
  const AttnWs w = carve_attn_ws(p, mask != nullptr, ws);
  if (ws_bytes < w.fixed_bytes) return SALE_ERR_WORKSPACE;
  if (p->n_seqs > 0) {
    const int rc = build_seq_table(p, w.seq_table, st);
    if (rc != SALE_OK) return rc;
    g.seq_start = w.seq_table;
  }
  u32x4 *kp = w.kp, *vp = w.vp;
  const size_t n_units = (size_t)g.n_qh * g.n_qb;
  const size_t n_slots_z = mask ? (ws_bytes - w.fixed_bytes) / kParkedRowBytes : 0;
  const int n_slots = (int)(n_slots_z < n_units ? n_slots_z : n_units);
  f32x4* st_o = (f32x4*)w.parked;                               // [slot] 32 KB
  float* st_ml = (float*)(w.parked + (size_t)n_slots * 2048 * 16);      // [slot] 1 KB
  const bool qk8 = (p->flags & SALE_FLAG_ATTN_INT8_QK) != 0;
  const bool pv8 = (p->flags & SALE_FLAG_ATTN_FP8_PV) != 0;      // (validated: only with qk8 and 64-key blocks)
  const bool windows = mask && use_windows(g, row_counts, n_slots);
  const bool counts = mask && row_counts;
  const BatchShape shape = batch_shape(p);
  bool halves = !windows && two_waves_per_row({(long)n_units, shape.even_rows, shape.longest, g.n_kvh, g.group, !mask,
                                               mask && g.bk == 32, qk8, pv8, p->n_seqs > 0 && !counts});
  // Rows that do not all start at once have to start longest first.  Without counts they are issued from the last block
  // on: longest first inside one sequence, not over packed ones.  With two waves per row (512 rows start at once) the long
  // rows of an early sequence then started when most others had run: 64 sequences of 1024 tokens, one head, dense, 64.6 us
  // (one wave per row 51.1) -> 46.0; where the long rows come early enough the sort is left out (it costs 2 - 3 %).
  int32_t* const order_at = mask ? w.order : ws_bytes - w.fixed_bytes >= dense_order_bytes(p) ? (int32_t*)w.parked : nullptr;
  const bool by_length = halves && !counts && shape.long_rows_wait;
  if (by_length && !order_at) halves = false;      // (a dense workspace without the order's bytes)
  const bool sort = !windows && (counts || (by_length && halves));
  const bool queues = counts && !windows && !halves && issue_by_queue({(long)n_units, shape.even_rows, shape.longest, g.n_kvh,
                                                                                g.group, false, g.bk == 32, qk8, pv8, false});
  const OrderJob job = {sort ? g.n_kvh : 0, queues ? (int*)w.load : nullptr, mask ? row_counts : nullptr, order_at};
  int32_t* const order = sort || windows ? order_at : nullptr;
  Int8Operands w8 = {};
  Fp8Operands wv = {};
  if (qk8) w8 = carve_int8_operands(p, (void*)w.ops8);
  if (pv8) wv = carve_fp8_operands(p, (void*)w.ops_fp8);
  const Pass8 pass = make_pass8(p, q, k, v, qk8 ? &w8 : nullptr, pv8 ? &wv : nullptr);
  // (with FP8 V there is nothing to copy: one workgroup, which clears the slot counter)
  const int tiles = pv8 ? (w.slot_counter ? 1 : 0) : g.n_kvh * (g.seq / 64);
  const dim3 first((unsigned)(job.heads + tiles + pass.blocks()));
  const Then8 then = {tiles, pass};
#define SALE_REARRANGE_ARGS (const uint16_t*)k, (const uint16_t*)v, kp, vp, w.slot_counter
  if (!qk8) rearrange_kv_kernel<true, true><<<first, dim3(256), 0, st>>>(g, job, NoPass8{}, SALE_REARRANGE_ARGS);
  else if (!pv8) rearrange_kv_kernel<false, true><<<first, dim3(256), 0, st>>>(g, job, then, SALE_REARRANGE_ARGS);
  else rearrange_kv_kernel<false, false><<<first, dim3(256), 0, st>>>(g, job, then, SALE_REARRANGE_ARGS);
#undef SALE_REARRANGE_ARGS
  if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  Qk8 q8o = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  if (qk8) {
    const int rc = launch_operands8(p, k, v, &w8, pv8 ? &wv : nullptr, pv8 ? 32 : 16, st);
    if (rc != SALE_OK) return rc;
    q8o = {w8.q8, (const u32x4*)w8.k8, w8.q_scale, w8.k_scale, w8.k_mean, (const u32x4*)wv.v8, wv.v_scale};
  }
  const uint16_t* qq = (const uint16_t*)q;
  const bf16x8 *kpp = (const bf16x8*)kp, *vpp = (const bf16x8*)vp;
  if (mask) {
#define SALE_SPARSE_ARGS g, qq, kpp, vpp, q8o, mask, row_counts, order, w.assign, w.load, w.slot_of, w.slot_counter, n_slots, \
                         (uint16_t*)o, o32, lse, st_o, st_ml, windows, halves, queues, st
    if (g.bk == 32) return qk8 ? launch_sparse_rows<true, true>(SALE_SPARSE_ARGS) : launch_sparse_rows<true, false>(SALE_SPARSE_ARGS);
    if (pv8) return launch_sparse_rows<false, true, true>(SALE_SPARSE_ARGS);
    return qk8 ? launch_sparse_rows<false, true>(SALE_SPARSE_ARGS) : launch_sparse_rows<false, false>(SALE_SPARSE_ARGS);
#undef SALE_SPARSE_ARGS
  }
  if (pv8) return launch_dense_rows<true, true>(g, qq, kpp, vpp, q8o, order, (uint16_t*)o, o32, lse, halves, st);
  return qk8 ? launch_dense_rows<true, false>(g, qq, kpp, vpp, q8o, order, (uint16_t*)o, o32, lse, halves, st)
             : launch_dense_rows<false, false>(g, qq, kpp, vpp, q8o, order, (uint16_t*)o, o32, lse, halves, st);
}

}  // namespace sale

using namespace sale;

extern "C" int sale_sparse_attn(const sale_params_t* p, const void* q, const void* k, const void* v,
                                const uint64_t* block_mask, const int32_t* row_counts, void* o, float* lse, void* ws,
                                size_t ws_bytes, void* stream) {
  if (!p || !q || !k || !v || !block_mask || !o) return SALE_ERR_NULL_ARG;
  int rc = validate_common(p, kGeomPath);
  if (rc != SALE_OK) return rc;
  // (any size from SALE_WS_SPARSE_ATTN_MIN on: what lies beyond the fixed part holds parking slots)
  const size_t need = sale_workspace_bytes(p, SALE_WS_SPARSE_ATTN_MIN);
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 15)) return SALE_ERR_WORKSPACE;
  return launch_attn_rows(p, q, k, v, block_mask, row_counts, o, nullptr, lse, ws, ws_bytes, (hipStream_t)stream);
}

extern "C" int sale_dense_attn(const sale_params_t* p, const void* q, const void* k, const void* v, void* o, float* lse,
                               void* ws, size_t ws_bytes, void* stream) {
  if (!p || !q || !k || !v || !o) return SALE_ERR_NULL_ARG;
  int rc = validate_common(p, kGeomPath);
  if (rc != SALE_OK) return rc;
  const size_t need = attn_fixed_bytes(p, false);      // (what SALE_WS_DENSE_ATTN asks for beyond it only makes packed calls faster)
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 15)) return SALE_ERR_WORKSPACE;
  return launch_attn_rows(p, q, k, v, nullptr, nullptr, o, nullptr, lse, ws, ws_bytes, (hipStream_t)stream);
}
