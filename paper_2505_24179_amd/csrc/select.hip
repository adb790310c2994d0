// Selection-Pass (Alg. 1): sink-local statistics from the unquantized Q, K,
// then the 4-bit Q~ K~^T estimate of every middle block scored against
// thr_r = ln(tau l~_r) + m~_r (Eq. 3 in the log form of Eq. 4), written as one
// bit per (query block, key block).
//
// Both kernels compute the TRANSPOSED tile, keys x queries (A operand = K rows,
// B operand = Q rows).  In the MFMA accumulator layouts a lane then owns keys of
// ONE query column per tile, so the per-query maximum over a key block is an
// in-lane max chain, the per-query threshold is a single register, and the
// "any row of the block passes" reduction is the wave-wide compare mask.
//
// CDNA4 has no int4 MFMA: the integer products run, exactly, on the FP6 MFMA
// (see below).
#include <mutex>

#include "row_split.h"
#include "sale_common.h"

namespace sale {

// Key blocks may be 64 or 32 tokens (MT = b_k / 32 MFMA row tiles per block); query blocks are 64 rows.
__device__ __forceinline__ int j_last_of(const Geo& g, int i) { return (i + 1) * (kBlockQ / g.bk) - 1; }

// Number of local key blocks of a row whose last visible key block is j_last.  With segments (Appendix C:
// the middle blocks are handled in groups of g.seg and the blocks left over at the end of the row are
// treated as local) the local area grows by that remainder.
__device__ __forceinline__ int local_of(const Geo& g, int j_last) {
  const int middle = j_last + 1 - g.sink_blocks - g.local_blocks;
  return g.local_blocks + (g.seg > 0 && middle > 0 ? middle % g.seg : 0);
}

__device__ __forceinline__ bool in_sink_local(const Geo& g, int j, int j_last, int local) {
  return j < g.sink_blocks || j > j_last - local;
}

// ---------------------------------------------------------------------------
// 4-bit estimate on the FP6 (E2M3) MFMA
// ---------------------------------------------------------------------------
// CDNA4 has no int4 MFMA.  Every integer in [-7, 7] is exactly representable in
// FP6 E2M3 (1 sign, 2 exponent, 3 mantissa bits, bias 1: 1 = 0b001000, 2 =
// 0b010000, 3 = 0b010100, 4 = 0b011000, 5 = 0b011010, 6 = 0b011100, 7 =
// 0b011110), products are at most 49 and a 128-term sum at most 6272 < 2^24, so
// v_mfma_f32_16x16x128_f8f6f4 with both operands in E2M3 and unit scales returns
// the integer product EXACTLY in its fp32 accumulator (checked on hardware
// against integer arithmetic, including all-(+-7) operands) at twice the int8
// MFMA rate.  (That shape because the kernel runs at the card's power limit: it contracts all 128 channels at once, so no
// accumulator is read back.  A loop of random operands with the maxima beside it: 44 products of 32x32x64 per us and
// SIMD, 94 of these, half as large; 96 if neighbours share an operand throughout.)
// A pre-pass re-encodes the nibble codes of K~ once into MFMA operand
// order ("X6"; Q~ is re-encoded by the wave that uses it): per group of 32 rows 2 fragments f (rows 16f..); lane l of a
// fragment owns row 16f + l%16 of the group, channels 32(l/16) + e, e = 0..31, as
// 32 six-bit codes = 6 dwords, stored as
//   [group][f][lane] 16 bytes (dwords 0..3)  followed by  [group][f][lane] 8 bytes (dwords 4..5).
constexpr int kX6GroupBytes = 2 * 64 * 24;   // 3072 bytes per 32 rows

// (about 30 vector instructions per 8 codes; code by code it took 64 and was 7 us of a wave of select_kernel)
// E2M3 codes of the four 4-bit two's-complement nibbles (-7..7) in the low halves of the bytes of n (the high halves
// are zero): two byte look-ups by the low three bits, for n >= 0 and n < 0, chosen by the sign bit.
__device__ __forceinline__ uint32_t e2m3_of_nibbles(uint32_t n) {
  const uint32_t at = n & 0x07070707u, sign = n & 0x08080808u;
  const uint32_t pos = __builtin_amdgcn_perm(0x1E1C1A18u, 0x14100800u, at);       // 0, 1, 2, 3 | 4, 5, 6, 7
  const uint32_t neg = __builtin_amdgcn_perm(0x28303438u, 0x3A3C3E20u, at);       // (-8: -0), -7, -6, -5 | -4, -3, -2, -1
  const uint32_t is_neg = (sign << 5) - (sign >> 3);                              // 0xFF in the bytes of negative codes
  return (neg & is_neg) | (pos & ~is_neg);
}

// 16 packed bytes (32 nibble codes, channel order) -> 32 six-bit codes in 6 dwords.
__device__ __forceinline__ void pack_fp6(const u32x4 w, uint32_t out[6]) {
  uint32_t f[8];      // 24 bits each: the codes of two bytes
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t lo = e2m3_of_nibbles(w[d] & 0x0F0F0F0Fu), hi = e2m3_of_nibbles((w[d] >> 4) & 0x0F0F0F0Fu);
    const uint32_t x0 = (lo & 0x00FF00FFu) | ((hi & 0x00FF00FFu) << 6);                  // 12 bits: bytes 0 and 2
    const uint32_t x1 = ((lo >> 8) & 0x00FF00FFu) | (((hi >> 8) & 0x00FF00FFu) << 6);    //          bytes 1 and 3
    f[2 * d] = (x0 & 0xFFFu) | ((x1 & 0xFFFu) << 12);
    f[2 * d + 1] = (x0 >> 16) | ((x1 >> 16) << 12);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {      // four 24-bit pieces make three dwords
    const uint32_t* p = f + 4 * t;
    out[3 * t] = p[0] | (p[1] << 24);
    out[3 * t + 1] = (p[1] >> 8) | (p[2] << 16);
    out[3 * t + 2] = (p[2] >> 16) | (p[3] << 8);
  }
}

// Re-encoding of a nibble-packed [32 * groups][64-byte] matrix: one thread per (32-row group, fragment, lane).  It is
// the last workgroups of the statistics launch (from number `first` on), which it does not depend on: a launch of its
// own cost 3 us in the smallest calls and its streaming (49 us at 128K) now runs beside the statistics.
struct PackFp6 {
  const uint8_t* x;
  uint8_t* y;
  long groups;
  int first;
  __device__ __forceinline__ void run(int block) const {
    const long grp = (long)(block - first) * (blockDim.x >> 7) + (threadIdx.x >> 7);
    if (grp >= groups) return;
    const int f = (threadIdx.x >> 6) & 1, lane = threadIdx.x & 63;
    const u32x4 w = *(const u32x4*)(x + ((size_t)grp * 32 + 16 * f + (lane & 15)) * 64 + 16 * (lane >> 4));
    uint32_t d[6];
    pack_fp6(w, d);
    uint8_t* yg = y + (size_t)grp * kX6GroupBytes;
    u32x4 lo;
    lo[0] = d[0]; lo[1] = d[1]; lo[2] = d[2]; lo[3] = d[3];
    u32x2 hi;
    hi[0] = d[4]; hi[1] = d[5];
    *(u32x4*)(yg + (f * 64 + lane) * 16) = lo;
    *(u32x2*)(yg + 2048 + (f * 64 + lane) * 8) = hi;
  }
};

// Rows that several waves of select_kernel share: the statistics kernel, which runs before it, clears their counts and
// (where several waves share a mask word) their mask words.
struct ClearRows {
  int32_t* row_counts;      // nullptr: nothing to clear
  uint64_t* mask;           // nullptr: words are stored whole
  __device__ __forceinline__ void row(const Geo& g, const Unit& u, int lane) const {
    const size_t r = (size_t)u.qh * g.n_qb + u.i;
    if (row_counts && lane == 0) row_counts[r] = 0;
    if (mask && lane < g.words) mask[r * g.words + lane] = 0;
  }
};

// ---------------------------------------------------------------------------
// Sink-local statistics (display equation of Sec. 3.2; first loop of Alg. 1)
// ---------------------------------------------------------------------------
//
// NT: 32-query tiles per wave.  NT = 2: one wave per row, four rows per workgroup.  NT = 1: the two waves of a workgroup
// take 32 queries each of one row; the same arithmetic per query, half of it per wave and step.
template <int MT, int NT>
__global__ __launch_bounds__(NT == 1 ? 128 : 256) void stats_kernel(Geo g, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                    const float* __restrict__ tau, int tau_len, float* __restrict__ thr,
                                                    float* __restrict__ m_out, float* __restrict__ l_out, ClearRows clear, PackFp6 pack) {
  if ((int)blockIdx.x >= pack.first) { pack.run(blockIdx.x); return; }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // wave-uniform by construction
  Unit u;
  int q0 = 0;                          // first query of this wave inside the row block
  if constexpr (NT == 1) {
    const int id = g.n_qb * g.group - 1 - (int)blockIdx.x / g.n_kvh;
    u.kvh = blockIdx.x % g.n_kvh;
    u.i = id / g.group;
    u.qh = u.kvh * g.group + id % g.group;
    q0 = 32 * wave;
  } else {
    u = unit_of(g, blockIdx.x, wave);
    if (!u.valid) return;
  }
  if (q0 == 0) clear.row(g, u, lane);
  const int c = lane & 31, h = lane >> 5;
  const float rsd = 0.08838834764831845f;   // 1 / sqrt(128)

  bf16x8 qf[NT][8];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const uint16_t* row = q + row_off(g.sq, u.qh, u.i * 64 + q0 + 32 * nt + c) + 8 * h;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[nt][s] = *(const bf16x8*)(row + 16 * s);
  }
  float m[NT], l[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) { m[nt] = -INFINITY; l[nt] = 0.0f; }
  const SeqPos sp = seq_pos(g, u.i);               // (variable-length batches: block indices inside the row's sequence)
  const int j_last = j_last_of(g, sp.il), local = local_of(g, j_last);
  // The sink-local blocks of the row, numbered t = 0 ..: the sink blocks that are not local ones, then the local
  // ones up to the diagonal.  They are swept in half-blocks of 32 keys (hs = t * MT + mt) with the operands of the
  // next half requested before the current one is multiplied: two register sets that swap roles, the last half
  // requesting itself again so that every step issues the same loads.
  const int lo_local = max(j_last - local + 1, 0);
  const int n_s = min(g.sink_blocks, lo_local);
  const int n_hs = (n_s + j_last - lo_local + 1) * MT;
  auto block_of = [&](int hs) { const int t = hs / MT; return t < n_s ? t : lo_local + (t - n_s); };
  auto fetch = [&](int hs, bf16x8 (&kk)[8]) __attribute__((always_inline)) {
    const uint16_t* row = k + row_off(g.sk, u.kvh, (sp.kb0 + block_of(hs)) * g.bk + 32 * (hs % MT) + c) + 8 * h;
#pragma unroll
    for (int s = 0; s < 8; ++s) kk[s] = *(const bf16x8*)(row + 16 * s);
  };
  const float kLog2e = 1.4426950408889634f;
  auto half = [&](int hs, const bf16x8 (&kk)[8], bf16x8 (&kn)[8]) __attribute__((always_inline)) {
    fetch(min(hs + 1, n_hs - 1), kn);
    f32x16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nt][r] = 0.0f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[s], qf[nt][s], acc[nt], 0, 0, 0);
    }
    const int j = block_of(hs), mt = hs % MT;
    // keys of this half that lie after a query row (only with SALE_FLAG_STATS_CAUSAL)
    const int ahead = j * g.bk + 32 * mt - sp.il * 64;      // first key of the half minus first query row
    if (g.stats_causal && ahead + 31 > 0) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (ahead + mfma32_row(r, lane) > q0 + 32 * nt + c) acc[nt][r] = -INFINITY;
    }
    // (VALU-bound: per score one half of a v_max3, one FMA that folds 1 / sqrt(d), log2(e) and the maximum,
    // one v_exp_f32 and one add)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      float mx = fmaxf(acc[nt][0], acc[nt][1]);
#pragma unroll
      for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, acc[nt][r]), acc[nt][r + 1]);
      const float m_new = fmaxf(m[nt], mx * rsd);      // rsd > 0: the maximum of the products is the product of the maximum
      const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
      const float mb = m_safe * kLog2e;
      float sum = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[nt][r], rsd * kLog2e, -mb));
      l[nt] = l[nt] * __builtin_amdgcn_exp2f(m[nt] * kLog2e - mb) + sum;
      m[nt] = m_new;
    }
  };
  {
    bf16x8 ka[8], kb[8];
    fetch(0, ka);                                   // (n_hs >= 1: the diagonal block is always local)
    for (int hs = 0; hs < n_hs; hs += 2) {
      half(hs, ka, kb);
      if (hs + 1 < n_hs) half(hs + 1, kb, ka);
    }
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float m_o = swap_half(m[nt]), l_o = swap_half(l[nt]);
    const float m_t = fmaxf(m[nt], m_o);
    const float m_safe = m_t == -INFINITY ? 0.0f : m_t;
    const float l_t = l[nt] * __expf(m[nt] - m_safe) + l_o * __expf(m_o - m_safe);
    if (h == 0) {
      const size_t idx = (size_t)u.qh * g.seq + u.i * 64 + q0 + 32 * nt + c;
      const float t = tau[tau_len == 1 ? 0 : u.qh % g.hq_per_b];
      thr[idx] = __logf(t * l_t) + m_t;
      if (m_out) m_out[idx] = m_t;
      if (l_out) l_out[idx] = l_t;
    }
  }
}

// The same statistics for GQA groups of a multiple of 4 heads: the 4 waves of a workgroup are then 4 heads of one
// KV head at the SAME query block (unit_of), i.e. they need the same key rows.  The kernel above is bound by the
// bytes its waves pull through the vector memory path (each wave reads its 5 key blocks itself); here a half-block of
// K (32 keys, 8 KB) is fetched ONCE per workgroup, staged through registers into LDS in MFMA operand order (two
// buffers, one barrier per half-block, the next half's global loads in flight meanwhile) and read from there by all
// four waves: 2.7 times fewer bytes from L2 / L1.
template <int MT>
__global__ __launch_bounds__(256) void stats_shared_kernel(Geo g, const uint16_t* __restrict__ q,
                                                           const uint16_t* __restrict__ k, const float* __restrict__ tau,
                                                           int tau_len, float* __restrict__ thr, float* __restrict__ m_out,
                                                           float* __restrict__ l_out, ClearRows clear, PackFp6 pack) {
  if ((int)blockIdx.x >= pack.first) { pack.run(blockIdx.x); return; }
  __shared__ bf16x8 k_lds[2][8 * 64];                // [buffer][s][lane] 16 bytes: the A operands of one half-block
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const Unit u = unit_of(g, blockIdx.x, wave);       // (group % 4 == 0: every wave is valid, all four share u.i and u.kvh)
  clear.row(g, u, lane);
  const int c = lane & 31, h = lane >> 5;
  const float rsd = 0.08838834764831845f;   // 1 / sqrt(128)

  bf16x8 qf[2][8];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const uint16_t* row = q + row_off(g.sq, u.qh, u.i * 64 + 32 * nt + c) + 8 * h;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[nt][s] = *(const bf16x8*)(row + 16 * s);
  }
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.0f, 0.0f};
  const SeqPos sp = seq_pos(g, u.i);
  const int j_last = j_last_of(g, sp.il), local = local_of(g, j_last);
  const int lo_local = max(j_last - local + 1, 0);
  const int n_s = min(g.sink_blocks, lo_local);
  const int n_hs = (n_s + j_last - lo_local + 1) * MT;
  auto block_of = [&](int hs) { const int t = hs / MT; return t < n_s ? t : lo_local + (t - n_s); };
  // Thread tid brings in chunks tid and tid + 256 of a half-block: chunk (s, lane') = the 16 bytes lane' of
  // fragment s needs (key row lane' % 32, channels 16 s + 8 (lane' / 32) ..).
  bf16x8 kreg[2];
  auto fetch = [&](int hs) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int id = tid + 256 * r, s = id >> 6, ln = id & 63;
      kreg[r] = *(const bf16x8*)(k + row_off(g.sk, u.kvh, (sp.kb0 + block_of(hs)) * g.bk + 32 * (hs % MT) + (ln & 31)) +
                                 16 * s + 8 * (ln >> 5));
    }
  };
  auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 2; ++r) k_lds[buf][tid + 256 * r] = kreg[r];
  };
  const float kLog2e = 1.4426950408889634f;
  fetch(0);
  stage(0);
  fetch(min(1, n_hs - 1));
  __syncthreads();
  for (int hs = 0; hs < n_hs; ++hs) {
    // the next half goes into the other buffer (every wave finished reading it before the last barrier), and
    // the one after next is requested
    stage((hs + 1) & 1);
    fetch(min(hs + 2, n_hs - 1));
    const bf16x8* kk = k_lds[hs & 1] + lane;
    f32x16 acc[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nt][r] = 0.0f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const bf16x8 a = kk[s * 64];
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[0][s], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[1][s], acc[1], 0, 0, 0);
    }
    const int j = block_of(hs), mt = hs % MT;
    const int ahead = j * g.bk + 32 * mt - sp.il * 64;      // first key of the half minus first query row
    if (g.stats_causal && ahead + 31 > 0) {                 // (only with SALE_FLAG_STATS_CAUSAL)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (ahead + mfma32_row(r, lane) > 32 * nt + c) acc[nt][r] = -INFINITY;
    }
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      float mx = fmaxf(acc[nt][0], acc[nt][1]);
#pragma unroll
      for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, acc[nt][r]), acc[nt][r + 1]);
      const float m_new = fmaxf(m[nt], mx * rsd);
      const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
      const float mb = m_safe * kLog2e;
      float sum = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[nt][r], rsd * kLog2e, -mb));
      l[nt] = l[nt] * __builtin_amdgcn_exp2f(m[nt] * kLog2e - mb) + sum;
      m[nt] = m_new;
    }
    __syncthreads();
  }
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const float m_o = swap_half(m[nt]), l_o = swap_half(l[nt]);
    const float m_t = fmaxf(m[nt], m_o);
    const float m_safe = m_t == -INFINITY ? 0.0f : m_t;
    const float l_t = l[nt] * __expf(m[nt] - m_safe) + l_o * __expf(m_o - m_safe);
    if (h == 0) {
      const size_t idx = (size_t)u.qh * g.seq + u.i * 64 + 32 * nt + c;
      const float t = tau[tau_len == 1 ? 0 : u.qh % g.hq_per_b];
      thr[idx] = __logf(t * l_t) + m_t;
      if (m_out) m_out[idx] = m_t;
      if (l_out) l_out[idx] = l_t;
    }
  }
}

// The 2 operand fragments (16 rows each) of 32-row group `grp` of an X6 array.
__device__ __forceinline__ void load_x6(__amdgpu_buffer_rsrc_t base, int grp, int lane, i32x8* f) {
  const int b = grp * kX6GroupBytes;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const u32x4 lo = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(base, lane * 16 + i * 1024, b, 0));
    const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(base, lane * 8 + 2048 + i * 512, b, 0));
    f[i][0] = lo[0]; f[i][1] = lo[1]; f[i][2] = lo[2]; f[i][3] = lo[3];
    f[i][4] = hi[0]; f[i][5] = hi[1]; f[i][6] = 0; f[i][7] = 0;
  }
}
// The same of 16 rows of nibble codes (64 bytes each).
__device__ __forceinline__ i32x8 fragment_of_nibbles(const uint8_t* rows16, int lane) {
  uint32_t d[6];
  pack_fp6(*(const u32x4*)(rows16 + (lane & 15) * 64 + 16 * (lane >> 4)), d);
  i32x8 f;
#pragma unroll
  for (int e = 0; e < 6; ++e) f[e] = d[e];
  f[6] = 0; f[7] = 0;
  return f;
}

// (16 K~ rows) (16 Q~ rows)^T, keys x queries, exact integers held in fp32: register r of a lane is key 4 (lane / 16) + r of
// query lane % 16.
__device__ __forceinline__ f32x4 qk_fp6(const i32x8& k, const i32x8& q) {
  const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(k, q, z, 2, 2, 0, 0, 0, 0);
}

// Maximum over the keys of a block of what one lane holds for query tile nt (16-bit estimate).
template <int MT>
__device__ __forceinline__ float lane_max32(const f32x16 acc[MT][2], int nt) {
  float mx = acc[0][nt][0];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = (mt == 0 ? 1 : 0); r < 16; ++r) mx = fmaxf(mx, acc[mt][nt][r]);
  return mx;
}

// One wave scores HPW query heads of one GQA group at the same query block, so every K~ fragment it
// loads feeds HPW x 4 MFMAs (HPW up to 4: launch_select).  What bounds it: 64 MFMAs of 16 cycles and 160 vector instructions
// per 64-key block and four heads on two waves per SIMD; the matrix pipe is busy 72 % of the clocks, which the power limit
// holds at 1.9 GHz.  (128K x 32 heads: 13.3 -> 12.7 ms against 32x32x64 products with their maxima taken head by head.)  A workgroup is 4 such waves (consecutive head sets / query blocks of one
// KV head); workgroups go round-robin over KV heads, longest rows first.  chunk > 0 (select_chunk): a wave scores
// blockIdx.y's `chunk` blocks of its rows only.  A mask word belongs to one wave if chunk is a multiple of 64,
// otherwise (a divisor of 64) its bits are joined by atomics, as are the counts (whole numbers: any order gives the same).
// (At least 2 waves per SIMD caps the register file at 256 VGPRs, which lets the MFMA results land in
// ordinary VGPRs instead of AGPRs that the max chain would have to copy out one by one.)
template <int HPW, int MT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void select_kernel(
    Geo g, const uint8_t* __restrict__ q4, const uint8_t* __restrict__ k6, const float* __restrict__ q_scale,
    const float* __restrict__ k_scale, const float* __restrict__ thr, uint64_t* __restrict__ mask,
    int32_t* __restrict__ row_counts, int chunk) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // wave-uniform by construction
  const int c = lane & 15;
  const int sets = g.group / HPW;                 // head sets per (KV head, query block)
  const int units = g.n_qb * sets;
  const int tiles = (units + 3) / 4;
  const int kvh = blockIdx.x % g.n_kvh;
  const int id = (tiles - 1 - blockIdx.x / g.n_kvh) * 4 + wave;
  if (id >= units) return;
  const int i = id / sets;
  const int qh0 = kvh * g.group + (id % sets) * HPW;
  SeqPos sp = seq_pos(g, i);
  sp.il = __builtin_amdgcn_readfirstlane(sp.il);      // (the same for the whole wave: all control flow below is scalar)
  sp.kb0 = __builtin_amdgcn_readfirstlane(sp.kb0);
  const int j_last = j_last_of(g, sp.il), local = local_of(g, j_last);
  // This wave's blocks of the row: r_lo .. r_hi - 1.
  const int r_lo = chunk ? (int)blockIdx.y * chunk : 0, r_hi = chunk ? min(r_lo + chunk, g.words * 64) : g.words * 64;
  const bool shared_word = chunk != 0 && chunk < 64;
  if (chunk && r_lo > j_last) {       // nothing of the row: its words stay empty (shared words were cleared)
    const int n_w = (r_hi - r_lo) >> 6;
    if (!shared_word)
      for (int e = lane; e < HPW * n_w; e += 64)
        mask[((size_t)(qh0 + e / n_w) * g.n_qb + i) * g.words + (r_lo >> 6) + e % n_w] = 0;
    return;
  }

  i32x8 qf[HPW][4];
  float th[HPW][4], cq[HPW];
#pragma unroll
  for (int a = 0; a < HPW; ++a) {
    // Q~ is used by this wave alone: its nibble codes are re-encoded here, once per row (K~, which every query
    // block reads again, comes re-encoded from the pre-pass).
#pragma unroll
    for (int qt = 0; qt < 4; ++qt) {
      qf[a][qt] = fragment_of_nibbles(q4 + ((size_t)(qh0 + a) * g.seq + i * 64 + 16 * qt) * 64, lane);
      th[a][qt] = thr[(size_t)(qh0 + a) * g.seq + i * 64 + 16 * qt + c];
    }
    cq[a] = q_scale[(size_t)(qh0 + a) * g.n_qb + i] * 0.08838834764831845f;   // s_q / sqrt(d)
  }
  const float* ks = k_scale + (size_t)kvh * g.n_kb;
  const int row_mid_hi = j_last - local;                          // the row's middle blocks: sink_blocks .. row_mid_hi
  const int mid_lo = max(g.sink_blocks, r_lo), mid_hi = min(row_mid_hi, r_hi - 1);      // those scored here
  const __amdgpu_buffer_rsrc_t kbuf = operand_buffer(k6 + ((size_t)kvh * g.n_kb + sp.kb0) * MT * kX6GroupBytes,
                                                     (j_last + 1) * MT * kX6GroupBytes);
  int count[HPW];
  uint64_t word[HPW];
  int wc = r_lo >> 6;                                               // mask word being assembled
  // Bits of word wc that are set without scoring: the sink and local blocks the row can see.
  auto fixed_bits = [&]() -> uint64_t {
    auto span = [&](int lo, int hi) -> uint64_t {                   // bits of blocks lo..hi that fall into word wc
      lo = max(max(lo, r_lo) - wc * 64, 0); hi = min(min(hi, r_hi - 1) - wc * 64, 63);
      return lo > hi ? 0ull : ((~0ull >> (63 - hi)) & (~0ull << lo));
    };
    return span(0, min(g.sink_blocks - 1, j_last)) | span(max(row_mid_hi + 1, 0), j_last);
  };
  // Completes word wc (store, count) and starts the next one.
  auto flush = [&]() {
#pragma unroll
    for (int a = 0; a < HPW; ++a) {
      uint64_t* at = mask + ((size_t)(qh0 + a) * g.n_qb + i) * g.words + wc;
      if (lane == 0) {
        if (shared_word) atomicOr((unsigned long long*)at, (unsigned long long)word[a]); else *at = word[a];
      }
      count[a] += __popcll(word[a]);
    }
    ++wc;
    const uint64_t fb = fixed_bits();
#pragma unroll
    for (int a = 0; a < HPW; ++a) word[a] = fb;
  };
  {
    const uint64_t fb = fixed_bits();
#pragma unroll
    for (int a = 0; a < HPW; ++a) { count[a] = 0; word[a] = fb; }
  }
  // The operands of a key block are requested one block ahead (two register sets that swap roles): the loads of
  // block j + 1 are in flight while block j is scored.  The last block requests itself again, so every step
  // issues the same loads and the wait counts stay exact.
  i32x8 kfa[2 * MT], kfb[2 * MT];
  float ska = 0.0f, skb = 0.0f;
  auto fetch = [&](int j, i32x8 (&kf)[2 * MT], float& sk) __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) load_x6(kbuf, j * MT + mt, lane, kf + 2 * mt);
    sk = ks[sp.kb0 + j];
  };
  // (as assembly, which says that the word is a scalar: the compiler kept the words in vector registers, 8 instructions a head)
  auto set_bits_if_any = [](uint64_t& w, uint64_t bits, uint64_t lanes) __attribute__((always_inline)) {
    uint64_t t;
    asm("s_cmp_lg_u64 %2, 0\n\ts_cselect_b64 %1, %3, 0\n\ts_or_b64 %0, %0, %1" : "+s"(w), "=&s"(t) : "s"(lanes), "s"(bits) : "scc");
  };
  auto score = [&](int j, const i32x8 (&kf)[2 * MT], float sk, i32x8 (&kn)[2 * MT], float& skn) __attribute__((always_inline)) {
    float cj[HPW];
#pragma unroll
    for (int a = 0; a < HPW; ++a) cj[a] = cq[a] * sk;
    __builtin_amdgcn_sched_barrier(0);      // (the wait for this block's scale must not become one for the next block's: scalar loads have no order)
    fetch(min(j + 1, mid_hi), kn, skn);
    while (wc < (j >> 6)) flush();
    // Unit u: query tile u % 4 of head u / 4, 2 MT products and the maximum over their 8 MT values per lane.  The products of
    // a unit are laid beside the maxima of the unit before it, one by one; neighbours share an operand.  (v_maximum3_f32:
    // for v_max3_f32 the compiler first quiets every product that enters, a fifth of the vector instructions.  All tiles are
    // always scored: most blocks fail, and a short-circuit is a branch.)
    constexpr int kTiles = 2 * MT, kUnits = 4 * HPW, kOps = 4 * MT + 2;
    f32x4 acc[2][kTiles];
    float m0 = 0.0f, m1 = 0.0f;
    bool pass[HPW];
    static_for<kUnits + 1>([&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value, v = u - 1;
      static_for<kTiles>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value, kt = u % 2 ? kTiles - 1 - k : k;
        if constexpr (u < kUnits) acc[u % 2][kt] = qk_fp6(kf[kt], qf[u / 4][u % 4]);
        if constexpr (v >= 0)
          static_for<(k + 1) * kOps / kTiles - k * kOps / kTiles>([&](auto oc) __attribute__((always_inline)) {
            constexpr int o = k * kOps / kTiles + decltype(oc)::value, a = v / 4, half = o / 2;
            auto at = [&](int n) { return acc[v % 2][n / 4][n % 4]; };
            auto max3 = [](float x, float y, float w) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), w); };
            constexpr int n1 = 4 * MT;      // the second chain's first value
            if constexpr (o < 4 * MT - 2) {      // two chains in turn
              if constexpr (half == 0) (o % 2 ? m1 : m0) = max3(at(o % 2 * n1), at(o % 2 * n1 + 1), at(o % 2 * n1 + 2));
              else if constexpr (o % 2 == 0) m0 = max3(m0, at(2 * half + 1), at(2 * half + 2));
              else m1 = max3(m1, at(n1 + 2 * half + 1), at(n1 + 2 * half + 2));
            } else if constexpr (o == 4 * MT - 2) m0 = max3(m0, at(n1 - 1), at(2 * n1 - 1));
            else if constexpr (o == 4 * MT - 1) m0 = __builtin_elementwise_maximum(m0, m1);
            else if constexpr (o == 4 * MT) m0 = m0 * cj[a];
            else pass[a] = (v % 4 == 0 ? false : pass[a]) | (m0 >= th[a][v % 4]);
          });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
#pragma unroll
    for (int a = 0; a < HPW; ++a) set_bits_if_any(word[a], 1ull << (j & 63), __builtin_amdgcn_ballot_w64(pass[a]));
  };
  if (mid_lo <= mid_hi) {
    fetch(mid_lo, kfa, ska);
    for (int j = mid_lo; j <= mid_hi; j += 2) {
      score(j, kfa, ska, kfb, skb);
      if (j + 1 <= mid_hi) score(j + 1, kfb, skb, kfa, ska);
    }
  }
  while (wc * 64 < r_hi) flush();
#pragma unroll
  for (int a = 0; a < HPW; ++a)
    if (lane == 0) {
      int32_t* at = row_counts + (size_t)(qh0 + a) * g.n_qb + i;
      if (chunk) atomicAdd(at, count[a]); else *at = count[a];
    }
}

// Appendix E ablation ("w/o QK Quant"): the same rule with the estimate taken from the 16-bit Q, K
// themselves (S~ = S, bf16 MFMA with fp32 accumulation): four times the MFMA work of the FP6 estimate.
template <int MT>
__global__ __launch_bounds__(256) void select16_kernel(Geo g, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                       const float* __restrict__ thr, uint64_t* __restrict__ mask,
                                                       int32_t* __restrict__ row_counts) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // wave-uniform by construction
  const Unit u = unit_of(g, blockIdx.x, wave);
  if (!u.valid) return;
  const int c = lane & 31, h = lane >> 5;
  const float rsd = 0.08838834764831845f;   // 1 / sqrt(128)
  bf16x8 qf[2][8];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const uint16_t* row = q + row_off(g.sq, u.qh, u.i * 64 + 32 * nt + c) + 8 * h;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[nt][s] = *(const bf16x8*)(row + 16 * s);
  }
  float th[2];
  th[0] = thr[(size_t)u.qh * g.seq + u.i * 64 + c];
  th[1] = thr[(size_t)u.qh * g.seq + u.i * 64 + 32 + c];
  uint64_t* mrow = mask + ((size_t)u.qh * g.n_qb + u.i) * g.words;
  const SeqPos sp = seq_pos(g, u.i);
  const int j_last = j_last_of(g, sp.il), local = local_of(g, j_last);
  int count = 0;
  for (int wc = 0; wc < g.words; ++wc) {
    uint64_t word = 0;
    const int j_end = min(64, j_last + 1 - wc * 64);
    for (int jj = 0; jj < j_end; ++jj) {
      const int j = wc * 64 + jj;
      if (in_sink_local(g, j, j_last, local)) { word |= 1ull << jj; continue; }
      f32x16 acc[MT][2];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[mt][nt][r] = 0.0f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const uint16_t* row = k + row_off(g.sk, u.kvh, (sp.kb0 + j) * g.bk + 32 * mt + c) + 8 * h;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const bf16x8 a = *(const bf16x8*)(row + 16 * s);
          acc[mt][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[0][s], acc[mt][0], 0, 0, 0);
          acc[mt][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[1][s], acc[mt][1], 0, 0, 0);
        }
      }
      const bool pass = (lane_max32<MT>(acc, 0) * rsd >= th[0]) || (lane_max32<MT>(acc, 1) * rsd >= th[1]);
      word |= (uint64_t)(__ballot(pass) != 0ull) << jj;
    }
    if (lane == 0) mrow[wc] = word;
    count += __popcll(word);
  }
  if (lane == 0) row_counts[(size_t)u.qh * g.n_qb + u.i] = count;
}

// Parity hook: the integer products themselves, one wave per key block, through the re-encoding (pack_fp6) and the product
// (qk_fp6) of select_kernel.  (Which takes K~ from the copies of the pre-pass, and looks at the products' maxima alone.)
template <int MT>
__global__ __launch_bounds__(64) void products_kernel(const uint8_t* __restrict__ q4_head, const uint8_t* __restrict__ k4_head,
                                                      int q_block, int k_begin, int n_kblocks, int32_t* __restrict__ out) {
  const int lane = threadIdx.x, c = lane & 15;
  const int jb = blockIdx.x;
  i32x8 qf[4], kf[2 * MT];
#pragma unroll
  for (int qt = 0; qt < 4; ++qt) qf[qt] = fragment_of_nibbles(q4_head + ((size_t)q_block * 4 + qt) * 1024, lane);
#pragma unroll
  for (int kt = 0; kt < 2 * MT; ++kt) kf[kt] = fragment_of_nibbles(k4_head + ((size_t)(k_begin + jb) * 2 * MT + kt) * 1024, lane);
  const size_t ld = (size_t)n_kblocks * (32 * MT);
#pragma unroll
  for (int kt = 0; kt < 2 * MT; ++kt)
#pragma unroll
    for (int qt = 0; qt < 4; ++qt) {
      const f32x4 acc = qk_fp6(kf[kt], qf[qt]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = 16 * kt + 4 * (lane >> 4) + r, qr = 16 * qt + c;
        out[(size_t)qr * ld + jb * (32 * MT) + key] = (int32_t)acc[r];
      }
    }
}

}  // namespace sale

using namespace sale;

namespace {

// Key blocks of a row that one wave of select_kernel scores (0: the whole row).  With one wave per row a call of few
// rows is as long as its longest row (4K tokens, 32 / 8 heads: 520 waves for 2048 places, 65 blocks one after the
// other), and up to 32K the last rows leave places empty.  The rows are cut so that at most
// 16384 (row, cut) waves are launched, more than half as many where the limits below do not stop it (about half of them lie
// above the diagonal and end at once), in powers of two from 8 blocks on (below, the re-encoding of Q~ costs more than the blocks:
// 4K took 62 us with 4).  Select call, before -> after with the 32x32x64 products it had then (the faster re-encoding of Q~
// is part of it; without the cut it gave 79.7 and 321): 4K tokens 85.7 -> 54.8 us, 16K 338 -> 301, 32K 1020 -> 990; with the
// present products 49.8, 287 and 974.  With twice as many waves 16K took 314 us, with four times 360; with half as many 304.
int select_chunk(const Geo& g, int hpw) {
  const long waves = (long)g.n_qb * (g.group / hpw) * g.n_kvh, blocks = (long)g.words * 64;
  long chunk = 8;
  while (chunk * 16384 < blocks * waves) chunk *= 2;
  return chunk < blocks ? (int)chunk : 0;
}

template <int MT>
int launch_select(const Geo& g, bool est16, const void* q, const void* k, const uint8_t* q4, const uint8_t* k4, uint8_t* k6,
                  const float* q_scale, const float* k_scale, const float* tau, int tau_len, const float* thr_c,
                  float* thr, uint64_t* block_mask, int32_t* row_counts, float* m_out, float* l_out, hipStream_t st) {
  const int tiles = (g.n_qb * g.group + 3) / 4;
  const int hpw = select_heads_per_wave(MT == 1, g.group, (long)g.n_qb * g.n_qh, g.words);
  const int chunk = est16 ? 0 : select_chunk(g, hpw);
  const ClearRows clear = {chunk ? row_counts : nullptr, chunk && chunk < 64 ? block_mask : nullptr};
  const long kgroups = est16 ? 0 : (long)g.n_kvh * (g.seq / 32);
  const bool shared = g.group % 4 == 0;      // (then 4 heads of one KV head at one query block share K)
  // Two waves per row while every row still finds a CU of its own.  Select call, us, one wave -> two: 252 rows (2.7K x 6
  // heads) 20.5 -> 14.5, 256 (8K x 2) 28.6 -> 22.0; beyond, 512 rows (8K x 4) 32.6 -> 31.7, 576 (6K x 6) 30.6 -> 34.5,
  // 1308 (7K x 12) 52.7 -> 58.5.  (Where K is shared it changes nothing: 50.8, 50.9 us at 4K.)
  const bool halves = !shared && (long)g.n_qb * g.n_qh <= 256;
  const int threads = halves ? 128 : 256;
  const PackFp6 pack = {k4, k6, kgroups, halves ? g.n_qb * g.n_qh : tiles * g.n_kvh};
  const dim3 stats_grid((unsigned)(pack.first + (kgroups + threads / 128 - 1) / (threads / 128)));
#define SALE_STATS_ARGS g, (const uint16_t*)q, (const uint16_t*)k, tau, tau_len, thr, m_out, l_out, clear, pack
  if (shared) stats_shared_kernel<MT><<<stats_grid, dim3(256), 0, st>>>(SALE_STATS_ARGS);
  else if (halves) stats_kernel<MT, 1><<<stats_grid, dim3(128), 0, st>>>(SALE_STATS_ARGS);
  else stats_kernel<MT, 2><<<stats_grid, dim3(256), 0, st>>>(SALE_STATS_ARGS);
#undef SALE_STATS_ARGS
  if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  if (est16) {
    select16_kernel<MT><<<dim3((unsigned)(tiles * g.n_kvh)), dim3(256), 0, st>>>(g, (const uint16_t*)q, (const uint16_t*)k,
                                                                                thr_c, block_mask, row_counts);
    return hipGetLastError() == hipSuccess ? SALE_OK : SALE_ERR_HIP;
  }
  const int wgs = (g.n_qb * (g.group / hpw) + 3) / 4;
  const dim3 grid((unsigned)(wgs * g.n_kvh), chunk ? (unsigned)((g.words * 64 + chunk - 1) / chunk) : 1u);
#define SALE_SELECT_ARGS g, q4, k6, q_scale, k_scale, thr_c, block_mask, row_counts, chunk
  if constexpr (MT == 2) {
    if (hpw == 4) select_kernel<4, MT><<<grid, dim3(256), 0, st>>>(SALE_SELECT_ARGS);
  }
  if (hpw == 2) select_kernel<2, MT><<<grid, dim3(256), 0, st>>>(SALE_SELECT_ARGS);
  if (hpw == 1) select_kernel<1, MT><<<grid, dim3(256), 0, st>>>(SALE_SELECT_ARGS);
#undef SALE_SELECT_ARGS
  return hipGetLastError() == hipSuccess ? SALE_OK : SALE_ERR_HIP;
}

}  // namespace

namespace {

// Checks shared by the two Selection-Pass entry points (everything but the workspace).
int check_select_args(const sale_params_t* p, const void* q, const void* k, const uint8_t* q4, const uint8_t* k4,
                      const float* q_scale, const float* k_scale, const float* tau, int32_t tau_len,
                      const uint64_t* block_mask, const int32_t* row_counts) {
  if (!p || !q || !k || !tau || !block_mask || !row_counts) return SALE_ERR_NULL_ARG;
  const bool est16 = (p->flags & SALE_FLAG_SELECT_16BIT) != 0;
  if (!est16 && (!q4 || !k4 || !q_scale || !k_scale)) return SALE_ERR_NULL_ARG;
  const int rc = validate_common(p, kGeomPath);
  if (rc != SALE_OK) return rc;
  if (tau_len != 1 && tau_len != p->n_q_heads) return SALE_ERR_BAD_SHAPE;
  return SALE_OK;
}

// The Selection-Pass on a workspace that has been checked.  Every byte of the workspace that a kernel reads is
// written earlier in the same call (thresholds and operand copies by the statistics launch),
// so nothing in it has to be cleared.
int run_select(const sale_params_t* p, const void* q, const void* k, const uint8_t* q4, const uint8_t* k4,
               const float* q_scale, const float* k_scale, const float* tau, int32_t tau_len, uint64_t* block_mask,
               int32_t* row_counts, float* m_out, float* l_out, void* ws, hipStream_t st) {
  const bool est16 = (p->flags & SALE_FLAG_SELECT_16BIT) != 0;
  Geo g = make_geo(p);
  float* thr = (float*)ws;
  uint8_t* k6 = (uint8_t*)ws + (size_t)g.n_qh * g.seq * sizeof(float);
  if (p->n_seqs > 0) {      // the per-block sequence table follows the operand copy
    int32_t* table = (int32_t*)(k6 + (size_t)g.n_kvh * (g.seq / 32) * kX6GroupBytes);
    const int rc = build_seq_table(p, table, st);
    if (rc != SALE_OK) return rc;
    g.seq_start = table;
  }
  return g.bk == 64 ? launch_select<2>(g, est16, q, k, q4, k4, k6, q_scale, k_scale, tau, tau_len, thr, thr, block_mask,
                                       row_counts, m_out, l_out, st)
                    : launch_select<1>(g, est16, q, k, q4, k4, k6, q_scale, k_scale, tau, tau_len, thr, thr, block_mask,
                                       row_counts, m_out, l_out, st);
}

}  // namespace

extern "C" int sale_select(const sale_params_t* p, const void* q, const void* k, const uint8_t* q4, const uint8_t* k4,
                           const float* q_scale, const float* k_scale, const float* tau, int32_t tau_len,
                           uint64_t* block_mask, int32_t* row_counts, float* m_out, float* l_out, void* ws,
                           size_t ws_bytes, void* stream) {
  const int rc = check_select_args(p, q, k, q4, k4, q_scale, k_scale, tau, tau_len, block_mask, row_counts);
  if (rc != SALE_OK) return rc;
  const size_t need = sale_workspace_bytes(p, SALE_WS_SELECT);
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 15)) return SALE_ERR_WORKSPACE;
  return run_select(p, q, k, q4, k4, q_scale, k_scale, tau, tau_len, block_mask, row_counts, m_out, l_out, ws,
                    (hipStream_t)stream);
}

// ---------------------------------------------------------------------------
// Selection-Pass for callers that cannot allocate: the workspace is a static device array of the library.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[SALE_SELECT_STATIC_MAX_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];      // per device: the address of that GPU's copy of `scratch`

// Device address of the current device's copy of `scratch` (in host code the array's name is only a handle:
// the address has to be asked for, once per device, with that device current).
int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SALE_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SALE_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return SALE_OK;
}

}  // namespace

extern "C" int sale_select_static(const sale_params_t* p, const void* q, const void* k, const uint8_t* q4,
                                  const uint8_t* k4, const float* q_scale, const float* k_scale, const float* tau,
                                  int32_t tau_len, uint64_t* block_mask, int32_t* row_counts, float* m_out,
                                  float* l_out, void* stream) {
  int rc = check_select_args(p, q, k, q4, k4, q_scale, k_scale, tau, tau_len, block_mask, row_counts);
  if (rc != SALE_OK) return rc;
  if (sale_workspace_bytes(p, SALE_WS_SELECT) > (size_t)SALE_SELECT_STATIC_MAX_BYTES) return SALE_ERR_WORKSPACE;
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != SALE_OK) return rc;
  return run_select(p, q, k, q4, k4, q_scale, k_scale, tau, tau_len, block_mask, row_counts, m_out, l_out, ws,
                    (hipStream_t)stream);
}

extern "C" int sale_qk_int4_products(const sale_params_t* p, const uint8_t* q4, const uint8_t* k4, int32_t q_head,
                                     int32_t q_block, int32_t k_block_begin, int32_t k_block_end, int32_t* out,
                                     void* stream) {
  if (!p || !q4 || !k4 || !out) return SALE_ERR_NULL_ARG;
  int rc = validate_common(p, kGeomPath);
  if (rc != SALE_OK) return rc;
  const Geo g = make_geo(p);
  if (q_head < 0 || q_head >= g.n_qh || q_block < 0 || q_block >= g.n_qb) return SALE_ERR_BAD_SHAPE;
  if (k_block_begin < 0 || k_block_end > g.n_kb || k_block_begin > k_block_end) return SALE_ERR_BAD_SHAPE;
  const int nkb = k_block_end - k_block_begin;
  if (nkb == 0) return SALE_OK;
  const uint8_t* qh = q4 + (size_t)q_head * g.seq * 64;
  const uint8_t* kh = k4 + (size_t)(q_head / g.group) * g.seq * 64;
  if (g.bk == 64)
    products_kernel<2><<<dim3((unsigned)nkb), dim3(64), 0, (hipStream_t)stream>>>(qh, kh, q_block, k_block_begin, nkb, out);
  else
    products_kernel<1><<<dim3((unsigned)nkb), dim3(64), 0, (hipStream_t)stream>>>(qh, kh, q_block, k_block_begin, nkb, out);
  return hipGetLastError() == hipSuccess ? SALE_OK : SALE_ERR_HIP;
}
