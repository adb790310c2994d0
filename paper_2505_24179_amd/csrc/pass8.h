// First pass over the operands of the quantized Computation-Pass: 8-bit codes of Q, column sums of K, column maxima of V.
// None depends on another, so they are the workgroups of ONE launch (256 threads each): beside the attention call's copies
// (rearrange_kv_kernel), or by themselves for the parity hooks (quantize8.hip).
#pragma once

#include "sale_common.h"

namespace sale {

// Exact column sums: bf16 values summed in fp64 lose nothing for any realistic value range, so the result
// does not depend on the order of the additions.  One workgroup per (KV head, 64-row tile): partial[c].
__device__ __forceinline__ void ksum_tile(const uint16_t* __restrict__ k, const Strided& lk, int tiles_per_head, int block,
                                          double* __restrict__ partial, double* other /* [128] */) {
  const int c = threadIdx.x & 127, phase = threadIdx.x >> 7;
  const uint16_t* rows = k + row_off(lk, block / tiles_per_head, (block % tiles_per_head) * 64 + phase * 32) + c;
  double s = 0.0;
#pragma unroll 8
  for (int r = 0; r < 32; ++r) s += (double)bf16_bits_to_float(rows[(size_t)r * lk.st]);
  if (phase == 1) other[c] = s;
  __syncthreads();
  if (phase == 0) partial[(size_t)block * 128 + c] = s + other[c];
}

// One workgroup per (head, 64-row block).  Thread t holds 32 channels (32 (t % 4) ..) of row t / 4.
// FRAG: codes go out in the operand order of the keys-as-rows product,
//   16: of v_mfma_i32_16x16x64_i8, [head][tile][kt 0..3][ks 0..1][lane 0..63] 16 bytes: channels 64ks + 16(lane/16) .. of
//       key row 16kt + lane%16;
//   32: of v_mfma_i32_32x32x32_i8, [head][tile][mt 0..1][ks 0..3][lane 0..63] 16 bytes: channels 32ks + 16(lane/32) .. of
//       key row 32mt + lane%32;
//   0: row-major [head][row][128 bytes].
template <int FRAG>
__device__ __forceinline__ void quantize8_block(const uint16_t* __restrict__ x, const Strided& lx,
                                                const float* __restrict__ mean, int tiles_per_head, int block,
                                                int8_t* __restrict__ codes, float* __restrict__ scale, float* wave_max /* [4] */) {
  const int t = threadIdx.x, r = t >> 2, cq = t & 3;
  const size_t blk = block;
  const u32x4* src = (const u32x4*)(x + row_off(lx, (int)(blk / tiles_per_head), (int)(blk % tiles_per_head) * 64 + r) + 32 * cq);
  float v[32];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const u32x4 w = __builtin_nontemporal_load(&src[i]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[8 * i + 2 * e] = __builtin_bit_cast(float, w[e] << 16);
      v[8 * i + 2 * e + 1] = __builtin_bit_cast(float, w[e] & 0xFFFF0000u);
    }
  }
  if (mean) {
    const float* m = mean + (blk / tiles_per_head) * 128 + 32 * cq;
#pragma unroll
    for (int e = 0; e < 32; ++e) v[e] = v[e] - m[e];
  }
  float amax = 0.0f;
#pragma unroll
  for (int e = 0; e < 32; ++e) amax = fmaxf(amax, fabsf(v[e]));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
  if ((t & 63) == 0) wave_max[t >> 6] = amax;
  __syncthreads();
  amax = fmaxf(fmaxf(wave_max[0], wave_max[1]), fmaxf(wave_max[2], wave_max[3]));
  const bool zero = amax == 0.0f;
  const float inv = zero ? 0.0f : 127.0f / amax;      // IEEE division, as in the definition
  if (t == 0) scale[blk] = zero ? 1.0f : amax / 127.0f;
  uint32_t packed[8];
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    uint32_t word = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const float y = rintf(v[4 * w + b] * inv);
      const int code = (int)fminf(fmaxf(y, -127.0f), 127.0f);
      word |= (uint32_t)(code & 0xFF) << (8 * b);
    }
    packed[w] = word;
  }
  u32x4 lo, hi;
  lo[0] = packed[0]; lo[1] = packed[1]; lo[2] = packed[2]; lo[3] = packed[3];
  hi[0] = packed[4]; hi[1] = packed[5]; hi[2] = packed[6]; hi[3] = packed[7];
  if (FRAG == 16) {
    u32x4* dst = (u32x4*)codes + blk * 512 + ((r >> 4) * 2 + (cq >> 1)) * 64 + 32 * (cq & 1) + (r & 15);
    dst[0] = lo;      // channels 32cq .. +15   -> lanes 32 (cq % 2) .. +15
    dst[16] = hi;     // channels 32cq+16 .. +31 -> the next 16 lanes
  } else if (FRAG == 32) {
    u32x4* dst = (u32x4*)codes + blk * 512 + ((r >> 5) * 4 + cq) * 64 + (r & 31);
    dst[0] = lo;      // channels 32cq .. +15   -> lanes 0..31
    dst[32] = hi;     // channels 32cq+16 .. +31 -> lanes 32..63
  } else {
    u32x4* dst = (u32x4*)(codes + (blk * 64 + r) * kHeadDim + 32 * cq);
    dst[0] = lo;
    dst[1] = hi;
  }
}

// Per (KV head, 64-row tile): partial[c] = max |v| over the tile's rows.
__device__ __forceinline__ void vamax_tile(const uint16_t* __restrict__ v, const Strided& lv, int tiles_per_head, int block,
                                           float* __restrict__ partial, float* other /* [128] */) {
  const int c = threadIdx.x & 127, phase = threadIdx.x >> 7;
  const uint16_t* rows = v + row_off(lv, block / tiles_per_head, (block % tiles_per_head) * 64 + phase * 32) + c;
  float m = 0.0f;
#pragma unroll 8
  for (int r = 0; r < 32; ++r) m = fmaxf(m, fabsf(bf16_bits_to_float(rows[(size_t)r * lv.st])));
  if (phase == 1) other[c] = m;
  __syncthreads();
  if (phase == 0) partial[(size_t)block * 128 + c] = fmaxf(m, other[c]);
}

struct Pass8 {
  int nq, nk, nv;      // workgroups: 64-row blocks of Q, 64-row tiles of K and of V (0: not asked for)
  int tiles;           // per head
  const uint16_t *q, *k, *v;
  int8_t* q8;
  float* q_scale;
  double* ksum;
  float* vamax;
  __host__ __device__ int blocks() const { return nq + nk + nv; }
  __device__ __forceinline__ void run(const Geo& g, int block, double* lds /* [128] */) const {
    if (block < nq) quantize8_block<0>(q, g.sq, nullptr, tiles, block, q8, q_scale, (float*)lds);
    else if (block < nq + nk) ksum_tile(k, g.sk, tiles, block - nq, ksum, lds);
    else vamax_tile(v, g.sv, tiles, block - nq - nk, vamax, (float*)lds);
  }
};

}  // namespace sale
