// Operands of the quantized Computation-Pass (Sec. 3.4 "Integration with SageAttention"): the mean key of
// every KV head is subtracted from its keys (the softmax cancels the shift), then Q and the smoothed K get
// symmetric 8-bit codes in [-127, 127] with one fp32 scale per (head, 64-row block) - the arithmetic of the
// 4-bit quantizer with 127 in place of 7.
//
// HBM-bound and tiny next to the attention they feed (K is read twice, Q once), so at short lengths their launches are what they
// cost.  Three launches: what needs nothing else (Pass8, beside the attention call's own first launch), the small reductions of
// its partial results, and what needs those.  As five launches (eight with FP8 V) the whole attention call took, us, before ->
// now: 64 tokens x 1 head int8 17.4 -> 13.7, FP8 22.5 -> 14.7; 1024 rows of 2K tokens 58 -> 53, 65 -> 52; 4160 tokens x 32 heads
// 120 -> 114, 125 -> 113; 64K tokens the same.
#include "pass8.h"

namespace sale {

__global__ __launch_bounds__(256) void pass8_kernel(Geo g, Pass8 pass) {
  __shared__ double lds[128];
  pass.run(g, blockIdx.x, lds);
}

// mean[kvh][c] = fp32(sum over the head's tiles / N).  One workgroup of 1024 threads per KV head: 8 threads per
// channel take every 8th tile each, four loads in flight, and meet in LDS.  (The partial sums are fp64 sums of
// bf16 values: exact for any data whose exponents span less than 53 - 8 - log2(N) bits, so the order is free.)
__device__ __forceinline__ void kmean_head(const double* __restrict__ partial, int tiles, int seq, int head,
                                           float* __restrict__ mean, double (*part)[128]) {
  const int c = threadIdx.x & 127, ph = threadIdx.x >> 7;
  const double* p = partial + (size_t)head * tiles * 128 + c;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  int t = ph;
  for (; t + 24 < tiles; t += 32) {
    s0 += p[(size_t)t * 128]; s1 += p[(size_t)(t + 8) * 128]; s2 += p[(size_t)(t + 16) * 128]; s3 += p[(size_t)(t + 24) * 128];
  }
  for (; t < tiles; t += 8) s0 += p[(size_t)t * 128];
  part[ph][c] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  if (ph == 0) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += part[i][c];
    mean[head * 128 + c] = (float)(s / (double)seq);
  }
}

// ---------------------------------------------------------------------------
// V of the low-precision second product: OCP FP8 E4M3 values with one fp32 scale per (KV head, channel),
//   amax = max over the head's N tokens of |v|;  scale = amax / 448;  value = fp8(v * (448 / amax))
// (IEEE fp32, one multiply, round to nearest even; an all-zero channel gets scale 1 and values 0).
// ---------------------------------------------------------------------------
// Per KV head: scale[c] = amax / 448 and inv[c] = 448 / amax (1 and 0 for an all-zero channel).  1024 threads as
// in kmean_head.
__device__ __forceinline__ void vscale_head(const float* __restrict__ partial, int tiles, int head, float* __restrict__ scale,
                                            float* __restrict__ inv, float (*part)[128]) {
  const int c = threadIdx.x & 127, ph = threadIdx.x >> 7;
  const float* p = partial + (size_t)head * tiles * 128 + c;
  float m0 = 0.0f, m1 = 0.0f, m2 = 0.0f, m3 = 0.0f;
  int t = ph;
  for (; t + 24 < tiles; t += 32) {
    m0 = fmaxf(m0, p[(size_t)t * 128]); m1 = fmaxf(m1, p[(size_t)(t + 8) * 128]);
    m2 = fmaxf(m2, p[(size_t)(t + 16) * 128]); m3 = fmaxf(m3, p[(size_t)(t + 24) * 128]);
  }
  for (; t < tiles; t += 8) m0 = fmaxf(m0, p[(size_t)t * 128]);
  part[ph][c] = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
  __syncthreads();
  if (ph == 0) {
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, part[i][c]);
    const bool zero = amax == 0.0f;
    scale[head * 128 + c] = zero ? 1.0f : amax / 448.0f;
    inv[head * 128 + c] = zero ? 0.0f : 448.0f / amax;
  }
}

// Workgroups 0 .. n_mean - 1: a KV head's mean key; the rest: its scales of V.
__global__ __launch_bounds__(1024) void reduce8_kernel(Int8Operands w8, Fp8Operands wv, int n_mean, int tiles, int seq) {
  __shared__ double lds[8][128];
  const int b = blockIdx.x;
  if (b < n_mean) kmean_head(w8.partial, tiles, seq, b, w8.k_mean, lds);
  else vscale_head(wv.partial, tiles, b - n_mean, wv.v_scale, wv.v_inv, (float (*)[128])lds);
}

__device__ __forceinline__ uint32_t fp8x4(float a, float b, float c, float d) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  return (uint32_t)w;
}

// One workgroup per (KV head, 64-key tile).
// FRAG: the values go out as the A operand of v_mfma_f32_32x32x64_f8f6f4 for O^T += V^T P^T,
//   [head][tile][dt 0..3][j 0..1][lane 0..63] 16 bytes: channel 32 dt + lane % 32 of the 16 keys
//   32 j + 8 (e / 4) + 4 (lane / 32) + e % 4, e = 0..15
// (the order in which the S^T accumulator registers of half-tile j hand P^T to the second product);
// otherwise row-major [head][key][128 bytes].
template <bool FRAG>
__device__ __forceinline__ void quantize_v8_tile(const uint16_t* __restrict__ v, const Strided& lv, int tiles_per_head, int block,
                                                 const float* __restrict__ inv, uint8_t* __restrict__ out,
                                                 float* sv /* [64][kHeadDim + 1]: v * inv, rows padded by one bank */) {
  const int tid = threadIdx.x;
  const size_t tile = block;
  const int head = (int)(tile / tiles_per_head);
  const uint16_t* vt = v + row_off(lv, head, (int)(tile % tiles_per_head) * 64);
  const float* iv = inv + (size_t)head * 128;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int chunk = tid + 256 * r;
    const int row = chunk >> 4, col = (chunk & 15) * 8;
    const u32x4 w = *(const u32x4*)(vt + (size_t)row * lv.st + col);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sv[row * (kHeadDim + 1) + col + 2 * e] = __builtin_bit_cast(float, w[e] << 16) * iv[col + 2 * e];
      sv[row * (kHeadDim + 1) + col + 2 * e + 1] = __builtin_bit_cast(float, w[e] & 0xFFFF0000u) * iv[col + 2 * e + 1];
    }
  }
  __syncthreads();
  if (FRAG) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int oc = tid + 256 * r;
      const int lane = oc & 63, j = (oc >> 6) & 1, dt = oc >> 7;
      const int d = 32 * dt + (lane & 31), h = lane >> 5;
      u32x4 o4;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int key = 32 * j + 8 * w + 4 * h;      // e = 4 w .. 4 w + 3
        o4[w] = fp8x4(sv[key * (kHeadDim + 1) + d], sv[(key + 1) * (kHeadDim + 1) + d], sv[(key + 2) * (kHeadDim + 1) + d],
                      sv[(key + 3) * (kHeadDim + 1) + d]);
      }
      ((u32x4*)out)[tile * 512 + oc] = o4;
    }
  } else {
    const int row = tid >> 2, cq = tid & 3;
    const float* src = sv + row * (kHeadDim + 1) + 32 * cq;
    u32x4 lo, hi;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      lo[w] = fp8x4(src[4 * w], src[4 * w + 1], src[4 * w + 2], src[4 * w + 3]);
      hi[w] = fp8x4(src[16 + 4 * w], src[17 + 4 * w], src[18 + 4 * w], src[19 + 4 * w]);
    }
    u32x4* dst = (u32x4*)(out + (tile * 64 + row) * kHeadDim + 32 * cq);
    dst[0] = lo;
    dst[1] = hi;
  }
}

// Workgroups 0 .. n_k - 1: codes of a 64-row tile of the smoothed K (layout KFRAG of quantize8_block); the rest: FP8 values of
// one of V (VFRAG: in fragment order; none with the bf16 second product, layout 16).
template <int KFRAG, bool VFRAG>
__global__ __launch_bounds__(256) void codes8_kernel(Geo g, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                     Int8Operands w8, Fp8Operands wv, int n_k, int tiles) {
  __shared__ float lds[KFRAG == 16 ? 4 : 64 * (kHeadDim + 1)];
  const int b = blockIdx.x;
  if (b < n_k) quantize8_block<KFRAG>(k, g.sk, w8.k_mean, tiles, b, w8.k8, w8.k_scale, lds);
  else if constexpr (KFRAG != 16) quantize_v8_tile<VFRAG>(v, g.sv, tiles, b - n_k, wv.v_inv, wv.v8, lds);
}

size_t fp8_operand_bytes(const sale_params_t* p) {
  const size_t kvrows = (size_t)p->batch * p->n_kv_heads * p->seq_len;
  // V values | scales | inverse scales | per-tile maxima
  return kvrows * kHeadDim + 2 * (size_t)p->batch * p->n_kv_heads * 128 * sizeof(float) + (kvrows / 64) * 128 * sizeof(float) + 64;
}

Fp8Operands carve_fp8_operands(const sale_params_t* p, void* base) {
  const size_t kvrows = (size_t)p->batch * p->n_kv_heads * p->seq_len;
  const size_t heads = (size_t)p->batch * p->n_kv_heads;
  Fp8Operands w;
  uint8_t* b = (uint8_t*)base;
  w.v8 = b;                   b += kvrows * kHeadDim;
  w.v_scale = (float*)b;      b += heads * 128 * sizeof(float);
  w.v_inv = (float*)b;        b += heads * 128 * sizeof(float);
  w.partial = (float*)b;
  return w;
}

size_t int8_operand_bytes(const sale_params_t* p) {
  const size_t rows = (size_t)p->batch * p->n_q_heads * p->seq_len;
  const size_t kvrows = (size_t)p->batch * p->n_kv_heads * p->seq_len;
  // Q codes | K codes | Q scales | K scales | key means | column-sum partials (fp64)
  return rows * kHeadDim + kvrows * kHeadDim + (rows / 64 + kvrows / 64) * sizeof(float) +
         (size_t)p->batch * p->n_kv_heads * 128 * sizeof(float) + (kvrows / 64) * 128 * sizeof(double) + 64;
}

Int8Operands carve_int8_operands(const sale_params_t* p, void* base) {
  const size_t rows = (size_t)p->batch * p->n_q_heads * p->seq_len;
  const size_t kvrows = (size_t)p->batch * p->n_kv_heads * p->seq_len;
  Int8Operands w;
  uint8_t* b = (uint8_t*)base;
  w.q8 = (int8_t*)b;                       b += rows * kHeadDim;
  w.k8 = (int8_t*)b;                       b += kvrows * kHeadDim;
  w.partial = (double*)b;                  b += (kvrows / 64) * 128 * sizeof(double);   // 8-byte aligned: all sizes above are multiples of 64
  w.q_scale = (float*)b;                   b += (rows / 64) * sizeof(float);
  w.k_scale = (float*)b;                   b += (kvrows / 64) * sizeof(float);
  w.k_mean = (float*)b;
  return w;
}

// The first pass over what is asked for (nullptr: not).
Pass8 make_pass8(const sale_params_t* p, const void* q, const void* k, const void* v, const Int8Operands* w8, const Fp8Operands* wv) {
  const int n_kvh = p->batch * p->n_kv_heads, n_qh = p->batch * p->n_q_heads, tiles = p->seq_len / 64;
  Pass8 s = {};
  s.tiles = tiles;
  if (w8) {
    s.nq = n_qh * tiles; s.nk = n_kvh * tiles;
    s.q = (const uint16_t*)q; s.k = (const uint16_t*)k;
    s.q8 = w8->q8; s.q_scale = w8->q_scale; s.ksum = w8->partial;
  }
  if (wv) { s.nv = n_kvh * tiles; s.v = (const uint16_t*)v; s.vamax = wv->partial; }
  return s;
}

// What follows the first pass.  kfrag: layout of the codes of K (16 or 32: in fragment order, see quantize8_block; 0: row-major);
// V goes into fragment order with 32.
int launch_operands8(const sale_params_t* p, const void* k, const void* v, const Int8Operands* w8, const Fp8Operands* wv, int kfrag,
                     hipStream_t st) {
  const int n_kvh = p->batch * p->n_kv_heads, tiles = p->seq_len / 64, mean = w8 ? n_kvh : 0, scale = wv ? n_kvh : 0;
  const Geo g = make_geo(p);
  const Int8Operands a = w8 ? *w8 : Int8Operands{};
  const Fp8Operands b = wv ? *wv : Fp8Operands{};
  reduce8_kernel<<<dim3((unsigned)(mean + scale)), dim3(1024), 0, st>>>(a, b, mean, tiles, p->seq_len);
  if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  const dim3 grid((unsigned)((mean + scale) * tiles));
#define SALE_CODES_ARGS g, (const uint16_t*)k, (const uint16_t*)v, a, b, mean * tiles, tiles
  if (kfrag == 16) codes8_kernel<16, false><<<grid, dim3(256), 0, st>>>(SALE_CODES_ARGS);
  else if (kfrag == 32) codes8_kernel<32, true><<<grid, dim3(256), 0, st>>>(SALE_CODES_ARGS);
  else codes8_kernel<0, false><<<grid, dim3(256), 0, st>>>(SALE_CODES_ARGS);
#undef SALE_CODES_ARGS
  return hipGetLastError() == hipSuccess ? SALE_OK : SALE_ERR_HIP;
}

namespace {
// All of it, for the parity hooks.
int all_operands8(const sale_params_t* p, const void* q, const void* k, const void* v, const Int8Operands* w8, const Fp8Operands* wv,
                  hipStream_t st) {
  const Pass8 pass = make_pass8(p, q, k, v, w8, wv);
  pass8_kernel<<<dim3((unsigned)pass.blocks()), dim3(256), 0, st>>>(make_geo(p), pass);
  if (hipGetLastError() != hipSuccess) return SALE_ERR_HIP;
  return launch_operands8(p, k, v, w8, wv, 0, st);
}
}  // namespace

}  // namespace sale

using namespace sale;

extern "C" int sale_attn_int8_operands(const sale_params_t* p, const void* q, const void* k, int8_t* q8, int8_t* k8,
                                       float* q_scale8, float* k_scale8, float* k_mean, void* ws, size_t ws_bytes,
                                       void* stream) {
  if (!p || !q || !k || !q8 || !k8 || !q_scale8 || !k_scale8 || !k_mean) return SALE_ERR_NULL_ARG;
  int rc = validate_common(p, kGeomPath);
  if (rc != SALE_OK) return rc;
  const size_t need = sale_workspace_bytes(p, SALE_WS_INT8_OPERANDS);
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 15)) return SALE_ERR_WORKSPACE;
  Int8Operands w;
  w.q8 = q8; w.k8 = k8; w.q_scale = q_scale8; w.k_scale = k_scale8; w.k_mean = k_mean;
  w.partial = (double*)ws;
  return all_operands8(p, q, k, nullptr, &w, nullptr, (hipStream_t)stream);
}

extern "C" int sale_attn_fp8_operands(const sale_params_t* p, const void* v, uint8_t* v8, float* v_scale, void* ws,
                                      size_t ws_bytes, void* stream) {
  if (!p || !v || !v8 || !v_scale) return SALE_ERR_NULL_ARG;
  int rc = validate_common(p, kGeomPath);
  if (rc != SALE_OK) return rc;
  const size_t need = sale_workspace_bytes(p, SALE_WS_FP8_OPERANDS);
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 15)) return SALE_ERR_WORKSPACE;
  Fp8Operands w;
  w.v8 = v8; w.v_scale = v_scale;
  w.v_inv = (float*)ws;
  w.partial = w.v_inv + (size_t)p->batch * p->n_kv_heads * 128;
  return all_operands8(p, nullptr, nullptr, v, nullptr, &w, (hipStream_t)stream);
}
