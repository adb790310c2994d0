// Shared device-side types and small helpers for the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "sale.h"

namespace sale {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr int kHeadDim = 128;   // d
constexpr int kBlockQ = 64;     // b_q
constexpr int kBlockK = 64;     // b_k of the Computation-Pass (the Selection-Pass also takes 32)
constexpr int kSegmentBlocks = 4;            // key blocks per segment (Appendix C)
constexpr int kMaskWordsMax = 64;            // longest mask row, in 64-bit words
constexpr int kMaxSeqLen = kMaskWordsMax * 64 * kBlockK;   // 262144 tokens (131072 with b_k = 32)

// f(integral_constant 0), f(integral_constant 1), ..: unrolled whatever its size, with indices that are constants.
template <class F, int... I>
__device__ __forceinline__ void static_for_each(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F f) { static_for_each(f, std::make_integer_sequence<int, N>{}); }

// How one of Q, K, V, O is laid out: element (flat head f = b * heads + h, token t, channel c) lies at
// (f / heads) * sb + (f % heads) * sh + t * st + c.
struct Strided {
  long long sb, sh, st;
  int heads;
};
__host__ __device__ __forceinline__ size_t row_off(const Strided& s, int flat_head, int token) {
  return (size_t)(flat_head / s.heads) * (size_t)s.sb + (size_t)(flat_head % s.heads) * (size_t)s.sh +
         (size_t)token * (size_t)s.st;
}

// Flattened geometry handed to kernels.
struct Geo {
  int n_qh;        // batch * n_q_heads
  int n_kvh;       // batch * n_kv_heads
  int hq_per_b;    // n_q_heads (to index tau)
  int group;       // n_q_heads / n_kv_heads
  int seq;         // N
  int n_qb;        // N / 64
  int bk;          // b_k: 64 or 32
  int n_kb;        // N / b_k
  int words;       // ceil(n_kb / 64)
  int sink_blocks;
  int local_blocks;
  int seg;         // segment size in key blocks (0 = no segment rule for the local area)
  int stats_causal;
  Strided sq, sk, sv, so;   // layouts of Q, K, V, O
  // Variable-length batch: [n_qb] first 64-row block of the sequence that block i belongs to (device), or
  // nullptr when every (batch, head) is one sequence.  n_qb, n_kb, seq then count the packed total and
  // `words` the mask words of the longest sequence.
  const int32_t* seq_start;
};

// Query block i of the packed token axis -> (its index inside its sequence, first key block of that sequence).
struct SeqPos { int il, kb0; };
__device__ __forceinline__ SeqPos seq_pos(const Geo& g, int i) {
  const int s0 = g.seq_start ? g.seq_start[i] : 0;
  SeqPos r;
  r.il = i - s0;
  r.kb0 = s0 * (kBlockQ / g.bk);
  return r;
}

__device__ __forceinline__ float bf16_bits_to_float(unsigned short b) {
  return __builtin_bit_cast(float, (unsigned)b << 16);
}

// Accumulator register r of lane `lane` in a 32x32 MFMA tile holds row
// 8*(r/4) + 4*(lane/32) + r%4 of column lane%32.
__device__ __forceinline__ int mfma32_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// Value held by the other half of the wave (lane ^ 32).
__device__ __forceinline__ float swap_half(float x) { return __shfl_xor(x, 32, 64); }

// Reads an integer register as a float.  The empty statement hides the value's origin from the optimizer: with
// this compiler, float arithmetic on elements 1.. of an integer vector that an intrinsic returned and that is
// reinterpreted as floats was folded away as if those elements were NaN (only element 0 survived a maximum).
__device__ __forceinline__ float int_bits_as_float(int x) {
  asm("" : "+v"(x));
  return __builtin_bit_cast(float, x);
}

__device__ __forceinline__ f32x4 int_bits_as_floats(i32x4 x) {      // (the same for four)
  f32x4 y = __builtin_bit_cast(f32x4, x);
  asm("" : "+v"(y));
  return y;
}

__device__ __forceinline__ f32x16 int_bits_as_floats(i32x16 x) {
  f32x16 y = __builtin_bit_cast(f32x16, x);
  asm("" : "+v"(y));
  return y;
}

// Between what the lanes of a wave write to LDS and what other lanes of it read: holds the compiler to that order (the hardware
// keeps it).  No instruction.
__device__ __forceinline__ void wave_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Some value, for an operand that does not matter: no instruction.
__device__ __forceinline__ int any_int() {
  int x;
  asm volatile("" : "=v"(x));      // (volatile: one register for all of them would be copied for each)
  return x;
}

// max(x, x of lane ^ 32) without going through LDS: v_permlane32_swap exchanges the upper 32 lanes of its
// first register with the lower 32 lanes of its second, so with x in both it leaves the lower half's values in
// both halves of one register and the upper half's in the other.  Written as inline assembly on purpose: through
// the builtin the compiler kept the instruction but dropped the maximum of the two results (it used the first
// alone), which went unnoticed as long as every consumer only needed SOME common reference value per row.
// (s_nop 1: the wait states the instruction needs after the VALU write of its operands.)
__device__ __forceinline__ float max_with_other_half(float x) {
  float lo = x, hi = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
  return fmaxf(lo, hi);
}

// The maximum over the four lanes that are equal modulo 16 (v_permlane16_swap exchanges odd rows of 16 lanes with even ones).
// A NaN stays.
__device__ __forceinline__ float max_over_rows(float v) {
  float w = v;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(v), "+v"(w));
  w = v = __builtin_elementwise_maximum(v, w);
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(v), "+v"(w));
  return __builtin_elementwise_maximum(v, w);
}

// Operand copies in fragment order are read through buffer descriptors: an address is descriptor base + scalar tile
// offset + lane * 16 + immediate, so a load costs no vector instruction for its address (with plain pointers the step
// of the attention kernel spent 26 of its 290 vector instructions besides the MFMAs on 64-bit addresses; bf16 sparse
// attention at 64K with 32-key blocks 7.94 -> 7.80 ms, dense at 32K 7.69 -> 7.61 ms; Selection-Pass at 128K 13.65 -> 13.32 ms).
// Base and size must be wave-uniform.  A descriptor covers one KV head of one sequence: at most 64 MB.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_buffer(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
}
// Chunk n (lane-contiguous 1 KB) from the scalar byte offset t on.
template <class T>
__device__ __forceinline__ T load_chunk(__amdgpu_buffer_rsrc_t r, int lane16, int t, int n) {
  return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, lane16 + (n & 3) * 1024, t + (n & ~3) * 1024, 0));
}

// Unit = (flattened query head, 64-row query block): the work of one wave.
// Units of one KV head are numbered block-major, head-in-group minor, so the
// four waves of a workgroup share their K (and V) rows.  Workgroups are dealt
// round-robin over KV heads (one KV head per XCD / L2 when there are 8) and
// longest rows first.
struct Unit {
  int kvh;     // flattened batch * kv head
  int qh;      // flattened batch * q head
  int i;       // query block
  bool valid;  // false for the padding waves of the last workgroup
};

__device__ __forceinline__ Unit unit_of(const Geo& g, int block, int wave) {
  const int units = g.n_qb * g.group;
  const int tiles = (units + 3) / 4;
  Unit u;
  u.kvh = block % g.n_kvh;
  const int t = tiles - 1 - block / g.n_kvh;
  const int id = t * 4 + wave;
  u.valid = id < units;
  u.i = u.valid ? id / g.group : 0;
  u.qh = u.kvh * g.group + (u.valid ? id % g.group : 0);
  return u;
}

// Which geometry a call accepts: any mix of 32 / 64 (quantization alone), b_q = 64 with b_k = 64 or 32
// and at most 4096 key blocks (everything else).
enum GeomClass { kGeomQuantize, kGeomPath };
int validate_common(const sale_params_t* p, GeomClass cls);
// attention launcher shared by the attention entry points and the calibration (attention.hip)
int launch_attn_rows(const sale_params_t* p, const void* q, const void* k, const void* v, const uint64_t* mask,
                     const int32_t* row_counts, void* o, float* o32, float* lse, void* ws, size_t ws_bytes, hipStream_t st);
// Bytes of an attention workspace without parking slots (sparse) / of the dense kernel's workspace.
size_t attn_fixed_bytes(const sale_params_t* p, bool sparse);
size_t dense_order_bytes(const sale_params_t* p);      // order in which a dense call of packed sequences issues its rows
constexpr size_t kParkedRowBytes = 2048 * 16 + 256 * 4;      // fp32 O^T accumulators + running max / sum of one row block
Geo make_geo(const sale_params_t* p);
int longest_sequence(const sale_params_t* p);      // tokens
// Variable-length batches: bytes of the per-block sequence table at the end of a workspace (0 without one), and
// the kernel launches that fill it from the host offsets.
size_t seq_table_bytes(const sale_params_t* p);
int build_seq_table(const sale_params_t* p, int32_t* table, hipStream_t st);
size_t calibrate_workspace_bytes(const sale_params_t* p);

// 8-bit operands of the quantized Computation-Pass (quantize8.hip).
struct Int8Operands {
  int8_t* q8;        // [q head][N][128] codes, row-major
  int8_t* k8;        // codes of the smoothed K: MFMA fragment order (attention) or row-major (parity hook)
  float* q_scale;    // [q head][N / 64]
  float* k_scale;    // [kv head][N / 64]
  float* k_mean;     // [kv head][128]
  double* partial;   // [kv head][N / 64][128] column sums per tile
};
// FP8 V of the low-precision second product (quantize8.hip).
struct Fp8Operands {
  uint8_t* v8;       // values: MFMA fragment order (attention) or row-major (parity hook)
  float* v_scale;    // [kv head][128]
  float* v_inv;      // [kv head][128]: 448 / amax
  float* partial;    // [kv head][N / 64][128] per-tile maxima
};
size_t fp8_operand_bytes(const sale_params_t* p);
Fp8Operands carve_fp8_operands(const sale_params_t* p, void* base);
size_t int8_operand_bytes(const sale_params_t* p);
Int8Operands carve_int8_operands(const sale_params_t* p, void* base);
struct Pass8;      // (pass8.h)
Pass8 make_pass8(const sale_params_t* p, const void* q, const void* k, const void* v, const Int8Operands* w8, const Fp8Operands* wv);
int launch_operands8(const sale_params_t* p, const void* k, const void* v, const Int8Operands* w8, const Fp8Operands* wv, int kfrag,
                     hipStream_t st);

}  // namespace sale
