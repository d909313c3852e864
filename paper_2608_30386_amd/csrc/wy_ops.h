// Device helpers shared by the two chunkwise WY refresh kernels (gfx950): operand
// types, bf16 hi/lo splitting, MFMA wrappers and raw buffer loads.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace dasc_wy {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ inline float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// The lanes of one wave see each other's LDS writes: the wave waits for its LDS accesses
// to finish, and the compiler moves no memory access across the wait.
__device__ inline void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Raw buffer resource over exactly `bytes` bytes: a load whose total offset (vector +
// scalar + immediate) reaches past the end returns zero instead of touching memory.
// Tokens past a window therefore arrive as k = v = 0, g = 0, beta = 0, which are
// identity steps of the recurrence, and no load needs a clamp or a mask.
__device__ inline __amdgpu_buffer_rsrc_t rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, 0x00020000);
}
__device__ inline float ldf(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ inline f32x2 ldf2(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ inline f32x4 ldf4(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

// Two values split at once into packed bf16 words: hi = (bf16(x0), bf16(x1)) by one packed
// conversion, lo = the remainders (x - hi, exact in fp32) rounded to bf16.  The remainders
// take a shift or mask and a subtraction each.  A packed dot product with a unit selector
// would form a remainder in one instruction, but v_dot2_f32_bf16 shares the matrix pipe: next
// to a wave that issues MFMAs it takes 9-13 cycles against 4 for a plain VALU instruction
// (16 values split next to 32x32x16 MFMAs: 235 cycles this way, 339 with dot products; both
// 224 alone).
__device__ inline void split2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x0, x1}, bf16x2));
  const float r0 = x0 - __uint_as_float(hi << 16), r1 = x1 - __uint_as_float(hi & 0xFFFF0000u);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{r0, r1}, bf16x2));
}

// Eight values split at once, two per packed word.
__device__ inline void split8(const float* x, bf16x8& hi, bf16x8& lo) {
  uint4 h, l;
  split2(x[0], x[1], h.x, l.x);
  split2(x[2], x[3], h.y, l.y);
  split2(x[4], x[5], h.z, l.z);
  split2(x[6], x[7], h.w, l.w);
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}

__device__ inline f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// a b with both operands split: a_lo b_hi + a_hi b_lo + a_hi b_hi (small terms first)
__device__ inline f32x4 mma3(bf16x8 ah, bf16x8 al, bf16x8 bh, bf16x8 bl, f32x4 c) {
  c = mma(al, bh, c);
  c = mma(ah, bl, c);
  return mma(ah, bh, c);
}

// The 32x32x16 form: lane l holds A[l % 32][8 (l / 32) + e], B[8 (l / 32) + e][l % 32] and
// D[(i % 4) + 8 (i / 4) + 4 (l / 32)][l % 32].  The same rate on the matrix pipe as 16x16x32
// (32 cycles for twice the work), but it keeps other instructions of the SIMD from issuing for
// about 10 of its 32 cycles, where two 16x16x32 keep them for about 16.
__device__ inline f32x16 mmb(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ inline f32x16 mmb3(bf16x8 ah, bf16x8 al, bf16x8 bh, bf16x8 bl, f32x16 c) {
  c = mmb(al, bh, c);
  c = mmb(ah, bl, c);
  return mmb(ah, bh, c);
}

// 16x16x16 bf16 MFMA on packed words: lane (q, r) holds A[r][4q .. 4q + 3] and
// B[4q .. 4q + 3][r], two bf16 per word
__device__ inline f32x4 mma16(uint2 a, uint2 b, f32x4 c) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a),
                                                   __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}

// 16x16x4 fp32 MFMA: lane (q, r) holds A[r][q], B[q][r] and D[4q + i][r]
__device__ inline f32x4 mma32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

}  // namespace dasc_wy
