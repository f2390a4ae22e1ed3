// What the network's kernels share: direct loads into LDS, the order of the transposed values, conversions, lane reductions.
#pragma once
#include "common.hpp"

namespace pg {

// 16 bytes per lane straight from global memory into LDS (no register staging): the wave writes the
// 1 KB starting at LDS address `lds_addr` (wave-uniform), lane l at +16 l.  Issued through inline
// assembly so that the operand reads of the other LDS stage are not made to wait for it; completion
// is awaited explicitly (wait_dma) before the barrier that publishes the stage.  The statement overwrites m0
// without naming it as clobbered: m0 is a reserved register for this compiler (it refuses it in a clobber list
// and writes m0 itself directly before each instruction of its own that reads it), so no value of the
// surrounding code lives in m0 across the statement.  The address is a wave-uniform base plus a 32-bit byte offset per
// lane (no vector arithmetic per request).
__device__ __forceinline__ void dma16(uint32_t off, const void* base, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_addr) : "memory");
}
// 4 bytes per lane, 256 a wave
__device__ __forceinline__ void dma4(uint32_t off, const void* base, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds_addr) : "memory");
}
// wait until no more than LEFT of this wave's loads are in flight (they complete in order)
template <int LEFT = 0>
__device__ __forceinline__ void wait_dma() {
  static_assert(LEFT < 64, "six bits count them");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (LEFT & 15) | (LEFT >> 4) << 14);
}

// Where token t of a transposed value row is stored: in every 16 tokens the second and third group of four change places,
// which puts the eight tokens that a lane of the attention kernel multiplies at a time (4 h .. 4 h + 3 and 8 + 4 h .. 8 + 4 h + 3,
// the order in which the score accumulators hold the keys) into one 16-byte chunk.  Its own inverse: position t holds token
// value_slot(t).
__device__ __forceinline__ int value_slot(int t) { return (t & ~12) | ((t & 4) << 1) | ((t & 8) >> 1); }

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __builtin_bit_cast(float, (uint32_t)b << 16); }
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// as vectors, so that one conversion takes two values (converted one by one they are put together by two more instructions)
__device__ __forceinline__ uint32_t pack_bf16x2(float x, float y) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{x, y}, bf16x2));
}
__device__ __forceinline__ uint2 pack_bf16x4(float4 v) { return uint2{pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)}; }

// gelu_tanh(x) = x/2 (1 + tanh(y)) = x / (1 + exp(-2y)),  y = sqrt(2/pi) (x + 0.044715 x^3);
// the exponent is taken in base 2: -2 y log2(e) = x (K1 + K3 x^2)
__device__ __forceinline__ float gelu_tanh(float x) {
  constexpr float K1 = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
  constexpr float K3 = K1 * 0.044715f;
  const float z = x * __builtin_fmaf(x * x, K3, K1);
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z));
}

// orders this wave's LDS accesses around a hand-over between its lanes (LDS serves one wave's accesses in issue order;
// this keeps the compiler from moving them across the hand-over)
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Sum over 16 (wide) or 8 adjacent lanes, the same in each of them: a butterfly of data-parallel-primitive adds inside a row of
// 16 lanes (quad permutations, then the mirrored half row and row, whose lanes hold the other quads' equal sums).  Shuffles
// through LDS cost the dual-stream QKV launch of 28272 rows 80 of its 428 us.
template <int CTRL>
__device__ __forceinline__ float add_permuted(float v) {
  const int w = __builtin_bit_cast(int, v);
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(w, w, CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float head_sum(float v, bool wide) {
  v = add_permuted<0xB1>(v);                        // lane ^ 1
  v = add_permuted<0x4E>(v);                        // lane ^ 2
  v = add_permuted<0x141>(v);                       // 7 - lane inside 8 lanes
  return wide ? add_permuted<0x140>(v) : v;         // 15 - lane inside 16 lanes
}

// op over the four lanes 16 apart (one of each row of 16), the same in each of them
template <class Op>
__device__ __forceinline__ float across_rows(float v, Op op) {
  uint32_t b = __builtin_bit_cast(uint32_t, v);
  const auto r = __builtin_amdgcn_permlane16_swap(b, b, false, false);         // (own row or its neighbour's) twice
  v = op(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
  b = __builtin_bit_cast(uint32_t, v);
  const auto q = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (uint32_t)q[0]), __builtin_bit_cast(float, (uint32_t)q[1]));
}
// sum over the wave, the same in every lane
__device__ __forceinline__ float wave_allsum(float v) {
  return across_rows(head_sum(v, true), [](float x, float y) { return x + y; });
}

}  // namespace pg
