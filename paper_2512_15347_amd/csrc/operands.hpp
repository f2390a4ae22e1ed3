// What the GEMM and the attention kernels share: direct loads into LDS and the order of the transposed values.
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
// wait until none of this wave's loads is in flight
__device__ __forceinline__ void wait_dma() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Where token t of a transposed value row is stored: in every 16 tokens the second and third group of four change places,
// which puts the eight tokens that a lane of the attention kernel multiplies at a time (4 h .. 4 h + 3 and 8 + 4 h .. 8 + 4 h + 3,
// the order in which the score accumulators hold the keys) into one 16-byte chunk.  Its own inverse: position t holds token
// value_slot(t).
__device__ __forceinline__ int value_slot(int t) { return (t & ~12) | ((t & 4) << 1) | ((t & 8) >> 1); }

}  // namespace pg
