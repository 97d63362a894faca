// Copies from global memory into LDS that pass no registers, and the waits that go with them (used by
// the contraction kernels' software pipelines).
#ifndef LT_DMA_H_
#define LT_DMA_H_
#include <hip/hip_runtime.h>

namespace ltk {

// One wave instruction of such a copy: 16 bytes per lane, each from an address of its own (base +
// lane_off), to 1 KiB of consecutive LDS.  Written in assembly on purpose: the compiler orders every
// later LDS read behind every copy it knows to be in flight (and loses track of them around a
// loop's back edge), so a pipeline deeper than one slice needs copies it does not know about and
// waits that the code spells out (landed(), below).  M0 holds the LDS base of the instruction;
// nothing else in the loop uses it, and the interpreter's register indexing sets it afresh.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy_1k(const void* base, uint32_t lane_off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_base), "v"(lane_off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

// Wait until at most `outstanding` of this wave's copies are still in flight (they complete in
// order).  s_waitcnt immediate: vmcnt in bits 3:0 and 15:14, the other counters left alone.
template <uint32_t outstanding>
__device__ __forceinline__ void landed() {
  static_assert(outstanding < 64u, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((int)((outstanding & 15u) | ((outstanding >> 4) << 14) | 0x0f70u));
}

// The same, and every LDS read of this wave has returned as well (lgkmcnt = 0).
template <uint32_t outstanding>
__device__ __forceinline__ void landed_and_read() {
  static_assert(outstanding < 64u, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((int)((outstanding & 15u) | ((outstanding >> 4) << 14) | 0x0070u));
}

}  // namespace ltk
#endif  // LT_DMA_H_
