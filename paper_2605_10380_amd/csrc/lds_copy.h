// Copies from memory to LDS without registers in between (global_load_lds), and the waits that go with them.
#pragma once

#include <hip/hip_runtime.h>

namespace ax {

// The 64 lanes of a wavefront copy 64 x 16 bytes to 1 KB of LDS at `lds` (wavefront-uniform byte address): lane l's 16 bytes come from
// base + off and land at lds + 16 l.  Written as assembly because the compiler orders every later LDS read
// behind such a copy with a full vmcnt wait; the kernel's own waits and barriers (below) are what orders them.
// m0, the LDS address of such a load, is an operand: the compiler sets it and knows what it holds.  (s_nop: one wait state between the two.)
__device__ __forceinline__ void copy_to_lds(const void* base, unsigned off, unsigned lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "{m0}"(__builtin_amdgcn_readfirstlane(lds)), "v"(off), "s"(base) : "memory");
}
// All but the last N copies of this wavefront have landed and its LDS reads have come back; then a barrier.  (The LDS wait is a builtin so
// that the compiler knows about it and waits for no later read because of an earlier one.)
template <int N>
__device__ __forceinline__ void wait_copies_and_sync() {
    __builtin_amdgcn_s_waitcnt(0xc07f);                        // lgkmcnt(0)
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(N) : "memory");
}

}  // namespace ax
