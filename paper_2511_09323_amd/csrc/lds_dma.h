// Loads from memory to LDS that pass no registers, and the waits for them.
#pragma once
#include "common.h"

namespace moc {

// 16 bytes per lane from memory to LDS (lane l to lds + 16 l).  Has no register result; the caller counts it in vmcnt.  (As the
// builtin, the compiler would wait for all of them before every LDS read, which it cannot tell apart.)
// m0 is an operand, so that the compiler, which has uses of its own for it, knows what it holds.  It does not look for hazards inside: the
// wait state between a write of m0 and the load is here; the five that a load needs after a vector instruction wrote part of its descriptor
// (v_readlane of a spilled one, for instance) are not (s_nop 3 costs 0.3 to 1 % of a training step), and tests/test_lds_dma.py looks
// for such writes in the built kernels.
// NT: a stream that nobody reads again.
template <bool NT = false> __device__ __forceinline__ void lds_load16(uint32_t off, u32x4_t rsrc, uint32_t lds) {
    if constexpr (NT) asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"{m0}"(lds), "v"(off), "s"(rsrc) : "memory");
    else asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(lds), "v"(off), "s"(rsrc) : "memory");
}
__device__ __forceinline__ u32x4_t buffer_desc(const void* p, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return u32x4_t{(uint32_t)a, (uint32_t)(a >> 32) & 0xFFFFu, bytes, 0x00020000u};
}
// At most VM of this wavefront's vector memory instructions still under way (and no LDS reads, with LDS).
template <int VM, bool LDS> __device__ __forceinline__ void wait_counts() {
    static_assert(VM >= 0 && VM < 64, "");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | ((LDS ? 0 : 15) << 8) | ((VM >> 4) << 14));
    asm volatile("" ::: "memory");
}

}  // namespace moc
