// gfx950 loads from memory straight into LDS, and the wait that goes with them.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe {

namespace {

// M0 is on the clobber list so that the compiler never orders this statement between its own
// write of M0 and the instruction that consumes it.  M0 is a reserved (non-allocatable)
// register, for which clang prints a generic "may not be preserved" warning: overwriting it is
// exactly what is declared here, so the warning is silenced for this one statement.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16(const void* gptr, uint32_t lds_addr) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_addr);   // wave-uniform: goes through M0
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(base)
                 : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    // gfx9 encoding: vmcnt[3:0] -> bits 3:0, vmcnt[5:4] -> bits 15:14; expcnt (6:4) and lgkmcnt (11:8) = no wait
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// As lds_dma16, from a wave-uniform base plus a 32-bit lane offset; NT: non-temporal.
// The base is copied by a scalar instruction inside the statement: a vector-memory instruction may read a scalar
// register no sooner than five wait states after a vector instruction (v_readfirstlane, a spilled register's
// v_readlane) wrote it, and the compiler adds no wait states in front of inline assembly.  Scalar instructions wait for such
// a write by themselves.  The copy is also the wait state that M0 needs before the load.
template <bool NT>
__device__ __forceinline__ void lds_dma16_at(const void* base, uint32_t lane_off, uint32_t lds_addr) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_addr);
    uint64_t from;
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0 nt"
                     : "=&s"(from) : "v"(lane_off), "s"(u), "s"(dst) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                     : "=&s"(from) : "v"(lane_off), "s"(u), "s"(dst) : "memory", "m0");
}
#pragma clang diagnostic pop

}  // namespace

}  // namespace moe
