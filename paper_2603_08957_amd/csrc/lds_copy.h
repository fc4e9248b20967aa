// Copies from global memory straight into LDS (global_load_lds: lane l's bytes
// land at the LDS address + 4 or 16 l) and their waits.  The copies are issued
// from inline assembly, which the compiler's own wait insertion does not see:
// a kernel waits for them explicitly (they complete in order) and drains them
// before its LDS is used otherwise.  The waits, not the copies, are the
// compiler's memory barriers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tre {

typedef __attribute__((address_space(3))) char lds_char;

__device__ inline uint32_t lds_address(const void* p) {
    return uint32_t(reinterpret_cast<uintptr_t>((lds_char*)(const_cast<void*>(p))));
}

__device__ inline uint64_t uniform64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(x));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(x >> 32));
    return (uint64_t(hi) << 32) | lo;
}

// 16 bytes per lane from base + voff (base uniform, voff the lane's) to
// lds_addr + 16 lane; NT: read once, not kept in L2.
template <bool NT>
__device__ inline void lds_copy16(uint32_t lds_addr, const void* base, uint32_t voff) {
    const uint32_t m = __builtin_amdgcn_readfirstlane(lds_addr);
    const uint64_t b = uniform64(reinterpret_cast<uint64_t>(base));
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(m), "v"(voff), "s"(b) : "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m), "v"(voff), "s"(b) : "m0");
}

// 4 bytes per lane
__device__ inline void lds_copy4(uint32_t lds_addr, const void* base, uint32_t voff) {
    const uint32_t m = __builtin_amdgcn_readfirstlane(lds_addr);
    const uint64_t b = uniform64(reinterpret_cast<uint64_t>(base));
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" ::"s"(m), "v"(voff), "s"(b) : "m0");
}

// until at most N of this wavefront's copies (and loads) are in flight
template <int N>
__device__ inline void lds_copy_wait() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit count");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// until this wavefront's LDS reads have returned (a copy may then overwrite
// what they read)
__device__ inline void lds_read_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

}  // namespace tre
