// Direct global->LDS loads and the wait for them, for the kernels that run their own pipelines.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace veda {

// 16 bytes per lane straight from global memory into LDS: lane i of the wave lands at LDS byte
// lds_base + 16*i (lds_base wave-uniform), from global address base + voff (base uniform).
// Written as inline assembly so that the compiler does not serialise later LDS reads of OTHER
// buffers behind these loads; completion is awaited explicitly (vmcnt) before the barrier that
// publishes the buffer.  M0 carries the LDS base (declared clobbered).
__device__ __forceinline__ void dma16_to_lds(uint32_t lds_base, const void* base, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_base), "v"(voff), "s"(base)
                 : "memory", "m0");
}

// N (1, 2 or 4) such loads with one M0 set-up: load j lands at lds_base + 1024*j + 16*lane and
// reads base + voff[j] + 1024*j -- the instruction's immediate offset moves the LDS address and
// the global address alike (measured on gfx950), so voff[j] is passed with 1024*j already taken off.
template <int N>
__device__ __forceinline__ void dma16_group_to_lds(uint32_t lds_base, const void* base, const uint32_t (&voff)[N]) {
    static_assert(N == 1 || N == 2 || N == 4, "1024*j must fit the 13-bit immediate offset");
    if constexpr (N == 4) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %5\n\t"
                     "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
                     "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
                     "global_load_lds_dwordx4 %4, %5 offset:3072"
                     :
                     : "s"(lds_base), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(base)
                     : "memory", "m0");
    } else if constexpr (N == 2) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %3\n\t"
                     "global_load_lds_dwordx4 %2, %3 offset:1024"
                     :
                     : "s"(lds_base), "v"(voff[0]), "v"(voff[1]), "s"(base)
                     : "memory", "m0");
    } else {
        dma16_to_lds(lds_base, base, voff[0]);
    }
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding).
template <int N> __device__ __forceinline__ void wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

}  // namespace veda
