// Copies from global memory straight to LDS (buffer_load ... lds), 16 bytes per lane and no registers.
// Device code.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace sparsert {

typedef int32_t int4v __attribute__((ext_vector_type(4)));

// At most N of this wave's loads, stores and copies are still on their way.
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// 16 bytes per lane from descriptor + voffset + soffset + OFFSET straight to LDS at lds_base + OFFSET + 16 * lane.
// Written as assembly because the compiler would otherwise wait for every copy before any read of LDS.
template <int OFFSET> __device__ __forceinline__ void copy_to_lds(const int4v &rsrc, int voffset, int soffset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen offset:%4 lds"
                 ::"s"(lds_base), "v"(voffset), "s"(rsrc), "s"(soffset), "n"(OFFSET) : "memory");
}

// The same with 4 bytes per lane, 256 bytes in all.
__device__ __forceinline__ void touch_to_lds(const int4v &rsrc, int voffset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds_base), "v"(voffset), "s"(rsrc) : "memory");
}

__device__ __forceinline__ int4v descriptor(const void *p, int bytes) {
    const uint64_t u = (uint64_t)p;
    return int4v{(int)(uint32_t)u, (int)((uint32_t)(u >> 32) & 0xffffu), bytes, 0x00020000};
}

}  // namespace sparsert
