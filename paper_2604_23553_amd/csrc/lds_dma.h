// Memory-to-LDS loads (no registers in between) and the buffer resources they take.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

namespace cfpp {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// 64 lanes x 16 bytes from memory straight into LDS: lane l's piece lands at lds_addr + 16 l.
// (Counted in vmcnt like any load; the callers wait by count.
// The scalar offset need not take part in the resource's range check: the callers keep every address inside.)
// (Winline-asm: M0 is reserved, nothing of the compiler's is kept in it; the clobber orders its own settings of it.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16(i32x4 rsrc, unsigned lds_addr, unsigned voff, unsigned soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
// The same for lines that are read once (non-temporal): whole 128-byte lines only.
__device__ __forceinline__ void lds_dma16_once(i32x4 rsrc, unsigned lds_addr, unsigned voff, unsigned soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 :: "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ i32x4 dma_rsrc(const void *p, unsigned bytes)
{
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    return i32x4{(int)(unsigned)a, (int)((unsigned)(a >> 32) & 0xffffu), (int)bytes, 0x00020000};
}
// LDS address of a pointer into the workgroup's memory
__device__ __forceinline__ unsigned lds_address(const char *p)
{
    return (unsigned)(size_t)(__attribute__((address_space(3))) const char *)p;
}

}  // namespace cfpp
