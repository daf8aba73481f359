// Building blocks of the 256 x 256 matrix-core tiles: asynchronous global -> LDS loads and transposing LDS reads.
#pragma once
#include "common.hpp"
#include "k_attend.hpp"

namespace sals {

// 16 bytes per lane from `src` straight into LDS at `lds_base` + 16 * lane (lds_base: byte offset of the wave's piece, wave
// uniform).  Inline assembly, so that the compiler does not order later LDS reads behind it: the caller counts the
// outstanding loads (vm_wait) and separates writers from readers with a barrier.
__device__ __forceinline__ void load_lds16(const void* src, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(src) : "memory");
}
// the same from a wave-uniform base and a 32-bit offset per lane
__device__ __forceinline__ void load_lds16(const void* base, uint32_t offset, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(offset), "s"(base) : "memory");
}
template <int N> __device__ __forceinline__ void vm_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wg_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
typedef __attribute__((address_space(3))) unsigned char lds_byte;
__device__ __forceinline__ uint32_t lds_offset(const void* p) { return (uint32_t)(uintptr_t)(const lds_byte*)p; }

typedef short s16x4 __attribute__((ext_vector_type(4)));
// Transposing LDS read (ds_read_b64_tr_b16): the 16 lanes of a row group hand in the 8-byte pieces of four rows of 16
// elements (lanes 4t .. 4t+3: row t) and lane i receives column i, rows 0 .. 3.
__device__ __forceinline__ s16x4 lds_read_tr(const unsigned char* p)
{
    typedef __attribute__((address_space(3))) s16x4 lv;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lv*)(lds_byte*)p);
}

}  // namespace sals
