// Shared device helpers for the SALS kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sals {

constexpr int kXcds = 8;       // accelerator dies, workgroups are dealt to them round-robin

// n / d for 0 <= n, d < 2^24: numbers of heads, sequences, slices, tiles and work items (a grid has fewer than 2^32 threads, 256 or
// more of them per workgroup).  A kernel's first loads wait for a chain of these, and 24 bits divide in 12 instructions (one float
// reciprocal and a correction), 32 signed ones in 26.
__device__ __forceinline__ int idiv(int n, int d) { return (int)(((unsigned)n & 0xffffffu) / ((unsigned)d & 0xffffffu)); }

// Workgroup `id` of N -> its item, one contiguous range of the list of N items per XCD.
__device__ __forceinline__ int xcd_item(int id, int N)
{
    const int xcd = (unsigned)id % kXcds, slot = (unsigned)id / kXcds, qn = (unsigned)N / kXcds, rem = (unsigned)N % kXcds;
    return xcd * qn + min(xcd, rem) + slot;
}

// Who is the last of a launch's workgroups?  One thread of each calls once, behind everything that must come before what the last one does:
// it is the one that gets n_wg - 1.  The count is zero between launches (the last arrival wraps it).  Nobody waits for anybody, and what
// an arrival costs is the round trip of its answer (1 us), which is asked for early and looked at late.
__device__ __forceinline__ uint32_t arrive(uint32_t* count, uint32_t n_wg) { return atomicInc(count, n_wg - 1); }

constexpr int kWave = 64;
constexpr int kHeadDim = 128;        // head width the kernels are written for
constexpr int kPairs = kHeadDim / 2; // RoPE pairs per head

typedef unsigned short bf16_t;       // raw bfloat16 bit pattern
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even (the hardware conversion, v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16_t f32_to_bf16(float f)
{
    return __builtin_bit_cast(bf16_t, (__bf16)f);
}

// low / high bf16 of a packed 32-bit word as fp32
__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

template <typename T> struct elem;
template <> struct elem<float> {
    static constexpr int vec = 4;  // elements per 16-byte chunk
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
    static __device__ __forceinline__ void unpack(const u32x4& c, float* f)
    {
        f[0] = __uint_as_float(c.x); f[1] = __uint_as_float(c.y);
        f[2] = __uint_as_float(c.z); f[3] = __uint_as_float(c.w);
    }
};
template <> struct elem<bf16_t> {
    static constexpr int vec = 8;
    static __device__ __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
    static __device__ __forceinline__ void unpack(const u32x4& c, float* f)
    {
        f[0] = bf16lo(c.x); f[1] = bf16hi(c.x); f[2] = bf16lo(c.y); f[3] = bf16hi(c.y);
        f[4] = bf16lo(c.z); f[5] = bf16hi(c.z); f[6] = bf16lo(c.w); f[7] = bf16hi(c.w);
    }
};

// A wave-uniform 32-bit value read through the vector memory path (the compiler would use a scalar load for a
// uniform address, and wait for it on its own before the wave's first vector load is issued): the request joins the
// wave's other loads; wave_uniform() hands the value to the scalar side where it is first needed.
__device__ __forceinline__ int ld_uniform_i32(const int32_t* p)
{
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));  // (opaque to the compiler: the address is no longer provably uniform)
    return p[zero];
}
__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// 16-byte global load
__device__ __forceinline__ u32x4 ld16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }
// the same for a long stream that is read once: the caches are told not to keep it (measured: 10-13 % faster for
// streams of 80 MB and more, slower for the few-MB weight streams and for gathered rows)
__device__ __forceinline__ u32x4 ld16_stream(const void* p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); }
__device__ __forceinline__ f32x4 ld16_f32_stream(const float* p) { return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p)); }

// Sum over each aligned group of 16 lanes (a DPP row); every lane gets the total.
__device__ __forceinline__ float row16_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false)); // row_ror:8
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false)); // row_ror:4
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false)); // row_ror:2
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false)); // row_ror:1
    return v;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Sum over each aligned group of 16 lanes, integer flavour.
__device__ __forceinline__ uint32_t row16_sum_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false); // row_ror:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false); // row_ror:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false); // row_ror:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false); // row_ror:1
    return v;
}

// inclusive prefix sum over the 64 lanes of a wave: shifts inside each 16-lane row, then the
// row totals are carried across rows by the two row broadcasts
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false); // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false); // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false); // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false); // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false); // row_bcast:15 -> rows 1,3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false); // row_bcast:31 -> rows 2,3
    return v;
}

// Wave-wide maximum / sum, every lane gets the result: DPP rotations inside each 16-lane row, then the
// four row results are combined through scalar registers.
__device__ __forceinline__ float row16_max(float v)
{
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false)));
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
    const int r = __float_as_int(row16_max(v));
    const float a = __int_as_float(__builtin_amdgcn_readlane(r, 0)), b = __int_as_float(__builtin_amdgcn_readlane(r, 16));
    const float c = __int_as_float(__builtin_amdgcn_readlane(r, 32)), d = __int_as_float(__builtin_amdgcn_readlane(r, 48));
    return fmaxf(fmaxf(a, b), fmaxf(c, d));
}
__device__ __forceinline__ float wave_sum(float v)
{
    const int r = __float_as_int(row16_sum(v));
    const float a = __int_as_float(__builtin_amdgcn_readlane(r, 0)), b = __int_as_float(__builtin_amdgcn_readlane(r, 16));
    const float c = __int_as_float(__builtin_amdgcn_readlane(r, 32)), d = __int_as_float(__builtin_amdgcn_readlane(r, 48));
    return (a + b) + (c + d);
}

// Wave-wide minimum / maximum / sum of unsigned integers, every lane gets the result (same scheme as above).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return min(min(a, b), min(c, d));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
    v = row16_sum_u32(v);
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return (a + b) + (c + d);
}

// order-preserving map fp32 -> uint32 (larger float <=> larger key); -0 counts as +0
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t u = __float_as_uint(s + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

}  // namespace sals
