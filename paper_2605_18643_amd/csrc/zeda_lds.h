// LDS reads and writes in inline asm, for kernels that keep global->LDS loads in flight.
#pragma once
#include "zeda_internal.h"

namespace zeda {

// LDS accesses the compiler does not see as such.  It orders every LDS access it knows about behind all
// global->LDS loads in flight (s_waitcnt vmcnt(0)), which would drain the ring at every table lookup and
// output transposition; these go around it and wait on lgkmcnt themselves.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)p; }  // low half of a flat LDS address
__device__ __forceinline__ uint32_t lds_read_b32(uint32_t a)
{
    uint32_t v;
    asm volatile("ds_read_b32 %0, %1" : "=v"(v) : "v"(a) : "memory");
    return v;
}
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t a)
{
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(a) : "memory");
    return v;
}
template <int OFF>
__device__ __forceinline__ u32x4 lds_read_b128_at(uint32_t a)  // a + OFF, the constant in the instruction's offset field
{
    static_assert(OFF >= 0 && OFF < 65536, "16-bit offset field");
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF) : "memory");
    return v;
}
__device__ __forceinline__ void lds_write_b64(uint32_t a, u32x2 v)
{
    asm volatile("ds_write_b64 %0, %1" ::"v"(a), "v"(v) : "memory");
}
// results of the reads above may be used after this
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void lds_wait(uint32_t &a) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a)::"memory"); }
__device__ __forceinline__ void lds_wait(u32x4 &a) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a)::"memory"); }
__device__ __forceinline__ void lds_wait(u32x4 &a, u32x4 &b) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a), "+v"(b)::"memory"); }

}  // namespace zeda
