// Direct loads into LDS, and the waits and scheduling that go with them.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pdelta {

// All of these set m0, and say so: the compiler never allocates m0, but it orders its own uses of it by what is
// declared (and warns that it will not save a reserved register, which is not asked of it).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane from base + off (per lane) to LDS address lds + 16 * lane.  As an asm statement so
// that the compiler does not wait for it before every LDS read; the kernel waits itself.
__device__ __forceinline__ void load_lds_16(uint32_t lds, uint32_t off, const void* base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
}
// 16 bytes per lane from its own address.
__device__ __forceinline__ void load_lds_16v(uint32_t lds, const void* p)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(p) : "m0", "memory");
}
// 4 bytes per lane to LDS address lds + 4 * lane.
__device__ __forceinline__ void load_lds_4(uint32_t lds, uint32_t off, const void* base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
}
// 2 bytes, zero-extended, per lane to LDS address lds + 4 * lane.
__device__ __forceinline__ void load_lds_2(uint32_t lds, uint32_t off, const void* base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ushort %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop
// Scheduling: V vector instructions after each of N MFMAs.
template <int N, int V>
__device__ __forceinline__ void interleave()
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
    }
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace pdelta
