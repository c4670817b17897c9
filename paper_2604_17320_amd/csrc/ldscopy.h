// Asynchronous copies from global memory to LDS, shared by the GEMM kernels.
#pragma once
#include "common.h"

// 16 (4) bytes per lane from global memory to LDS, lane l at lds + 16 l (4 l), without passing registers.
// In assembly because the compiler, which cannot tell the LDS buffers apart, would make every LDS read
// wait for the copies just started; the kernel waits for them itself (drain) before the barrier that
// hands the buffer over.  The LDS base goes into m0 as an operand, so that the compiler knows m0 taken; the
// chip wants one wait state between that write and the copy.  Both sides lie at multiples of what a lane copies: what a
// caller hands in is checked with on_lds_copies.
inline bool on_lds_copies(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
__device__ __forceinline__ void copy16_to_lds(const void *base, unsigned off, unsigned lds)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(lds), "v"(off), "s"(base) : "memory");
}
__device__ __forceinline__ void copy4_to_lds(const void *base, unsigned off, unsigned lds)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %1, %2" ::"{m0}"(lds), "v"(off), "s"(base) : "memory");
}
// All of this wave's loads and copies have arrived.  In assembly, because the compiler drops a wait that
// it thinks has nothing to wait for; the builtin as well, so that it knows its own loads have arrived.
__device__ __forceinline__ void drain()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);
}

// The address of a __shared__ object as the copies take it.
__device__ __forceinline__ unsigned lds_address(const void *p)
{
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
