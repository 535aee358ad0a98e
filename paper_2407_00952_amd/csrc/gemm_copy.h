// Asynchronous global -> LDS copies of the bf16 GEMM kernels.
#pragma once
#include "common.h"

// 16 bytes per lane (the 64 lanes fill 1 KB) with a scalar 64-bit base and a 32-bit per-lane byte offset, which keeps
// the address down to one VGPR per row.  `lds` is the wave-uniform LDS byte address the 1 KB lands at.  Waiting for
// completion (vmcnt + barrier) is the caller's job.
__device__ __forceinline__ void glds_soff(const void *sbase, unsigned voff, unsigned lds)
{
    // M0 carries the LDS address; one wait state is required between its write and the copy.  The compiler
    // treats M0 as reserved and does not accept it on a clobber list, so nothing else in a file that uses this may
    // depend on M0: tests/test_kernel_isa.py checks in the compiled code that every write of M0 is the one
    // below and that nothing but these copies reads it.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds), "v"(voff), "s"(sbase)
                 : "memory");
}
// the same with all lanes (mask -1) or none (mask 0: moves nothing, and still counts); all 64 are enabled around it
__device__ __forceinline__ void glds_soff_if(const void *sbase, unsigned voff, unsigned lds, int mask)
{
    asm volatile("s_mov_b32 exec_lo, %3\n\ts_mov_b32 exec_hi, %3\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1"
                 :
                 : "s"(lds), "v"(voff), "s"(sbase), "s"(mask)
                 : "memory");
}
// 4 bytes per lane (256 bytes), by all lanes or none
__device__ __forceinline__ void glds4_soff_if(const void *sbase, unsigned voff, unsigned lds, int mask)
{
    asm volatile("s_mov_b32 exec_lo, %3\n\ts_mov_b32 exec_hi, %3\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2\n\ts_mov_b64 exec, -1"
                 :
                 : "s"(lds), "v"(voff), "s"(sbase), "s"(mask)
                 : "memory");
}
__device__ __forceinline__ unsigned lds_addr(const void *p)
{
    return (unsigned)(unsigned long long)(const __attribute__((address_space(3))) char *)p;
}
