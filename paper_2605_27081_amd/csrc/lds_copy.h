// Direct global -> LDS copies and the waits that go with them, written as assembly.
#pragma once

#include "common.h"

namespace remoe {

// 64 lanes x 16 bytes, global -> LDS without passing through registers: lane l's 16 bytes, read from
// base + off (wave-uniform 64-bit base, per-lane byte offset), land at lds_base + 16 l
// (lds_base wave-uniform, handed over in M0).  Written as assembly so that the compiler keeps no
// books on these copies: its own bookkeeping makes every later LDS read wait for all of them,
// which would undo the overlap.  Every wait for such a copy is therefore explicit.
// The compiler pads its own instructions with the wait states the hardware asks for but does not
// look inside an assembly block, so the block must not depend on any:
//   * the address goes in as a per-lane 64-bit value in vector registers (the compiler's own add of
//     base and offset in front of the block).  With the base in a scalar register pair the copy
//     would read a scalar register as a memory address, and a scalar register that a vector
//     instruction has just written (a spilled base restored with v_readlane) may not be used that
//     way for five wait states: whether that happened would depend on register allocation;
//   * M0 is written inside the block and the one wait state the copy needs behind that write is
//     part of the block.  Nothing else in these kernels touches M0 (the compiler reserves it and has
//     no use for it there; a host-side test of the grouped GEMM's generated code checks that).
template <typename Offset> __device__ __forceinline__ void copy16_to_lds(const char *base, Offset off, const void *lds_base)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t dst = (uint32_t)(uintptr_t)lds_base;   // the low 32 bits of a generic LDS pointer are the LDS offset
    const char *src = base + off;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory");
#else
    (void)base;
    (void)off;
    (void)lds_base;
#endif
}

// Until at most N of this wavefront's vector memory operations are outstanding (they complete in order).
template <int N> __device__ __forceinline__ void wait_vmem()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}

// Workgroup barrier that orders LDS traffic only.  (__syncthreads would also wait for every copy in flight.)
__device__ __forceinline__ void lds_barrier()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

}  // namespace remoe
