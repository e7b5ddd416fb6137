// Loads from memory straight to shared memory.  Written as assembly because the compiler makes every later read of shared memory wait
// for all such loads; whoever uses these counts the waits by hand.  Included by the kernel sources only.
#pragma once

#include <hip/hip_runtime.h>

namespace bmgd {
namespace {

// 16 bytes per lane from its own address to shared memory at lds + 16 * lane
__device__ __forceinline__ void load_to_lds(const unsigned short* src, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %1\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, off"
                 :: "v"(src), "s"(lds) : "memory", "m0");
}

// the same at device scope: never from the compute unit's own cache
__device__ __forceinline__ void load_to_lds_agent(const unsigned short* src, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %1\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, off sc1"
                 :: "v"(src), "s"(lds) : "memory", "m0");
}

// 4 bytes per lane to shared memory at lds + 4 * lane
__device__ __forceinline__ void load_word_to_lds(const int* src, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %1\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dword %0, off"
                 :: "v"(src), "s"(lds) : "memory", "m0");
}

}  // namespace
}  // namespace bmgd
