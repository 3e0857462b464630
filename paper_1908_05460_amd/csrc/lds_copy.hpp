// Loads that go from a buffer to LDS without passing through registers.
#pragma once
#include "common.hpp"

namespace wgrad {

typedef uint32_t br_u4 __attribute__((ext_vector_type(4)));

// 16 bytes a lane from the buffer to LDS at dst + 16 * lane, not waited for.  (The whole offset is the lanes': the range check
// subtracts a scalar one from the buffer's size, which wraps where it is the larger.)
__device__ __forceinline__ void rows_copy(br_u4 buf, uint32_t off, uint32_t dst)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(off), "s"(buf) : "memory");
}
__device__ __forceinline__ br_u4 rows_buffer(const void *p, uint32_t bytes)
{
    const uint64_t a = (uint64_t)p;
    return br_u4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}

}  // namespace wgrad
