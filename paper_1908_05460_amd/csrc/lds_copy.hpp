// Loads that go from a buffer to LDS without passing through registers.
#pragma once
#include "common.hpp"

namespace wgrad {

typedef uint32_t br_u4 __attribute__((ext_vector_type(4)));

// 16 bytes a lane from the buffer to LDS at dst + 16 * lane, not waited for.  (The whole offset is the lanes': the range check
// subtracts a scalar one from the buffer's size, which wraps where it is the larger.  The five wait states are those between a
// lane read or the like that wrote the descriptor and a load that reads it: the compiler puts none into asm.)
// (m0 is named so that no value the compiler has put there is taken to be left; it remarks that the register is its own.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void rows_copy(br_u4 buf, uint32_t off, uint32_t dst)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(off), "s"(buf) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ br_u4 rows_buffer(const void *p, uint32_t bytes)
{
    const uint64_t a = (uint64_t)p;
    return br_u4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}

}  // namespace wgrad
