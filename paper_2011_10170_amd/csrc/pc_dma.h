// Direct loads from memory to LDS, shared by the convolution kernels that use them.
#ifndef PC_DMA_H
#define PC_DMA_H
#include "pc_mfma.h"

#define DM_OOB 0x80000000u           // past the end of any tensor taken here, also with a chunk's offset added

// 64 lanes x 16 bytes from a buffer to the 1 KiB of LDS at lds_off; an offset past the buffer's end writes zeros. As inline
// assembly because the compiler orders every later LDS read behind a direct load it knows of: here the wait is one
// s_waitcnt in front of a barrier. (The compiler warns that it saves no reserved register for the statement: m0 holds nothing
// of its own that it would have to.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dm_load(const v4u32 &rsrc, int voff, int soff, int lds_off)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop

// All but the last N vector memory operations of this wavefront are complete, and every wavefront has come here.
template <int N> __device__ __forceinline__ void dm_wait_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(N) : "memory");
}

// The words of a buffer resource (what __builtin_amdgcn_make_buffer_rsrc builds, as an operand of inline assembly).
__device__ __forceinline__ v4u32 dm_rsrc(const void *p, uint32_t bytes)
{
    const uint64_t a = (uint64_t)p;
    const v4u32 r = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu)),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
    return r;
}
#endif
