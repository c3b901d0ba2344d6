// Loads from memory to LDS that bypass the registers, and the waits that count them.
#pragma once
#include "common.h"

namespace fate {

// 16 (4) bytes per lane from sbase + voff (vaddr) to lds + lane*16 (*4).  The loads are outside the
// compiler's sight: it must not wait for them (it would wait for all of them), the pipeline's
// own counted waits do.  m0 is named as overwritten, so that no value the compiler keeps there is taken
// to survive; it warns that the register is reserved, which is what makes the name right.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_load16(uint32_t lds, const void* sbase, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds), "v"(voff), "s"(sbase) : "memory", "m0");
}
__device__ __forceinline__ void lds_load4(uint32_t lds, const void* vaddr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :: "s"(lds), "v"(vaddr) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// Waits until at most `left` stages of LPS loads are outstanding (left <= MOST).
template <int LPS, int MOST>
__device__ __forceinline__ void wait_stages(int left) {
    if constexpr (MOST == 0) wait_loads<0>();
    else if (left >= MOST) wait_loads<MOST * LPS>();
    else wait_stages<LPS, MOST - 1>(left);
}
// Workgroup barrier that orders LDS traffic only: the stages in flight stay in flight.
__device__ __forceinline__ void lds_only_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

}  // namespace fate
