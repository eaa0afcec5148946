// Direct-to-LDS loads and the wait that goes with them.
#pragma once
#include <stdint.h>

#include <type_traits>

namespace reqat {

// Lane i's 16 (4) bytes at base + voff land at LDS address l + 16 i (4 i).  Inline
// asm, so that the compiler does not wait for all of them before every LDS read; the
// kernels order them themselves.  The compiler does not see a memory instruction
// here and leaves out its wait states: the one that m0 needs is written out, and
// base has to come from scalar instructions (a readfirstlane next to the load
// would be read too early; a base in vector registers does not compile).
__device__ __forceinline__ void g2l16(const uint8_t *base, uint32_t voff, uint8_t *l) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "{m0}"((uint32_t)(uintptr_t)l));
}
__device__ __forceinline__ void g2l4(const uint8_t *base, uint32_t voff, uint8_t *l) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(voff), "s"(base), "{m0}"((uint32_t)(uintptr_t)l));
}

// All but the wave's N newest loads have landed and its LDS reads are done; then
// the workgroup's barrier.  The LDS wait is the builtin, so that the compiler
// knows it: it would otherwise wait for the reads of the next stage before the
// first MFMA on operands that were read long ago.
template <int N> __device__ __forceinline__ void wait_and_meet() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);                     // lgkmcnt(0), the other counters at their maximum
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Calls f(integral_constant<int, J>) for J = B .. E-1, unrolled at compile time.
template <int B, int E, typename F> __device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

}  // namespace reqat
