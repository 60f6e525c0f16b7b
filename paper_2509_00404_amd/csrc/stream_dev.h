// Pieces shared by the GEMM kernels whose operands stream into LDS without passing through registers.
#pragma once
#include "common.h"
#include <utility>

namespace {

// Transfers global memory -> LDS that pass through no register: the lane's 16 bytes go to lds + AT + 16 lane.  lds and base
// are uniform.  Two hazards that the compiler does not look for inside asm are closed here: m0 must have been written two
// instructions before, and a base that a vector instruction wrote (v_readfirstlane, or v_readlane where it was spilled) may be read by
// a memory instruction only five wait states later.  The scalar copy waits for either writer by itself, and stands where m0 needs an
// instruction in between.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"          // m0 is one of the compiler's reserved registers, and is to be clobbered
template <int AT>
__device__ __forceinline__ void gs_dma16(uint32_t lds, uint32_t voff, const uint8_t* base) {
    const uint8_t* copy;
    asm volatile("s_add_u32 m0, %1, %4\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0"
                 : "=&s"(copy) : "s"(lds), "v"(voff), "s"(base), "n"(AT) : "memory", "m0", "scc");
}
// the lane's 4 bytes to lds + AT + 4 lane
template <int AT>
__device__ __forceinline__ void gs_dma4(uint32_t lds, uint32_t voff, const uint8_t* base) {
    const uint8_t* copy;
    asm volatile("s_add_u32 m0, %1, %4\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dword %2, %0"
                 : "=&s"(copy) : "s"(lds), "v"(voff), "s"(base), "n"(AT) : "memory", "m0", "scc");
}
#pragma clang diagnostic pop
// all but the N youngest of the wave's transfers have arrived and its LDS reads are done; then the workgroup meets
template <int N>
__device__ __forceinline__ void gs_meet() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}
// The lane's number, computed where it is used: what is derived from it is then not kept in registers over the whole kernel.
__device__ __forceinline__ int gs_fresh_lane() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

#define GS_INLINE __attribute__((always_inline))
// f(0), f(1), ... f(N - 1) with constants (a loop of this size with the bodies below is not unrolled by pragma)
template <int... I, typename F>
__device__ __forceinline__ void gs_each(std::integer_sequence<int, I...>, const F& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void gs_for(const F& f) { gs_each(std::make_integer_sequence<int, N>{}, f); }

// a uniform pointer that stays in scalar registers
__device__ __forceinline__ const uint8_t* gs_uniform(const uint8_t* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const uint8_t*)((uint64_t)hi << 32 | lo);
}
// Lanes exchange what they staged: the compiler may order one lane's read and write of different addresses as it likes, and LDS keeps
// the wave's order.  (No instruction.)
__device__ __forceinline__ void gs_wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace
