// What the tile kernels of the projection and the linear layers share (gfx950, bf16).
#pragma once

#include "proj_common.h"

namespace pkv {

constexpr int kEpiStride = 272;                  // bytes per token of the store staging

// 16 bytes per lane from global memory straight into LDS: lane i of the wave
// writes LDS bytes [lds_base + 16 i, +16); lds_base must be wave-uniform.
__device__ __forceinline__ void dma16(const void* gptr, uint32_t lds_base) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off"
        :
        : "s"(lds_base), "v"(gptr)
        : "memory", "m0");
}
// c += a . b on a 16 x 16 tile, 32 of the contraction.  Written out so that the accumulator
// stays where it is: left to itself the register allocator rotates the 64 accumulators of a
// wave through copies (584 of them per two steps) once they are four registers each.  The
// compiler does not see the result's latency: acc_settle(), then acc_take() before a read.  (What it
// adds by itself, such as copies at the end of a loop, can still come before that:
// test_matrix_result_waits.py looks for it in the built code.)
__device__ __forceinline__ void mfma_16x16x32(f32x4& c, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// the wait behind the last product, which nothing is moved across
__device__ __forceinline__ void acc_settle() {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// an accumulator on its way to its readers: they depend on this statement, and this one comes
// behind the wait
__device__ __forceinline__ void acc_take(f32x4& c) { asm volatile("" : "+v"(c)); }
template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// silu(a) = a / (1 + e^-a) with the hardware reciprocal (1 ulp): the result is rounded to
// bf16 right away, and a full-precision division would cost ten instructions per element
__device__ __forceinline__ float silu_f32(float a) {
    return a * __builtin_amdgcn_rcpf(1.f + __expf(-a));
}

// gather_qkv_proj_tiles.hip: the launch of p with p.n_ksplit splits of the contraction
// (hid % (64 n_ksplit) == 0) on tiles of 128 features x 64 or 128 tokens
template <int MODE, bool EXTRA>
pkv_status launch_proj_small(int tokens, const ProjParams& p, hipStream_t st);

}  // namespace pkv
