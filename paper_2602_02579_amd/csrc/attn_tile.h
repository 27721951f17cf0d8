// What the pipelined bf16 kernels for head_dim 128 are written in: fills of LDS straight from global
// memory and the wait for them, accumulators that stay in their registers, the transposing LDS
// read.  (sparse_row_attn_w8.hip, _w8n, _pair and _short, query_score_dma.hip)
#pragma once

#include "pkv_common.h"

namespace pkv {

// 16 bytes per lane from global memory straight into LDS: lane i of the wave
// writes LDS bytes [lds_base + 16 i, +16); lds_base must be wave-uniform.
__device__ __forceinline__ void dma16(const void* gbase, uint32_t voffset, uint32_t lds_base) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2"
        :
        : "s"(lds_base), "v"(voffset), "s"(gbase)
        : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// accumulators pinned to their registers (never touched by the VALU inside the loop)
__device__ __forceinline__ void mfma32_acc(bf16x8 a, bf16x8 b, f32x16& c) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

// Four 16-bit elements per lane through the transposing LDS read: within each group of 16
// lanes, lane i receives as element e the element i % 4 of what lane 4 e + i / 4 addressed.
// With lane 4 e + j addressing V[key + e][d0 + 4 j .. d0 + 4 j + 3] of a tile stored key-major,
// lane i ends up with V[key .. key + 3][d0 + i]: an A-operand fragment of V^T.
__device__ __forceinline__ bf16x4 lds_read_tr(const unsigned char* ptr) {
    typedef short i16x4 __attribute__((ext_vector_type(4)));
    const i16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)ptr);
    return __builtin_bit_cast(bf16x4, v);
}

}  // namespace pkv
