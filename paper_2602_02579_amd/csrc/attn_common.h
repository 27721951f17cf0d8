// Declarations shared by the MFMA attention kernels (gfx950, bf16).
#pragma once

#include "pkv_common.h"

namespace pkv {

constexpr int kBN = 64;           // keys per LDS tile
constexpr int kAttnThreads = 256; // 4 waves per workgroup

struct AttnParams {
    const bf16_t* q;
    const bf16_t* k;
    const bf16_t* vt;        // [hkv, D, n_pad], zero beyond n_keys
    const bf16_t* v;         // [n_keys, hkv, D] as the cache holds it, or nullptr: when set, the
                             // pipelined kernel reads it, and vt is not used
    const int32_t* row_pos;  // [m] or nullptr when fixed_limit >= 0
    bf16_t* out;             // [m, hq, D]
    float* lse;              // [m, hq] or nullptr
    float* part_ml;          // [n_splits, m*hq, 2] (max in raw logits, sum) or nullptr
    const int* order;        // [n_tiles * dma_splits] or null: a kv head's jobs, the heaviest first
    int* queue;              // [hkv] next unclaimed row tile per kv head, zero before the
                             // launch, or nullptr: one job per workgroup (pipelined kernel)
    int dealt;               // workgroups whose first job goes by their number: all (the grid) or 0
    float* part_o;           // [dma_splits, m, hq, D] normalised partial outputs, and
    float* part_lse;         // [dma_splits, m, hq] their log-sum-exp (pipelined kernel with
                             // dma_splits > 1 only)
    float* lse_ctx;          // [m, hq] or nullptr: log-sum-exp over the keys below ctx_keys
    int ctx_keys;            // a multiple of dma_split_len (and of 64) when lse_ctx is set
    int dma_splits, dma_split_len;   // key ranges per row tile in the pipelined kernel
    int m, n_keys, n_pad, hq, hkv, group, bm, n_tiles, n_splits, split_len;
    int fixed_limit;         // >= 0: every row sees keys 0..fixed_limit
    int n_chunks, chunk_len; // sparse_row_attn_short.hip, n_chunks > 1: the m rows and the m keys
                             // are runs of chunk_len, each attending within itself
    float scale_log2;        // softmax scale * log2(e)
    float scale;
};

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// head_dim 128 attention proper: the software-pipelined kernels (sparse_row_attn_w8.hip,
// sparse_row_attn_w8n.hip), K / V tiles brought into LDS by direct global->LDS loads, and the
// merge of their key ranges (sparse_row_attn_dma.hip)
pkv_status launch_attn_dma128(const AttnParams& p, hipStream_t st);
pkv_status launch_attn_w8_main(const AttnParams& p, hipStream_t st);
pkv_status launch_attn_w8n_main(AttnParams p, int n_cu, hipStream_t st);
// sparse_row_attn_short.hip: up to 1024 keys, at most one job of 128 columns per CU; n_splits is
// what the pipelined kernel would cut the keys into
bool attn_short_applies(const pkv_layer_cfg& cfg, int64_t n_keys, int64_t m, int n_splits);
pkv_status launch_attn_short(AttnParams p, hipStream_t st);
// most keys of a chunk that the same kernel takes when many chunks share a launch
constexpr int kShortChunk = 1024;
// sparse_row_attn_pair.hip: jobs of 128 columns whose two groups of waves share the keys
bool attn_pair_applies(const pkv_layer_cfg& cfg, int64_t n_keys, int64_t m);
pkv_status launch_attn_pair(AttnParams p, hipStream_t st);
// compute units of the current device (0: could not be asked)
int attn_cu_count();
constexpr int kPlanCus = 256;   // and those that the plans reckon with
// Where the pipelined kernel can take the values from: 1 = from a V^T copy made by a pre-pass
// (PKV_ATTN_VT=1 in the environment), 0 = from the cache as it is (PKV_ATTN_VT=0), -1 = either,
// the caller chooses by size.  Read at every call; for comparisons and tests.
int attn_dma128_v_source();

}  // namespace pkv
