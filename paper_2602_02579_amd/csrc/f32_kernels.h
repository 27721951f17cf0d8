// Declarations of the fp32 matrix-core kernels (f32_kernels.hip).
#pragma once

#include "pkv_common.h"

namespace pkv {

enum F32Mode { kF32Rope = 0, kF32Plain = 1, kF32Gated = 2 };

struct F32GemmParams {
    const float* x;            // [rows, k]
    const int32_t* row_idx;    // [m] or null
    const float* w[3];         // wq, wk, wv; or w; or w_gate, w_up
    float* out[3];             // q, k, v; or y
    int m, k;
    int n_out;                 // plain and gated
    const float* residual;     // plain: [m, n_out] or null
    // projection: tiles of 16 rotary pairs, first tile of Q, K, V, end
    int tile_begin[4];
    int hq, hkv, d;
    const int32_t* row_pos;    // [m]
    const int32_t* dst_row;    // [m] or null: rows of K and V
    const float* bias[3];      // or null
    // gains [k] of an RMS norm of the rows of x before the product, where norm_f32_pays, or null
    const float* norm_w;
    float norm_eps;
};
// projection and gated: the rows normalised inside the launch cost less than by one of their own
bool norm_f32_pays(int mode, const F32GemmParams& p);
pkv_status launch_gemm_f32(int mode, const F32GemmParams& p, const RopeTable& tab,
                           hipStream_t st);
// pointers of a linear layer allow 16-byte accesses (null counts as aligned), rows fit the grid
bool linear_f32_supported(const void* x, const void* w0, const void* w1, const void* residual,
                          const void* y, int64_t m);
// whether it beats a wave per output element
bool linear_f32_pays(bool gated, int64_t m, int64_t k_in, int64_t n_out);

// fp32 with head_dim 32, 64 or 128: score and attention below
bool f32_tiles_supported(const pkv_layer_cfg& cfg);
pkv_status launch_attn_f32(const pkv_layer_cfg& cfg, const float* q, const float* k,
                           const float* v, const int32_t* row_pos, float* out, float* lse,
                           int64_t m, int64_t n_keys, float scale, hipStream_t st,
                           int64_t chunk_len = 0);   // > 0: rows and keys are runs of that
                                                     // length, each attending within itself

struct F32ScorePlan {
    int n_splits, split_len;
};
F32ScorePlan plan_score_f32(const pkv_layer_cfg& cfg, int64_t n_ctx, int64_t nq);
// a float per column, or with several splits two per split and column
size_t score_f32_ws_bytes(const pkv_layer_cfg& cfg, int64_t n_ctx, int64_t nq);
// lse null: both passes, ws holds score_f32_ws_bytes; else pass 2 with these normalisers
pkv_status launch_score_f32(const pkv_layer_cfg& cfg, const float* q, const float* k,
                            const float* lse, const int32_t* row_pos, float* score, int64_t nq,
                            int64_t n_ctx, float scale, int accumulate, void* ws,
                            hipStream_t st);

}  // namespace pkv
