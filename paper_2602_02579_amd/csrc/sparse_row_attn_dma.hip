// Step 5, head_dim 128, bf16: the launch of the pipelined attention kernels
// (sparse_row_attn_w8.hip, sparse_row_attn_w8n.hip) and the merge of their key ranges.
#include <atomic>
#include <cstdlib>

#include "attn_common.h"

namespace pkv {

namespace {

constexpr int D = 128;

// Merge of the key ranges of a split launch: out = sum_s w_s O_s / sum_s w_s with
// w_s = exp(lse_s - max lse), over the ranges that begin at or below the row's limit.
// 32 lanes of four output elements per (row, head), eight of them per workgroup.  Rows whose
// keys all lie in the first range were written by that range's job.
constexpr int kMergeCols = 8;
static_assert(D == 128, "one (row, head) is 32 lanes of four floats");
__global__ __launch_bounds__(32 * kMergeCols) void attn_merge_splits_kernel(AttnParams p) {
    const int64_t col = (int64_t)blockIdx.x * kMergeCols + (threadIdx.x >> 5);   // row * hq + head
    if (col >= (int64_t)p.m * p.hq) return;
    const int row = (int)(col / p.hq), head = (int)(col % p.hq);
    const int limit = min(p.row_pos[row], p.n_keys - 1);
    const int n_s = limit / p.dma_split_len + 1;   // <= dma_splits
    if (n_s == 1) return;
    const int l = threadIdx.x & 31;
    // (unrolled by four so that the loads of four ranges are in flight together: with up to
    // 32 ranges per row the loop is otherwise a chain of memory latencies)
    const float* const lse_col = p.part_lse + (int64_t)row * p.hq + head;
    const float* const o_col = p.part_o + ((int64_t)row * p.hq + head) * D + 4 * l;
    const int64_t lse_step = (int64_t)p.m * p.hq, o_step = lse_step * D;
    float mx = -INFINITY;
#pragma unroll 4
    for (int sp = 0; sp < n_s; ++sp) mx = fmaxf(mx, lse_col[sp * lse_step]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float wsum = 0.f;
#pragma unroll 4
    for (int sp = 0; sp < n_s; ++sp) {
        const float w = __expf(lse_col[sp * lse_step] - mx);
        const f32x4 o = *reinterpret_cast<const f32x4*>(o_col + sp * o_step);
        wsum += w;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += w * o[e];
    }
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (bf16_t)(acc[e] / wsum);
    *reinterpret_cast<bf16x4*>(p.out + col * D + 4 * l) = v;
    if (p.lse && l == 0) p.lse[col] = mx + logf(wsum);
    if (p.lse_ctx && l == 0) {
        // the ranges that lie below ctx_keys (a range boundary): the same sum, cut there
        const int n_c = min(n_s, p.ctx_keys / p.dma_split_len);
        float mc = -INFINITY;
        for (int sp = 0; sp < n_c; ++sp)
            mc = fmaxf(mc, p.part_lse[((int64_t)sp * p.m + row) * p.hq + head]);
        float wc = 0.f;
        for (int sp = 0; sp < n_c; ++sp)
            wc += __expf(p.part_lse[((int64_t)sp * p.m + row) * p.hq + head] - mc);
        p.lse_ctx[col] = mc + logf(wc);
    }
}

}  // namespace

int attn_dma128_v_source() {
    // read at every call, so that one process can run both sources side by side
    const char* e = std::getenv("PKV_ATTN_VT");
    return !e ? -1 : (e[0] == '1' ? 1 : (e[0] == '0' ? 0 : -1));
}

int attn_cu_count() {
    static std::atomic<int> n_cu_cached{0};   // per process; the devices of one machine are alike
    int n_cu = n_cu_cached.load(std::memory_order_relaxed);
    if (n_cu == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            v <= 0)
            return 0;   // asked again at the next call
        n_cu = v;
        n_cu_cached.store(v, std::memory_order_relaxed);
    }
    return n_cu;
}

pkv_status launch_attn_dma128(const AttnParams& p, hipStream_t st) {
    if (!p.q || !p.k || !(p.v || p.vt) || !p.row_pos || !p.out) return PKV_ERR_NULL;
    if (p.dma_splits < 1 || p.dma_split_len < kBN || p.dma_split_len % kBN ||
        (int64_t)p.dma_splits * p.dma_split_len < p.n_keys)
        return PKV_ERR_SHAPE;
    if (p.dma_splits > 1 && (!p.part_o || !p.part_lse)) return PKV_ERR_WORKSPACE;
    const int n_cu = attn_cu_count();
    if (n_cu == 0) return PKV_ERR_LAUNCH;
    // without counters every workgroup is one job, and all of them have to be launched
    if (!p.queue && (int64_t)p.n_tiles * p.dma_splits * p.hkv > n_cu) return PKV_ERR_LAUNCH;
    // one job per workgroup, or a queue of them for one workgroup per CU: see the two kernels
    const pkv_status rc = p.queue ? launch_attn_w8n_main(p, n_cu, st) : launch_attn_w8_main(p, st);
    if (rc != PKV_OK) return rc;
    if (p.dma_splits > 1)
        hipLaunchKernelGGL(attn_merge_splits_kernel,
                           dim3((unsigned)(((int64_t)p.m * p.hq + kMergeCols - 1) / kMergeCols)),
                           dim3(32 * kMergeCols), 0, st, p);
    return launch_status();
}

}  // namespace pkv
