// Step 1: rotary position restore on the assembled, position-free keys.
// (Paper: Sec. 1 footnote on position-independent key caches; Appendix E:
// positions go onto the old key cache once, before cache replacement.)
//
// HBM-bound streaming kernel.  One work item owns, for one token, a 16-byte
// run of pair indices i (8 bf16 or 4 fp32) and walks over all kv heads, so
// the sin/cos of a (token, i) pair is computed once and reused by every
// head.  Consecutive lanes own consecutive 16-byte runs, so a wave reads
// whole 128-byte (bf16, D=128) half-head segments of consecutive tokens.
#include "pkv_common.h"

#include <algorithm>
#include <cmath>

namespace pkv {

constexpr int kRopeLayers = 8;    // caches of a launch (its arguments grow with them)
constexpr int kRopeFull = 256;    // workgroups that a launch is brought to, see below

void fill_rope_table(RopeTable* t, int head_dim, double theta) {
    const int half = head_dim / 2;
    for (int i = 0; i < kMaxHalfDim; ++i)
        t->inv_freq[i] = i < half ? std::pow(theta, -2.0 * i / head_dim) : 0.0;
}

// The caches of several layers share a launch (blockIdx.y): one chunk of 512 tokens is 16 workgroups
// and as long as their chain of loads, sines and stores.  Where even that leaves the chip idle the
// heads of a token are dealt out too (blockIdx.z, heads_each of them): 512 tokens of 8 heads 4.7 ->
// 3.8 us, 4001 5.9 -> 5.3; past one workgroup per CU the sines made again cost more than the shorter
// chain gives (8192 tokens on 256, 512 and 1024 workgroups: 7.3, 7.5 and 7.8).  Launches of a
// single cache, and those that do not deal heads out, have neither in them: the pointers by the
// layer's number and the heads between two variables cost 1 to 4 % (34.5k tokens of 8 heads 25.5 and
// 25.1, 55k of 4 heads of 64 12.4 and 12.0).
template <int L>
struct RopeCaches {
    const void* in[L];
    void* out[L];
};

template <typename T, int L, bool DEAL>
__global__ __launch_bounds__(256) void rope_restore_kernel(
    RopeCaches<L> caches, const int32_t* __restrict__ pos, int64_t pos_base, int64_t n, int n_heads,
    int head_dim, RopeTable tab, int heads_each) {
    const int layer = L == 1 ? 0 : blockIdx.y;
    const T* const k_in = static_cast<const T*>(caches.in[layer]);
    T* const k_out = static_cast<T*>(caches.out[layer]);
    const int head0 = DEAL ? blockIdx.z * heads_each : 0;
    const int head_end = DEAL ? min(n_heads, head0 + heads_each) : n_heads;
    constexpr int V = Vec16<T>::N;
    typedef typename Vec16<T>::type vec_t;
    const int half = head_dim / 2;
    const int chunks = half / V;  // work items per token
    const int64_t total = n * chunks;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < total;
         w += stride) {
        const int64_t t = w / chunks;
        const int i0 = (int)(w - t * chunks) * V;
        const double p = pos ? (double)pos[t] : (double)(pos_base + t);
        const T* src = k_in + t * (int64_t)n_heads * head_dim + i0;
        T* dst = k_out + t * (int64_t)n_heads * head_dim + i0;
        // heads in batches of HB: all loads of a batch are issued before its
        // stores, which keeps many 16-byte requests in flight per lane without
        // assuming that k_in and k_out do not alias (in place is allowed); the
        // first batch is requested before the sines and cosines are worked out,
        // so that arithmetic runs under the memory latency
        constexpr int HB = 8;
        vec_t a[HB], b[HB];
        auto load_batch = [&](int h0) {
#pragma unroll
            for (int u = 0; u < HB; ++u) {
                if (h0 + u < head_end) {
                    // streamed once: non-temporal, so that the lines do not displace what the
                    // caches hold for the kernels around this one
                    a[u] = __builtin_nontemporal_load(
                        reinterpret_cast<const vec_t*>(src + (h0 + u) * head_dim));
                    b[u] = __builtin_nontemporal_load(
                        reinterpret_cast<const vec_t*>(src + (h0 + u) * head_dim + half));
                }
            }
        };
        load_batch(head0);
        float sn[V], cs[V];
#pragma unroll
        for (int j = 0; j < V; ++j) rope_sincos(p, tab.inv_freq[i0 + j], &sn[j], &cs[j]);
        for (int h0 = head0; h0 < head_end; h0 += HB) {
            if (h0 > head0) load_batch(h0);
#pragma unroll
            for (int u = 0; u < HB; ++u) {
                if (h0 + u < head_end) {
                    vec_t ra, rb;
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        const float x = Elem<T>::to_f32(a[u][j]);
                        const float y = Elem<T>::to_f32(b[u][j]);
                        ra[j] = Elem<T>::from_f32(x * cs[j] - y * sn[j]);
                        rb[j] = Elem<T>::from_f32(y * cs[j] + x * sn[j]);
                    }
                    __builtin_nontemporal_store(ra, reinterpret_cast<vec_t*>(dst + (h0 + u) * head_dim));
                    __builtin_nontemporal_store(
                        rb, reinterpret_cast<vec_t*>(dst + (h0 + u) * head_dim + half));
                }
            }
        }
    }
}

template <typename T, int L, bool DEAL>
static void rope_restore_launch(dim3 grid, const void* const* k_in, void* const* k_out,
                                const int32_t* pos, int64_t pos_base, int64_t n,
                                const pkv_layer_cfg& cfg, int heads_each, const RopeTable& tab,
                                hipStream_t st) {
    RopeCaches<L> caches = {};
    for (unsigned l = 0; l < grid.y; ++l) {
        caches.in[l] = k_in[l];
        caches.out[l] = k_out[l];
    }
    hipLaunchKernelGGL((rope_restore_kernel<T, L, DEAL>), grid, dim3(256), 0, st, caches, pos,
                       pos_base, n, cfg.n_kv_heads, cfg.head_dim, tab, heads_each);
}

pkv_status launch_rope_restore(const pkv_layer_cfg& cfg, const void* const* k_in,
                               void* const* k_out, int n_layers, const int32_t* pos,
                               int64_t pos_base, int64_t n, hipStream_t st) {
    if (n == 0 || n_layers == 0) return PKV_OK;
    RopeTable tab;
    fill_rope_table(&tab, cfg.head_dim, (double)cfg.rope_theta);
    const int half = cfg.head_dim / 2;
    const int v = cfg.dtype == PKV_BF16 ? 8 : 4;
    const int64_t total = n * (half / v);
    const int block = 256;
    int64_t grid = ceil_div(total, block);
    if (grid > 256 * 64) grid = 256 * 64;  // grid-stride beyond 64 blocks per CU
    // heads in as many parts as bring the launch to kRopeFull workgroups
    const int layers = n_layers < kRopeLayers ? n_layers : kRopeLayers;
    const int64_t parts = std::min<int64_t>(
        cfg.n_kv_heads, std::max<int64_t>(1, kRopeFull / (grid * layers)));
    const int heads_each = (int)ceil_div(cfg.n_kv_heads, parts);
    const bool bf16 = cfg.dtype == PKV_BF16, deal = heads_each < cfg.n_kv_heads;
    for (int l0 = 0; l0 < n_layers; l0 += kRopeLayers) {
        const int cnt = n_layers - l0 < kRopeLayers ? n_layers - l0 : kRopeLayers;
        const dim3 g((unsigned)grid, (unsigned)cnt, (unsigned)ceil_div(cfg.n_kv_heads, heads_each));
#define PKV_ROPE(T, L) (deal ? rope_restore_launch<T, L, true> : rope_restore_launch<T, L, false>)
        auto* const launch = cnt == 1 ? (bf16 ? PKV_ROPE(bf16_t, 1) : PKV_ROPE(float, 1))
                                      : (bf16 ? PKV_ROPE(bf16_t, kRopeLayers)
                                              : PKV_ROPE(float, kRopeLayers));
#undef PKV_ROPE
        launch(g, k_in + l0, k_out + l0, pos, pos_base, n, cfg, heads_each, tab, st);
    }
    return launch_status();
}

}  // namespace pkv
