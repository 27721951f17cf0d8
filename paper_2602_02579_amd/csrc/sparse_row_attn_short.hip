// Step 5, head_dim 128, bf16, for short caches and few rows: one retrieved chunk through its own
// keys (up to 1024 of them), when every job has a CU of its own.
// (Paper: Sec. 4.3 / Algorithm 1; the producer of the chunk caches runs every row of a chunk.)
//
// Such a launch is a chain: load, two products and a softmax per key tile, store.  Nothing fills
// the chip, so the chain is what is cut.  A workgroup of 8 waves owns 128 (row, head) columns of
// a kv head, half of what the pipelined kernels take, and its two groups of four waves (32
// columns per wave) take every other tile of 64 keys and meet in LDS at the end.  The loop is
// small (running maximum, no unrolled pipeline): the pipelined kernel's four-tile body is read
// from memory once per launch for a handful of tiles, and its masked form, which all of these
// tiles take, is the slow one.
// Arithmetic and LDS layouts are those of sparse_row_attn_w8.hip:
//     S^T = K Q^T,   O^T += V^T P^T     (v_mfma_f32_32x32x16_bf16)
// with value rows as the cache holds them, transposed by the LDS read.
//
// Many chunks of one document share a launch (pkv_chunk_attn): a job is then a tile of one
// chunk, the tiles that see most keys first over all chunks.  A launch per chunk -> one for all
// (32 / 8 heads, us): 8 chunks of 64 keys 64 -> 18, 8 of 256 83 -> 26, 4 of 512 62 -> 30, 8 of 1024
// (two jobs per CU each, which took the pipelined kernels one by one) 204 -> 136; the same at 40 / 8
// and 8 / 2 heads and up to 64 chunks, so every chunk length of this kernel shares.
#include <atomic>

#include "attn_common.h"
#include "attn_tile.h"

namespace pkv {

namespace {

constexpr int D = 128;
constexpr int KC = D / 16;               // contraction chunks of S^T
constexpr int DB = D / 32;               // 32-row blocks of O^T
constexpr int kCols = 128;               // columns of a workgroup
constexpr int kThreads = 512;
constexpr int kTileBytes = kBN * D * 2;  // 16 KB: 64 keys of K or V
constexpr int kPair = 4 * kTileBytes;    // K and V of two tiles
constexpr int kLdsBytes = 2 * kPair;

__device__ __forceinline__ void dma16(const void* gptr, uint32_t lds_base) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off"
        :
        : "s"(lds_base), "v"(gptr)
        : "memory", "m0");
}

__global__ __launch_bounds__(kThreads) void attn_short_kernel(AttnParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_red[8];
    __shared__ float s_ml[2][kCols];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave >> 2, cw = wave & 3;   // key half, column block
    const int hh = lane >> 5, l32 = lane & 31;
    const int g = blockIdx.x % p.hkv;
    // the longer tiles first; rows and keys of a chunk start at row0
    int job = (int)(blockIdx.x / p.hkv), row0 = 0, n_rows = p.m, n_keys = p.n_keys;
    if (p.n_chunks > 1) {
        row0 = job % p.n_chunks * p.chunk_len;
        job /= p.n_chunks;
        n_rows = n_keys = min(p.chunk_len, p.m - row0);
    }
    const int tile = p.n_tiles - 1 - job;

    // ---- global -> LDS: this wave fills rows 16 cw .. + 16 of its half's key tile ----------
    // K row r at byte r*256, 16-byte chunk c at c ^ (r & 15); V row r likewise at c ^ (4 (r & 3))
    const uint32_t lds_fill = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)smem + half * 2 * kTileBytes + cw * 16 * 256);
    const int64_t row_elems = (int64_t)p.hkv * D;
    auto fill_pair = [&](int pair) {
        const int key0 = (2 * pair + half) * kBN;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * cw + 4 * i + (lane >> 4);
            const int64_t off = (int64_t)(row0 + min(key0 + r, n_keys - 1)) * row_elems + g * D;
            const uint32_t dst = lds_fill + (pair & 1) * kPair + i * 1024;
            dma16(p.k + off + ((lane & 15) ^ (r & 15)) * 8, dst);
            dma16(p.v + off + ((lane & 15) ^ (4 * (r & 3))) * 8, dst + kTileBytes);
        }
    };
    fill_pair(0);   // in bounds whatever the rows see

    // ---- this lane's column ---------------------------------------------------------------
    const int col = cw * 32 + l32;
    const int rl = col / p.group;
    const int row_in = tile * p.bm + rl, row = row0 + row_in;
    const int head = g * p.group + col % p.group;
    const bool valid = rl < p.bm && row_in < n_rows;
    const int limit = valid ? min(p.row_pos[row], n_keys - 1) : -1;
    bf16x8 qreg[KC];
    {
        const bf16_t* qp = p.q + ((int64_t)row * p.hq + head) * D + hh * 8;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            if (valid) {
                qreg[kc] = *reinterpret_cast<const bf16x8*>(qp + kc * 16);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) qreg[kc][e] = (bf16_t)0.0f;
            }
        }
    }
    int lmax = limit, lmin = valid ? limit : 0x7fffffff;
    for (int o = 32; o > 0; o >>= 1) {
        lmax = max(lmax, __shfl_xor(lmax, o, 64));
        lmin = min(lmin, __shfl_xor(lmin, o, 64));
    }
    lmax = __builtin_amdgcn_readfirstlane(lmax);
    lmin = __builtin_amdgcn_readfirstlane(lmin);
    if (lane == 0) s_red[wave] = lmax;
    __syncthreads();
    int key_max = -1;
#pragma unroll
    for (int w = 0; w < 4; ++w) key_max = max(key_max, s_red[w]);
    const int n_pairs = __builtin_amdgcn_readfirstlane((key_max + 2 * kBN) / (2 * kBN));
    if (n_pairs > 1) fill_pair(1);

    // ---- LDS -> operands (sparse_row_attn_w8.hip) ----------------------------------------------
    const int prow = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
    uint32_t kaddr[KC], vaddr[DB];
    {
        const uint32_t a0 = half * 2 * kTileBytes + prow * 256 + (((prow & 15) ^ hh) * 16);
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kaddr[kc] = a0 ^ (kc << 5);
        const int e = (lane >> 2) & 3, j = lane & 3, gh = (lane >> 4) & 1;
#pragma unroll
        for (int db = 0; db < DB; ++db)
            vaddr[db] = (uint32_t)(half * 2 * kTileBytes + kTileBytes + (8 * hh + e) * 256 +
                                   (((db ^ e) * 4 + gh * 2 + (j >> 1)) * 16) + (j & 1) * 8);
    }
    const float c2 = p.scale_log2;
    float m_run = -INFINITY, l_run = 0.f;   // l_run: this lane's keys only
    f32x16 o_acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o_acc[db][r] = 0.f;

    for (int pair = 0; pair < n_pairs; ++pair) {
        if (pair + 1 < n_pairs) wait_vm<8>();   // this pair has landed, the next is on its way
        else wait_vm<0>();
        __syncthreads();
        const int key0 = (2 * pair + half) * kBN;
        if (key0 <= lmax) {                     // else nobody in this wave sees the tile
            const unsigned char* st = smem + (pair & 1) * kPair;
            f32x16 s[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                                  0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                s[h] = z;
            }
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    s[h] = mfma32(*reinterpret_cast<const bf16x8*>(st + h * 32 * 256 + kaddr[kc]),
                                  qreg[kc], s[h]);
            if (key0 + kBN - 1 > lmin) {
                // element r of block h is key 32 h + 16 (r / 8) + 8 hh + r % 8 of the tile
                const int lim = limit - key0 - 8 * hh;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (32 * h + 16 * (r / 8) + r % 8 > lim) s[h][r] = -INFINITY;
            }
            float mx = m_run;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[h][r]);
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float ref = mx == -INFINITY ? 0.f : mx;
            const float corr = __builtin_amdgcn_exp2f((m_run - ref) * c2);
            m_run = mx;
            if (__any(corr != 1.f)) {
                l_run *= corr;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o_acc[db][r] *= corr;
            }
            const float msc = ref * c2;
            bf16x8 pb[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float e = __builtin_amdgcn_exp2f(s[h][r] * c2 - msc);
                    l_run += e;
                    pb[h][r / 8][r % 8] = (bf16_t)e;
                }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        const unsigned char* a = st + (32 * h + 16 * kk) * 256 + vaddr[db];
                        const bf16x4 lo = lds_read_tr(a), hi = lds_read_tr(a + 4 * 256);
                        const bf16x8 va = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                        o_acc[db] = mfma32(va, pb[h][kk], o_acc[db]);
                    }
        }
        __syncthreads();                        // everybody is done with this pair
        if (pair + 2 < n_pairs) fill_pair(pair + 2);
    }
    wait_vm<0>();                               // a job without keys still has a fill in flight

    // ---- the two halves of the keys meet ----------------------------------------------------
    float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    __syncthreads();
    float* const ex = reinterpret_cast<float*>(smem) + cw * (DB * 16 * 64) + lane;
    if (half == 1) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) ex[(db * 16 + r) * 64] = o_acc[db][r];
        if (hh == 0) {
            s_ml[0][col] = m_run;
            s_ml[1][col] = l_tot;
        }
    }
    __syncthreads();
    if (half == 1 || !valid || n_pairs <= 0) return;
    const float m1 = s_ml[0][col], l1 = s_ml[1][col];
    const float m = fmaxf(m_run, m1), ref = m == -INFINITY ? 0.f : m;
    const float w0 = __builtin_amdgcn_exp2f((m_run - ref) * c2);
    const float w1 = __builtin_amdgcn_exp2f((m1 - ref) * c2);
    l_tot = l_tot * w0 + l1 * w1;
    const float inv = 1.f / l_tot;
    const float a0 = w0 * inv, a1 = w1 * inv;
    const int64_t colg = (int64_t)row * p.hq + head;
    bf16_t* op = p.out + colg * D + 4 * hh;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = (bf16_t)(o_acc[db][4 * r4 + e] * a0 + ex[(db * 16 + 4 * r4 + e) * 64] * a1);
            *reinterpret_cast<bf16x4*>(op + db * 32 + r4 * 8) = v;
        }
    if (hh == 0 && p.lse) p.lse[colg] = m * p.scale + logf(l_tot);
}

}  // namespace

// Measured, pipelined kernel -> this one (us; 32 query heads on 8 kv heads, every row of a chunk):
// 64 keys 18 -> 7.4, 256 24 -> 10, 512 28 -> 14, 768 33 -> 19, 1024 39 -> 24, about 5 + 1.2 per
// 64 keys.  The pipelined kernel with its keys in ranges (few jobs) stands at 19 to 25 from 512
// keys on, so beyond 768 keys such launches stay there (64 rows over 1024: 20).  With more than one
// job per CU or more keys the pipelined kernels' rate decides.
bool attn_short_applies(const pkv_layer_cfg& cfg, int64_t n_keys, int64_t m, int n_splits) {
    const int group = cfg.n_q_heads / cfg.n_kv_heads;
    return group <= kCols && n_keys <= (n_splits == 1 ? 1024 : 768) &&
           ceil_div(m, kCols / group) * cfg.n_kv_heads <= 256;
}

pkv_status launch_attn_short(AttnParams p, hipStream_t st) {
    static std::atomic<bool> configured{false};   // set twice at worst: the calls are idempotent
    if (!configured.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(attn_short_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLdsBytes) != hipSuccess)
            return PKV_ERR_LAUNCH;
        configured.store(true, std::memory_order_release);
    }
    p.bm = kCols / p.group;
    p.n_tiles = (int)ceil_div(p.n_chunks > 1 ? p.chunk_len : p.m, p.bm);
    const int64_t grid = (int64_t)p.n_tiles * p.hkv * (p.n_chunks > 1 ? p.n_chunks : 1);
    if (grid > INT32_MAX) return PKV_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(attn_short_kernel, dim3((unsigned)grid), dim3(kThreads), kLdsBytes, st, p);
    return launch_status();
}

}  // namespace pkv
