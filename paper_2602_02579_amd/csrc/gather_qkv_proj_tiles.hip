// Step 4a and the linear layers on tiles of 128 output features x 64 or 128 tokens
// (head_dim 128, bf16), for launches whose 256 x 256 tiles would leave most of the chip idle:
// the user-query rows of the scoring stage, one retrieved chunk, small models.
// (Paper: Algorithm 1, "Calculate user query KV cache" / "Recompute KV cache at layer l".)
//
// A workgroup of 4 waves (2 token halves x 2 feature halves) owns one head, or 128 outputs of
// a linear layer; a wave owns 16 NT tokens and the 64 features {32 wf .. + 32} and
// {64 + 32 wf .. + 32}, so that both members of a rotary pair (and gate and up of one output)
// sit in the same lane and register index, as in the large tiles.
//
// The contraction runs in steps of 64 through a ring of S stages filled by direct
// global->LDS loads of whole 128-byte lines; layout and swizzle are those of the slab kernel.
// The operands of step t + 1 are read into registers while step t is multiplied, so a stage is
// free again one barrier after its reads and S - 1 steps are in flight.
//
// The accumulators (32 or 64 registers) fit the ordinary vector registers beside the operands,
// and the matrix instructions are the compiler's own, so that it keeps the distance between a
// result and its reader.  Written out in assembly, as the large tiles need them, they left it
// free to put the register copies of the odd last step one slot behind the instruction whose
// result they copy (eight are needed).
//
// What bounds it: few rows stream the weights (64 rows x 28672 outputs x 4096: 235 MB in 45 us,
// 5.2 TB/s, against 64 us on 256 x 256 tiles whose matrix work is three quarters padding); on a
// small model the latency of one tile's chain of steps (256 rows x 1536 x 1024: 21 -> 8 us with
// its finishing launch gone); hundreds of rows the operand bytes through L2, which a small tile
// multiplies (512 rows x 4096 x 4096: 427 MB of L2 requests in 23 us, 71 bytes per ns and CU,
// with the matrix pipe 27 % busy).  64 tokens: three stages of 24 KB, so that two workgroups share a
// CU (six stages for one workgroup measured the same).  128 tokens: four stages of 32 KB and one
// workgroup; two stages and two workgroups were 1 to 30 % slower below 700 rows.
#include <atomic>
#include <type_traits>

#include "proj_tile.h"

namespace pkv {

namespace {

constexpr int kSmallFeat = 128;
constexpr int kSmallStrideF32 = 528;             // bytes per token of a staged fp32 tile row

template <int NT, int S>
struct SmallTile {
    static constexpr int TM = 32 * NT;                        // tokens per tile
    static constexpr int kStage = (kSmallFeat + TM) * 128;    // feature rows, then token rows
    static constexpr int kRing = S * kStage;
    static constexpr int kStaging = TM * kSmallStrideF32;
    static constexpr int kLds = kRing > kStaging ? kRing : kStaging;
    static constexpr int kPerCu = 2 * kLds <= 160 * 1024 ? 2 : 1;
};

template <int MODE, bool EXTRA, int NT, int S>
__global__ __launch_bounds__(256, (SmallTile<NT, S>::kPerCu)) void proj_small_kernel(
    ProjParams p, int n_tok_tiles, int n_tiles, int per_xcd) {
    typedef SmallTile<NT, S> Tile;
    constexpr int TM = Tile::TM;
    constexpr int FILLS = 4 + NT;                // fill instructions of a wave per stage
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;
    const int wt = wave >> 1, wf = wave & 1;

    // ---- which tile: every XCD has its own run of tiles, a few thousand tokens deep -------
    constexpr int kDeep = 2048 / TM;
    int logical = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (logical >= n_tiles * p.n_ksplit) return;
    const int split = logical / n_tiles;
    logical -= split * n_tiles;
    const int n_feat_tiles = 2 * p.tile_begin[3];
    const int per_group = kDeep * n_feat_tiles;
    const int group = logical / per_group;
    const int first_tok = group * kDeep;
    const int rows_in_group = min(kDeep, n_tok_tiles - first_tok);
    const int within = logical - group * per_group;
    const int row0 = (first_tok + within % rows_in_group) * TM;
    const int ft = within / rows_in_group;
    int mat = 0;
    if (MODE == kProjRope) {
        if (ft >= 2 * p.tile_begin[1]) mat = 1;
        if (ft >= 2 * p.tile_begin[2]) mat = 2;
    }
    const int feat0 = (ft - 2 * p.tile_begin[mat]) * kSmallFeat;
    const bf16_t* w = p.w[mat];
    bf16_t* out = p.out[mat];
    if (out == nullptr) return;                  // uniform over the workgroup
    const int n_T = p.hid / 64 / p.n_ksplit;     // steps of this split, >= 1
    const int k_begin = split * n_T * 64;

    // ---- fill side: 8 rows x 128 B per instruction; wave w fills feature rows 32 w .. + 32
    // and token rows 8 NT w .. + 8 NT.  Row r of either operand keeps its 16-byte chunk c at
    // position c ^ ((r >> 1) & 7)
    const int rl = lane >> 3;
    const bf16_t* wptr[4];
    const bf16_t* xptr[NT];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 32 * wave + 8 * j + rl;
        const int gchunk = (lane & 7) ^ ((r >> 1) & 7);
        if (MODE == kProjGated)
            wptr[j] = p.w[r >> 6] + (int64_t)(ft * 64 + (r & 63)) * p.hid + k_begin + gchunk * 8;
        else
            wptr[j] = w + (int64_t)(feat0 + r) * p.hid + k_begin + gchunk * 8;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int r = 8 * NT * wave + 8 * j + rl;
        const int gchunk = (lane & 7) ^ ((r >> 1) & 7);
        const int gr = min(row0 + r, p.m - 1);
        const int64_t src_row = p.row_idx ? p.row_idx[gr] : gr;
        xptr[j] = p.hidden + src_row * p.hid + k_begin + gchunk * 8;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane(lds0 + wave * 4 * 1024);
    const uint32_t lds_x =
        __builtin_amdgcn_readfirstlane(lds0 + kSmallFeat * 128 + wave * NT * 1024);
    // adv is 64, or 0 once the last step has been requested: the ring then re-reads that step
    // into stages nobody uses any more, which keeps the wait counts uniform
    auto issue = [&](uint32_t stage_off, int j, int adv) {
        if (j < 4) {
            dma16(wptr[j], lds_w + stage_off + j * 1024);
            wptr[j] += adv;
        } else {
            dma16(xptr[j - 4], lds_x + stage_off + (j - 4) * 1024);
            xptr[j - 4] += adv;
        }
    };

    // ---- read side: sub-step ks (chunks 4 ks + g4).  Feature block mt starts at tile row
    // 64 (mt / 2) + 32 wf + 16 (mt % 2), token block nt at 16 NT wt + 16 nt
    uint32_t base_w[2], base_x[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const uint32_t swz = (uint32_t)(((4 * ks + g4) ^ (l16 >> 1)) * 16);
        base_w[ks] = (wf * 32 + l16) * 128 + swz;
        base_x[ks] = (kSmallFeat + wt * 16 * NT + l16) * 128 + swz;
    }
    auto ld = [&](uint32_t off) { return *reinterpret_cast<const bf16x8*>(smem + off); };
    bf16x8 fw[2][2][4], fx[2][2][NT];   // [step parity][sub-step][block]
    auto ld_w = [&](uint32_t stage_off, int par, int ks, int mt) {
        fw[par][ks][mt] = ld(stage_off + base_w[ks] + (mt >> 1) * 8192 + (mt & 1) * 2048);
    };
    auto ld_x = [&](uint32_t stage_off, int par, int ks, int nt) {
        fx[par][ks][nt] = ld(stage_off + base_x[ks] + nt * 2048);
    };

    f32x4 acc[4][NT];   // [feature block][token block]
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mt][nt][r] = 0.f;

    // ---- prologue: S steps requested, the operands of step 0 in registers ------------------
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int j = 0; j < FILLS; ++j) issue(s * Tile::kStage, j, s + 1 < n_T ? 64 : 0);
    wait_vm<(S - 1) * FILLS>();
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) ld_w(0, 0, ks, mt);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) ld_x(0, 0, ks, nt);
    }

    // One step: behind the barrier every wave holds the operands of step t, so its stage is
    // refilled with step t + S while the operands of step t + 1 (landed) are read.
    uint32_t off_cur = 0;
    auto step = [&](int t, auto parity) {
        constexpr int PAR = decltype(parity)::value;
        const uint32_t off_next = off_cur + Tile::kStage == Tile::kRing ? 0 : off_cur + Tile::kStage;
        const int adv = t + S + 1 < n_T ? 64 : 0;
        wait_vm<(S - 2) * FILLS>();
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 8; ++g) {            // (sub-step, feature block)
            const int ks = g >> 2, mt = g & 3;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    fw[PAR][ks][mt], fx[PAR][ks][nt], acc[mt][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (g < FILLS) issue(off_cur, g, adv);
            if (g < 6) {                         // 8 feature and 2 NT token operands
                if (g < 4) {
                    ld_w(off_next, PAR ^ 1, g >> 1, 2 * (g & 1));
                    ld_w(off_next, PAR ^ 1, g >> 1, 2 * (g & 1) + 1);
                } else {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) ld_x(off_next, PAR ^ 1, g - 4, nt);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        off_cur = off_next;
    };
    int t = 0;
    for (; t + 1 < n_T; t += 2) {
        step(t, std::integral_constant<int, 0>());
        step(t + 1, std::integral_constant<int, 1>());
    }
    if (t < n_T) step(t, std::integral_constant<int, 0>());
    wait_vm<0>();                 // the ring's trailing fills must not land in the staging
    __syncthreads();

    // ---- epilogue: the tile meets in LDS, whole rows leave 16 B per lane --------------------
    const int tok0 = wt * 16 * NT + l16;         // token of block 0 inside the tile
    if (p.n_ksplit > 1) {
        const int f_total = kSmallFeat * n_feat_tiles;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                *reinterpret_cast<f32x4*>(smem + (tok0 + nt * 16) * kSmallStrideF32 +
                                          ((mt >> 1) * 64 + wf * 32 + (mt & 1) * 16 + 4 * g4) * 4) =
                    acc[mt][nt];
        __syncthreads();
        float* dst = p.partial + ((int64_t)split * p.m + row0) * f_total + ft * kSmallFeat;
#pragma unroll
        for (int it = 0; it < TM / 8; ++it) {
            const int idx = it * 256 + tid;
            const int tok = idx >> 5, ch = idx & 31;
            const f32x4 v = *reinterpret_cast<const f32x4*>(smem + tok * kSmallStrideF32 + ch * 16);
            if (row0 + tok < p.m)
                *reinterpret_cast<f32x4*>(dst + (int64_t)tok * f_total + ch * 4) = v;
        }
        return;
    }
    if (MODE == kProjGated) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a = (float)(bf16_t)acc[j][nt][e];
                    const float b = (float)(bf16_t)acc[j + 2][nt][e];
                    const float s = (float)(bf16_t)silu_f32(a);
                    v[e] = (bf16_t)(s * b);
                }
                *reinterpret_cast<bf16x4*>(smem + (tok0 + nt * 16) * kEpiStride +
                                           (wf * 32 + j * 16 + 4 * g4) * 2) = v;
            }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < TM / 32; ++it) {
            const int idx = it * 256 + tid;
            const int tok = idx >> 3, ch = idx & 7;
            const uint4 v = *reinterpret_cast<const uint4*>(smem + tok * kEpiStride + ch * 16);
            if (row0 + tok < p.m)
                *reinterpret_cast<uint4*>(out + (int64_t)(row0 + tok) * p.n_out + ft * 64 + ch * 8) =
                    v;
        }
        return;
    }
    if (MODE == kProjPlain) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (bf16_t)acc[mt][nt][e];
                *reinterpret_cast<bf16x4*>(
                    smem + (tok0 + nt * 16) * kEpiStride +
                    ((mt >> 1) * 64 + wf * 32 + (mt & 1) * 16 + 4 * g4) * 2) = v;
            }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < TM / 16; ++it) {
            const int idx = it * 256 + tid;
            const int tok = idx >> 4, ch = idx & 15;
            bf16x8 v = *reinterpret_cast<const bf16x8*>(smem + tok * kEpiStride + ch * 16);
            if (row0 + tok < p.m) {
                const int64_t o = (int64_t)(row0 + tok) * p.n_out + feat0 + ch * 8;
                if (p.residual) {
                    const bf16x8 r = *reinterpret_cast<const bf16x8*>(p.residual + o);
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = (bf16_t)((float)v[e] + (float)r[e]);
                }
                *reinterpret_cast<bf16x8*>(out + o) = v;
            }
        }
        return;
    }
    // Q | K | V: bias, head norm, rotation; features 32 wf + 16 j + 4 g4 + e and + 64
    const int head = feat0 / kSmallFeat;
    const int heads_out = mat == 0 ? p.hq : p.hkv;
    const bool rotate = mat != 2;
    const bf16_t* bias = EXTRA && p.bias[mat] ? p.bias[mat] + head * kSmallFeat : nullptr;
    const bf16_t* gain = EXTRA && mat != 2 ? p.norm_w[mat] : nullptr;
    float* const s_sq = reinterpret_cast<float*>(smem + TM * kEpiStride);   // [2][TM]
    if (EXTRA && bias) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const bf16x4 bv = *reinterpret_cast<const bf16x4*>(
                bias + (mt >> 1) * 64 + wf * 32 + (mt & 1) * 16 + 4 * g4);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[mt][nt][e] += (float)bv[e];
        }
    }
    if (EXTRA && gain) {
        // the lane holds 16 of the token's 128 features, lanes ^ 16, ^ 32 and ^ 48 another 48,
        // the wave of the other feature half the rest
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float ss = 0.f;
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int e = 0; e < 4; ++e) ss += acc[mt][nt][e] * acc[mt][nt][e];
            ss += __shfl_xor(ss, 16);
            ss += __shfl_xor(ss, 32);
            if (g4 == 0) s_sq[wf * TM + tok0 + nt * 16] = ss;
        }
        __syncthreads();
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int tok = tok0 + nt * 16;
        const float4* cs =
            reinterpret_cast<const float4*>(p.cs + (int64_t)min(row0 + tok, p.m - 1) * 64);
        float rnorm = 1.f;
        if (EXTRA && gain)
            rnorm = 1.0f / sqrtf((s_sq[tok] + s_sq[TM + tok]) * (1.0f / kSmallFeat) + p.norm_eps);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i0 = wf * 32 + j * 16 + 4 * g4;   // pair index of element 0
            float a[4], b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = acc[j][nt][e];
                b[e] = acc[j + 2][nt][e];
            }
            if (EXTRA && gain) {
                const bf16x4 ga = *reinterpret_cast<const bf16x4*>(gain + i0);
                const bf16x4 gb = *reinterpret_cast<const bf16x4*>(gain + i0 + 64);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a[e] = a[e] * rnorm * (float)ga[e];
                    b[e] = b[e] * rnorm * (float)gb[e];
                }
            }
            if (rotate) {
                const float4 t0 = cs[i0 / 2], t1 = cs[i0 / 2 + 1];
                const float c[4] = {t0.x, t0.z, t1.x, t1.z};
                const float s[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float ra = a[e] * c[e] - b[e] * s[e];
                    const float rb = b[e] * c[e] + a[e] * s[e];
                    a[e] = ra;
                    b[e] = rb;
                }
            }
            bf16x4 va, vb;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                va[e] = (bf16_t)a[e];
                vb[e] = (bf16_t)b[e];
            }
            *reinterpret_cast<bf16x4*>(smem + tok * kEpiStride + i0 * 2) = va;
            *reinterpret_cast<bf16x4*>(smem + tok * kEpiStride + (i0 + 64) * 2) = vb;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < TM / 16; ++it) {
        const int idx = it * 256 + tid;
        const int tok = idx >> 4, ch = idx & 15;
        const uint4 v = *reinterpret_cast<const uint4*>(smem + tok * kEpiStride + ch * 16);
        const int row = row0 + tok;
        if (row < p.m) {
            const int64_t orow = (EXTRA && mat != 0 && p.dst_row) ? p.dst_row[row] : row;
            *reinterpret_cast<uint4*>(out + (orow * heads_out + head) * kSmallFeat + ch * 8) = v;
        }
    }
}

template <int MODE, bool EXTRA, int NT, int S>
pkv_status launch_one(const ProjParams& p, hipStream_t st) {
    static std::atomic<bool> configured{false};   // set twice at worst: the calls are idempotent
    typedef SmallTile<NT, S> Tile;
    if (!configured.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(
                reinterpret_cast<const void*>(proj_small_kernel<MODE, EXTRA, NT, S>),
                hipFuncAttributeMaxDynamicSharedMemorySize, Tile::kLds) != hipSuccess)
            return PKV_ERR_LAUNCH;
        configured.store(true, std::memory_order_release);
    }
    const int n_tok_tiles = (int)ceil_div(p.m, Tile::TM);
    const int64_t n_tiles = (int64_t)n_tok_tiles * 2 * p.tile_begin[3];
    if (n_tiles * p.n_ksplit > (1 << 30)) return PKV_ERR_SHAPE;
    const int per_xcd = (int)ceil_div(n_tiles * p.n_ksplit, 8);
    hipLaunchKernelGGL((proj_small_kernel<MODE, EXTRA, NT, S>), dim3((unsigned)(per_xcd * 8)),
                       dim3(256), Tile::kLds, st, p, n_tok_tiles, (int)n_tiles, per_xcd);
    return PKV_OK;
}

}  // namespace

template <int MODE, bool EXTRA>
pkv_status launch_proj_small(int tokens, const ProjParams& p, hipStream_t st) {
    return tokens == 64 ? launch_one<MODE, EXTRA, 2, 3>(p, st)
                        : launch_one<MODE, EXTRA, 4, 4>(p, st);
}
template pkv_status launch_proj_small<kProjRope, false>(int, const ProjParams&, hipStream_t);
template pkv_status launch_proj_small<kProjRope, true>(int, const ProjParams&, hipStream_t);
template pkv_status launch_proj_small<kProjPlain, false>(int, const ProjParams&, hipStream_t);
template pkv_status launch_proj_small<kProjGated, false>(int, const ProjParams&, hipStream_t);

}  // namespace pkv
