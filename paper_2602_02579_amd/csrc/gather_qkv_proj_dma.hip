// Step 4a on the matrix cores, head_dim 128, bf16: the gathered projection
// C^T[features, tokens] = W . X^T with the rotation of Q and K fused into the
// store.  (Paper: Algorithm 1, "Recompute KV cache at layer l" / "Calculate
// user query KV cache"; Appendix E: only the selected rows go through the
// projection.)
//
// One workgroup (4 waves, 2 x 2) owns 256 tokens x 256 output features (two
// heads); a wave owns 128 tokens x one head as 8 x 8 accumulators of
// v_mfma_f32_16x16x32_bf16 with the features on the accumulator rows.  A lane
// then holds, for one token, features 4(l/16) + {0..3} of every 16-block:
// both members (i, i + 64) of a rotary pair sit in the same lane and register
// index, and four consecutive features make one 8-byte piece of the output row.
//
// Why 16 x 16 x 32 and not 32 x 32 x 16 (same rate on paper, same operand bytes from LDS):
// the launch is held by the power limit, and the smaller tile moves half the accumulator
// bytes per product through the register file.  In registers alone, on Gaussian
// activations x N(0, 0.02^2) weights, 256 CUs sustain 2044 TFLOP/s with it against 1757
// (2444 / 2422 on zeros, where nothing is limited).  Measured on this kernel, 8192^3:
// 1358 -> 1467 TFLOP/s; 6656 rows x 28672 outputs x 4096: 1293 -> 1386.
//
// The contraction runs in steps of 32 through a 5-stage LDS ring filled by
// direct global->LDS loads (16 bytes per lane; the gather is free, every lane
// carries its own row pointer).  A row of a stage is 64 bytes; the 16-byte
// chunk c of row r is stored at position c ^ ((r >> 2) & 3), which makes both
// the 1 KB-contiguous fill and the ds_read_b128 of the MFMA operands
// conflict-free.  One barrier per stage, placed between the two halves of the
// token blocks so that the operands of the next stage are already in flight
// while the second half's MFMAs run.
//
// Tiles are numbered so that each XCD (workgroup id mod 8) works through its own
// contiguous run of tiles, 8 token tiles deep, and its L2 sees few distinct
// operand panels at a time.
//
// A launch that cannot fill 256 CUs with such tiles takes lower or smaller ones
// (plan_tiles) and, with very few rows (the user-query projection of the scoring stage),
// splits its contraction: every split writes fp32 partial tiles, and a second small
// kernel adds them in a fixed order, rotates and rounds (deterministic: no atomics).
#include <algorithm>
#include <atomic>

#include "proj_tile.h"

namespace pkv {

namespace {

constexpr int D = 128;
constexpr int T = kProjDmaTile;                  // tokens and features per tile
constexpr int BK = 32;                           // contraction per stage
constexpr int NS = 5;                            // LDS stages
constexpr int kRowBytes = BK * 2;                // 64
constexpr int kOperandBytes = T * kRowBytes;     // 16 KB: 256 rows of one operand
constexpr int kStageBytes = 2 * kOperandBytes;   // token rows, then feature rows
constexpr int kLdsBytes = NS * kStageBytes;      // 160 KB, all of a CU's LDS
constexpr int kEpiStrideF32 = 528;               // same for fp32 partial tiles (32 tokens)
constexpr int kGroup = 8;                        // token tiles per group

// EXTRA (Q | K | V mode only): the launch has projection biases, per-head norm gains and/or
// a fused cache update (K/V rows stored at dst_row)
// what a tile is and which part of it a lane owns (filled by the kernels, read by the
// epilogue)
struct TileCtx {
    int lane, wave, g4, l16, wt, wf;
    int split, ft, mat, feat0, row0, heads_out;
    bf16_t* out;
};

// rotate pairs in registers / add the residual / gate, round, stage through LDS, store
// 16 B per lane; or store the fp32 partial tile of a split contraction.  Called after the
// main loop, when nothing is still writing the LDS stages.
template <int MODE, bool EXTRA, int NQ>
__device__ __forceinline__ void tile_epilogue(const ProjParams& p, f32x4 (&acc)[8][2 * NQ],
                                              const TileCtx& c, unsigned char* smem) {
    const int lane = c.lane, wave = c.wave, g4 = c.g4, l16 = c.l16, wt = c.wt, wf = c.wf;
    const int split = c.split, ft = c.ft, mat = c.mat, feat0 = c.feat0, row0 = c.row0;
    const int heads_out = c.heads_out;
    bf16_t* out = c.out;
    // ---- epilogue: rotate pairs in registers, round once, stage, store 16 B per lane ----
    if (out == nullptr) return;   // uniform over the workgroup
    __syncthreads();              // LDS stages are free
    if (p.n_ksplit > 1) {
        // fp32 partial tile of this split, staged so that a lane stores 16 B and a
        // row 512 B: partial[split][row][256 ft + 128 wf + feature]
        unsigned char* epf = smem + wave * (32 * kEpiStrideF32);
        const int f_total = T * p.tile_begin[3];
#pragma unroll
        for (int tb = 0; tb < NQ; ++tb) {
            const int rbase = row0 + wt * (32 * NQ) + tb * 32;
            if (rbase >= p.m) break;   // wave-uniform
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int mt = 0; mt < 8; ++mt) {
                    acc_take(acc[mt][tb * 2 + nt]);
                    *reinterpret_cast<f32x4*>(epf + (nt * 16 + l16) * kEpiStrideF32 +
                                              (mt * 16 + 4 * g4) * 4) = acc[mt][tb * 2 + nt];
                }
#pragma unroll
            for (int it = 0; it < 16; ++it) {
                const int idx = it * 64 + lane;
                const int tok = idx >> 5, ch = idx & 31;
                const int row = rbase + tok;
                const f32x4 v = *reinterpret_cast<const f32x4*>(epf + tok * kEpiStrideF32 + ch * 16);
                if (row < p.m)
                    *reinterpret_cast<f32x4*>(p.partial + ((int64_t)split * p.m + row) * f_total +
                                              ft * T + wf * 128 + ch * 4) = v;
            }
        }
        return;
    }
    unsigned char* epi = smem + wave * (16 * NQ * kEpiStride);
    if (MODE == kProjPlain) {
        // the wave's 32 NQ tokens x 128 outputs: round the products, stage, then add the
        // residual (if any) 16 B per lane and round again
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int nt = 0; nt < NQ; ++nt) {
                unsigned char* erow = epi + (nt * 16 + l16) * kEpiStride;
#pragma unroll
                for (int mt = 0; mt < 8; ++mt) {
                    acc_take(acc[mt][half * NQ + nt]);
                    bf16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (bf16_t)acc[mt][half * NQ + nt][e];
                    *reinterpret_cast<bf16x4*>(erow + (mt * 16 + 4 * g4) * 2) = v;
                }
            }
#pragma unroll
            for (int it = 0; it < 4 * NQ; ++it) {
                const int idx = it * 64 + lane;
                const int tok = idx >> 4, ch = idx & 15;
                const int row = row0 + wt * (32 * NQ) + half * (16 * NQ) + tok;
                bf16x8 v = *reinterpret_cast<const bf16x8*>(epi + tok * kEpiStride + ch * 16);
                if (row < p.m) {
                    const int64_t o = (int64_t)row * p.n_out + feat0 + wf * 128 + ch * 8;
                    if (p.residual) {
                        const bf16x8 r = *reinterpret_cast<const bf16x8*>(p.residual + o);
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = (bf16_t)((float)v[e] + (float)r[e]);
                    }
                    *reinterpret_cast<bf16x8*>(out + o) = v;
                }
            }
        }
        return;
    }
    if (MODE == kProjGated) {
        // the wave's 32 NQ tokens x 64 outputs: gate in feature blocks 0..3 and up in 4..7
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int nt = 0; nt < NQ; ++nt) {
                const int tt = half * NQ + nt;
                unsigned char* erow = epi + (nt * 16 + l16) * kEpiStride;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    acc_take(acc[mt][tt]);
                    acc_take(acc[mt + 4][tt]);
                    bf16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float a = (float)(bf16_t)acc[mt][tt][e];
                        const float b = (float)(bf16_t)acc[mt + 4][tt][e];
                        const float s = (float)(bf16_t)silu_f32(a);
                        v[e] = (bf16_t)(s * b);
                    }
                    *reinterpret_cast<bf16x4*>(erow + (mt * 16 + 4 * g4) * 2) = v;
                }
            }
#pragma unroll
            for (int it = 0; it < 2 * NQ; ++it) {
                const int idx = it * 64 + lane;
                const int tok = idx >> 3, ch = idx & 7;
                const int row = row0 + wt * (32 * NQ) + half * (16 * NQ) + tok;
                const uint4 v = *reinterpret_cast<const uint4*>(epi + tok * kEpiStride + ch * 16);
                if (row < p.m)
                    *reinterpret_cast<uint4*>(out + (int64_t)row * p.n_out + ft * 128 + wf * 64 +
                                              ch * 8) = v;
            }
        }
        return;
    }
    const int head = feat0 / D + wf;
    const bool rotate = mat != 2;
    // block variants: bias of this head's features, gains of the head norm (Q and K only)
    const bf16_t* bias = EXTRA && p.bias[mat] ? p.bias[mat] + head * D : nullptr;
    const bf16_t* gain = EXTRA && mat != 2 ? p.norm_w[mat] : nullptr;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int nt = 0; nt < NQ; ++nt) {
            const int tt = half * NQ + nt;
            const int row = min(row0 + wt * (32 * NQ) + tt * 16 + l16, p.m - 1);
            const float4* cs = reinterpret_cast<const float4*>(p.cs + (int64_t)row * (D / 2));
            unsigned char* erow = epi + (nt * 16 + l16) * kEpiStride;
#pragma unroll
            for (int mt = 0; mt < 8; ++mt) acc_take(acc[mt][tt]);
            float rnorm = 1.f;
            if (EXTRA) {
                if (bias) {
#pragma unroll
                    for (int mt = 0; mt < 8; ++mt) {
                        const bf16x4 bv =
                            *reinterpret_cast<const bf16x4*>(bias + mt * 16 + 4 * g4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[mt][tt][e] += (float)bv[e];
                    }
                }
                if (gain) {
                    // the lane holds 32 of the token's 128 features, lanes ^ 16, ^ 32 and
                    // ^ 48 the others
                    float ss = 0.f;
#pragma unroll
                    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) ss += acc[mt][tt][e] * acc[mt][tt][e];
                    ss += __shfl_xor(ss, 16);
                    ss += __shfl_xor(ss, 32);
                    rnorm = 1.0f / sqrtf(ss * (1.0f / D) + p.norm_eps);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const int i0 = mt * 16 + 4 * g4;   // pair index of element 0
                float a[4], b[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a[e] = acc[mt][tt][e];
                    b[e] = acc[mt + 4][tt][e];
                }
                if (EXTRA && gain) {
                    const bf16x4 ga = *reinterpret_cast<const bf16x4*>(gain + i0);
                    const bf16x4 gb = *reinterpret_cast<const bf16x4*>(gain + i0 + D / 2);
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
                *reinterpret_cast<bf16x4*>(erow + i0 * 2) = va;
                *reinterpret_cast<bf16x4*>(erow + (i0 + D / 2) * 2) = vb;
            }
        }
        // the wave's own 16 NQ tokens x 256 B, now 16 B per lane and 256 B per row
#pragma unroll
        for (int it = 0; it < 4 * NQ; ++it) {
            const int idx = it * 64 + lane;
            const int tok = idx >> 4, ch = idx & 15;
            const int row = row0 + wt * (32 * NQ) + half * (16 * NQ) + tok;
            const uint4 v = *reinterpret_cast<const uint4*>(epi + tok * kEpiStride + ch * 16);
            if (row < p.m) {
                const int64_t orow = (EXTRA && mat != 0 && p.dst_row) ? p.dst_row[row] : row;
                *reinterpret_cast<uint4*>(out + (orow * heads_out + head) * D + ch * 8) = v;
            }
        }
    }
}


template <int MODE, bool EXTRA = false>
__global__ __launch_bounds__(256) void proj_dma_kernel(ProjParams p, int n_tok_tiles,
                                                       int n_tiles, int per_xcd) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;
    const int wt = wave >> 1, wf = wave & 1;

    // ---- which tile --------------------------------------------------------------
    int logical = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (logical >= n_tiles * p.n_ksplit) return;
    const int split = logical / n_tiles;
    logical -= split * n_tiles;
    const int n_feat_tiles = p.tile_begin[3];
    const int per_group = kGroup * n_feat_tiles;
    const int group = logical / per_group;
    const int first_tok = group * kGroup;
    const int rows_in_group = min(kGroup, n_tok_tiles - first_tok);
    const int within = logical - group * per_group;
    const int tok_tile = first_tok + within % rows_in_group;
    const int ft = within / rows_in_group;
    int mat = 0;
    if (MODE == kProjRope) {
        if (ft >= p.tile_begin[1]) mat = 1;
        if (ft >= p.tile_begin[2]) mat = 2;
    }
    const int feat0 = (ft - p.tile_begin[mat]) * T;   // first output feature of the tile
    const bf16_t* w = p.w[mat];
    bf16_t* out = p.out[mat];
    const int heads_out = mat == 0 ? p.hq : p.hkv;
    const int row0 = tok_tile * T;

    const int n_k = p.hid / BK / p.n_ksplit;   // stages of this split; >= NS (launcher)
    const int k_begin = split * n_k * BK;

    // ---- fill side: wave w, instruction j covers rows 16 (4w + j) .. + 16 ------------
    const int sw = (lane & 3) ^ ((lane >> 4) & 3);   // global chunk that lands at lane & 3
    const bf16_t* xptr[4];
    const bf16_t* wptr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = (wave * 4 + j) * 16 + (lane >> 2);
        const int gr = min(row0 + r, p.m - 1);
        const int64_t src_row = p.row_idx ? p.row_idx[gr] : gr;
        xptr[j] = p.hidden + src_row * p.hid + k_begin + sw * 8;
        if (MODE == kProjGated) {
            // tile row r: half r / 128 of the tile's 128 outputs, then 64 gate rows and
            // 64 up rows, so that accumulator blocks (0, 1) and (2, 3) of a wave hold
            // gate and up of the same outputs
            const int f = ft * 128 + (r >> 7) * 64 + (r & 63);
            wptr[j] = p.w[(r >> 6) & 1] + (int64_t)f * p.hid + k_begin + sw * 8;
        } else {
            wptr[j] = w + (int64_t)(feat0 + r) * p.hid + k_begin + sw * 8;
        }
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const uint32_t lds_fill = __builtin_amdgcn_readfirstlane(lds0 + wave * 4 * 1024);
    // one fill instruction: 16 rows of the token operand (which = 0) or of the
    // feature operand (which = 1).  adv is BK, or 0 once the last stage has been
    // requested: the ring then keeps re-reading that stage into slots nobody reads
    // any more, which keeps the loop and its wait counts uniform.
    auto issue_one = [&](int stage, int j, int which, int adv) {
        const uint32_t base = lds_fill + stage * kStageBytes + j * 1024;
        if (which == 0) {
            dma16(xptr[j], base);
            xptr[j] += adv;
        } else {
            dma16(wptr[j], base + kOperandBytes);
            wptr[j] += adv;
        }
    };

    // ---- read side -----------------------------------------------------------------
    // operand of row r (16 rows per MFMA block, contraction chunk g4 of the stage's four):
    // position g4 ^ ((r >> 2) & 3)
    const int pos = g4 ^ ((l16 >> 2) & 3);
    const int off_x = (wt * 128 + l16) * kRowBytes + pos * 16;
    const int off_w = kOperandBytes + (wf * 128 + l16) * kRowBytes + pos * 16;
    bf16x8 fw[8], fx[2][4];   // [feature block], [half of the token blocks][token block]
    auto ld_w = [&](int stage, int mt) {
        return *reinterpret_cast<const bf16x8*>(smem + stage * kStageBytes + off_w +
                                                mt * 16 * kRowBytes);
    };
    auto ld_x = [&](int stage, int nt) {
        return *reinterpret_cast<const bf16x8*>(smem + stage * kStageBytes + off_x +
                                                nt * 16 * kRowBytes);
    };

    f32x4 acc[8][8];   // [feature block][token block]
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
        for (int nt = 0; nt < 8; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mt][nt][r] = 0.f;
    // Half a stage: 32 MFMAs on token blocks 4 half .. + 4, one fill instruction after every
    // eighth (half a stage's fills per half, so the memory pipeline sees a steady trickle
    // instead of a burst that stalls the wave).  The operands of the next half are read from
    // LDS in the same rhythm: token blocks 4..7 of this stage, or token blocks 0..3 of stage
    // lstage and its feature blocks, each right after its last use.
    auto mfma32 = [&](int half, int fill_stage, int j0, int adv, int lstage) {
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            fx[half ^ 1][n] = ld_x(lstage, half == 0 ? 4 + n : n);
#pragma unroll
            for (int mt = 2 * n; mt < 2 * n + 2; ++mt) {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    mfma_16x16x32(acc[mt][4 * half + nt], fw[mt], fx[half][nt]);
                if (half == 1) fw[mt] = ld_w(lstage, mt);
            }
            __builtin_amdgcn_sched_barrier(0);
            issue_one(fill_stage, j0 + (n >> 1), n & 1, adv);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // prologue: stages 0 .. NS-3 and the first half of stage NS-2 in flight
#pragma unroll
    for (int s = 0; s < NS - 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            issue_one(s, j, 0, BK);
            issue_one(s, j, 1, BK);
        }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        issue_one(NS - 2, j, 0, BK);
        issue_one(NS - 2, j, 1, BK);
    }
    wait_vm<8 * (NS - 3) + 4>();  // stage 0 of this wave has landed
    __syncthreads();              // ... and everyone's
#pragma unroll
    for (int mt = 0; mt < 8; ++mt) fw[mt] = ld_w(0, mt);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) fx[0][nt] = ld_x(0, nt);
    int st_cur = 0;               // t mod NS
    for (int t = 0; t < n_k; ++t) {
        const int st_next = st_cur + 1 == NS ? 0 : st_cur + 1;
        const int st_fill = st_cur == 0 ? NS - 1 : st_cur - 1;          // (t + NS - 1) mod NS
        const int st_fill_b = st_fill == 0 ? NS - 1 : st_fill - 1;      // (t + NS - 2) mod NS
        mfma32(0, st_fill_b, 2, t + NS - 1 < n_k ? BK : 0, st_cur);
        wait_vm<8 * (NS - 3)>();  // stage t+1 has landed; the younger ones stay in flight
        __syncthreads();          // ... for everyone; and everyone is done with stage t-1
        mfma32(1, st_fill, 0, t + NS < n_k ? BK : 0, st_next);
        st_cur = st_next;
    }
    wait_vm<0>();                 // the ring's trailing fills must not land in the staging
    acc_settle();

    // ---- epilogue -----------------------------------------------------------------------
    TileCtx ctx;
    ctx.lane = lane; ctx.wave = wave; ctx.g4 = g4; ctx.l16 = l16; ctx.wt = wt; ctx.wf = wf;
    ctx.split = split; ctx.ft = ft; ctx.mat = mat; ctx.feat0 = feat0; ctx.row0 = row0;
    ctx.heads_out = heads_out; ctx.out = out;
    tile_epilogue<MODE, EXTRA, 4>(p, acc, ctx, smem);
}

// ---------------------------------------------------------------------------------------
// The same tile, or one of 64 NQ = 192 tokens, with the contraction in steps of 64 ("slabs"): every fill instruction
// fetches whole 128-byte lines (8 rows x 128 B), which the memory pipeline serves at
// 1.7 x the rate of the 64-byte row pieces of the kernel above and at a higher clock.
//
// LDS: two steps' worth of units of 8 KB; a unit is 64 rows x 128 B of one operand.  A step T
// needs four feature units W0..W3 (tile rows 64 i ..) and NQ token units X0.., where
// X_q holds the rows both token halves consume in part q of the step: tile rows
// 32 q .. + 32 and 32 NQ + 32 q .. + 32.  Step T uses the units of its parity.
// The 16-byte chunk c of unit row r is stored at position c ^ ((r >> 1) & 7): two 128-byte
// rows span the 64 banks, so the sixteen lanes that an operand read serves per clock (rows
// r .. r + 15, one logical chunk) must differ in (r & 1, position) - with c ^ (r & 7) rows r
// and r + 8 met in one bank group and every read took two passes (SQ_LDS_BANK_CONFLICT).
//
// A step is NQ quarters (of the 256-token tile's 128 MFMAs per wave) of 32 MFMAs; quarter q
// multiplies the wave's eight feature blocks by its token blocks 2 q, 2 q + 1 for both 32-wide
// sub-steps.  The feature operands of a whole step live in registers (loaded during the last
// two quarters of the previous step), so the W units of step T are free again when T begins and
// are refilled with step T + 2 from its first quarter on; X_q is free after quarter q - 1 and is
// refilled behind them.  One barrier per quarter, two fill instructions per wave
// and unit, one fill instruction every eight MFMAs where there are four quarters; with three the
// features' fills all go out in the first, so that they have three quarters to land.
// Needs an even number (>= 2) of steps per split.
constexpr int kUnitBytes = 64 * 128;
template <int NQ>
constexpr int kSlabLdsBytes = 2 * (4 + NQ) * kUnitBytes;

template <int MODE, bool EXTRA, int NQ>
__device__ __forceinline__ void slab_tile(const ProjParams& p, unsigned char* smem, int row0,
                                          int ft, int split) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;
    const int wt = wave >> 1, wf = wave & 1;

    int mat = 0;
    if (MODE == kProjRope) {
        if (ft >= p.tile_begin[1]) mat = 1;
        if (ft >= p.tile_begin[2]) mat = 2;
    }
    const int feat0 = (ft - p.tile_begin[mat]) * T;
    const bf16_t* w = p.w[mat];
    bf16_t* out = p.out[mat];
    const int heads_out = mat == 0 ? p.hq : p.hkv;

    const int n_T = p.hid / 64 / p.n_ksplit;   // steps of this split: even, >= 2 (launcher)
    const int k_begin = split * n_T * 64;

    // ---- fill side: wave w issues instructions j = 0, 1 of every unit: unit rows
    // 8 (2 w + j) .. + 8; lane = (row in the eight, position), fetching the chunk that
    // belongs at that position: pos ^ ((unit row >> 1) & 7) = pos ^ (4 j + (row >> 1))
    constexpr int kFills = 8 + 2 * NQ;   // fill instructions of a wave per step
    const int rl = lane >> 3;
    const bf16_t* wptr[4][2];
    const bf16_t* xptr[NQ][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int ur = 8 * (2 * wave + j) + rl;   // row inside the unit
            const int gchunk = (lane & 7) ^ ((ur >> 1) & 7);
            const int r = 64 * i + ur;                // feature row of the tile
            if (MODE == kProjGated) {
                const int f = ft * 128 + (r >> 7) * 64 + (r & 63);
                wptr[i][j] = p.w[(r >> 6) & 1] + (int64_t)f * p.hid + k_begin + gchunk * 8;
            } else {
                wptr[i][j] = w + (int64_t)(feat0 + r) * p.hid + k_begin + gchunk * 8;
            }
            if (i >= NQ) continue;
            const int xr = 32 * i + (ur < 32 ? ur : 32 * NQ - 32 + ur);   // token row of the tile
            const int gr = min(row0 + xr, p.m - 1);
            const int64_t src_row = p.row_idx ? p.row_idx[gr] : gr;
            xptr[i][j] = p.hidden + src_row * p.hid + k_begin + gchunk * 8;
        }
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const uint32_t lds_fill = __builtin_amdgcn_readfirstlane(lds0 + wave * 2 * 1024);
    // unit i of the feature (which = 1) or token (which = 0) operand of a step with
    // parity par; adv is 64, or 0 once the last step has been requested
    auto issue_w = [&](int par, int i, int j, int adv) {
        dma16(wptr[i][j], lds_fill + (par * (4 + NQ) + i) * kUnitBytes + j * 1024);
        wptr[i][j] += adv;
    };
    auto issue_x = [&](int par, int i, int j, int adv) {
        dma16(xptr[i][j], lds_fill + (par * (4 + NQ) + 4 + i) * kUnitBytes + j * 1024);
        xptr[i][j] += adv;
    };

    // ---- read side: byte offsets of the lane's operand pieces --------------------------
    // sub-step ks (32 of the contraction: chunks 4 ks + g4); feature block mt (16 rows):
    // base_w + mt * 2048; token block nt of quarter q: base_x + q * 8192 + nt * 2048
    uint32_t base_w[2][2], base_x[2][2];
#pragma unroll
    for (int par = 0; par < 2; ++par)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint32_t swz = (uint32_t)(((4 * ks + g4) ^ (l16 >> 1)) * 16);
            base_w[par][ks] = par * (4 + NQ) * kUnitBytes + 2 * wf * kUnitBytes + l16 * 128 + swz;
            base_x[par][ks] = par * (4 + NQ) * kUnitBytes + 4 * kUnitBytes + (wt * 32 + l16) * 128 + swz;
        }
    auto ld = [&](uint32_t off) { return *reinterpret_cast<const bf16x8*>(smem + off); };

    bf16x8 fw0[2][8];   // [step parity][feature block], sub-step 0
    bf16x8 fw1[8];      // [feature block], sub-step 1
    bf16x8 fx[2][2][2]; // [quarter parity][sub-step][token block]

    f32x4 acc[8][2 * NQ];   // [feature block][token block]
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2 * NQ; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mt][nt][r] = 0.f;

    // ---- prologue: steps 0 and 1 requested; operands of step 0, quarter 0 loaded --------
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        const int adv = par + 1 < n_T ? 64 : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) issue_w(par, i, j, adv);
#pragma unroll
        for (int i = 0; i < NQ; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) issue_x(par, i, j, adv);
    }
    wait_vm<2 * kFills - 12>();   // W0..W3, X0 and X1 of step 0 (the first twelve) landed
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < 8; ++mt) {
        fw0[0][mt] = ld(base_w[0][0] + mt * 2048);
        fw1[mt] = ld(base_w[0][1] + mt * 2048);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) fx[0][ks][nt] = ld(base_x[0][ks] + nt * 2048);
    __syncthreads();   // everybody holds step 0's feature operands: its W units may be refilled

    // One quarter: 32 MFMAs in four groups (sub-step outer, token block inner, eight feature
    // blocks each) on token blocks 2 Q, 2 Q + 1; one fill instruction after every group.
    // The LDS reads of the quarter (token operands of the next quarter; in quarter 2 the
    // sub-step 0 feature operands of the next step into the other register set; in quarter 3
    // the sub-step 1 ones, each right after its last use - which is why quarter 3 runs
    // sub-step 1 first) all go out in the first three groups, so that they have returned when
    // the barrier that ends the quarter waits for them.  PAR = parity of the step.
#define PKV_QUARTER(PAR, Q, ADV)                                                          \
    {                                                                                     \
        _Pragma("unroll") for (int g_ = 0; g_ < 4; ++g_) {                                \
            const int ks = (Q) == NQ - 1 ? 1 - (g_ >> 1) : g_ >> 1;                       \
            const int nt = g_ & 1;                                                        \
            constexpr int qp_ = (PAR) * (NQ & 1);   /* an odd NQ flips the parity */      \
            _Pragma("unroll") for (int mt = 0; mt < 8; ++mt) {                            \
                const bf16x8 a_ = ks == 0 ? fw0[PAR][mt] : fw1[mt];                       \
                mfma_16x16x32(acc[mt][2 * (Q) + nt], a_, fx[((Q) + qp_) & 1][ks][nt]);    \
                if ((Q) == NQ - 1 && g_ == 1)   /* last use: take step T + 1's operand */ \
                    fw1[mt] = ld(base_w[(PAR) ^ 1][1] + mt * 2048);                       \
            }                                                                             \
            __builtin_amdgcn_sched_barrier(0);                                            \
            /* fill, 4 quarters: feature units 2 Q, 2 Q + 1, then token units in twos; */ \
            /* 3 quarters: all feature units, token units 0 and 1, token unit 2        */ \
            if (NQ == 4) {                                                                \
                if ((Q) < 2) issue_w(PAR, 2 * (Q) + (g_ >> 1), g_ & 1, ADV);              \
                else issue_x(PAR, 2 * ((Q) - 2) + (g_ >> 1), g_ & 1, ADV);                \
            } else if ((Q) == 0) {                                                        \
                issue_w(PAR, g_, 0, ADV);                                                 \
                issue_w(PAR, g_, 1, ADV);                                                 \
            } else if ((Q) == 1) {                                                        \
                issue_x(PAR, g_ >> 1, g_ & 1, ADV);                                       \
            } else if (g_ < 2) {                                                          \
                issue_x(PAR, 2, g_, ADV);                                                 \
            }                                                                             \
            /* token operands of the next quarter: 2, 1, 1, 0 per group */                \
            _Pragma("unroll") for (int n_ = 0; n_ < 4; ++n_) {                            \
                if ((n_ < 2 ? 0 : n_ - 1) != g_) continue;                                \
                const int k2 = n_ >> 1, t2 = n_ & 1;                                      \
                if ((Q) < NQ - 1)                                                         \
                    fx[((Q) + qp_ + 1) & 1][k2][t2] =                                     \
                        ld(base_x[PAR][k2] + ((Q) + 1) * 8192 + t2 * 2048);               \
                else fx[((Q) + qp_ + 1) & 1][k2][t2] = ld(base_x[(PAR) ^ 1][k2] + t2 * 2048); \
            }                                                                             \
            /* last quarter but one: sub-step 0 feature operands of the next step */      \
            if ((Q) == NQ - 2) {                                                          \
                _Pragma("unroll") for (int mt = 0; mt < 8; ++mt) {                        \
                    if ((mt < 2 ? 0 : mt < 6 ? 1 : 2) != g_) continue;                    \
                    fw0[(PAR) ^ 1][mt] = ld(base_w[(PAR) ^ 1][0] + mt * 2048);            \
                }                                                                         \
            }                                                                             \
            __builtin_amdgcn_sched_barrier(0);                                            \
        }                                                                                 \
    }
    // Outstanding fills allowed at the barrier before a quarter.  Quarter q reads token unit
    // q + 1 of its step (the last one unit 0 of the next step), the last two quarters the
    // feature units of the next step; a wave's fills land in order, so what may be outstanding
    // is what was issued behind the youngest of those: the rest of its step's kFills, all of
    // the step after, and this step's fills so far (0, 4, 8, 12 with four quarters; 0, 8, 12
    // with three).
#define PKV_STEP(PAR, ADV)                                                                \
    PKV_QUARTER(PAR, 0, ADV) wait_vm<(NQ == 4 ? 22 : 14)>(); __syncthreads();             \
    PKV_QUARTER(PAR, 1, ADV) wait_vm<16>(); __syncthreads();                              \
    if constexpr (NQ == 4) {                                                              \
        PKV_QUARTER(PAR, 2, ADV) wait_vm<18>(); __syncthreads();                          \
    }                                                                                     \
    PKV_QUARTER(PAR, NQ - 1, ADV) wait_vm<(NQ == 4 ? 20 : 16)>(); __syncthreads();

    for (int t = 0; t < n_T; t += 2) {
        const int adv0 = t + 3 < n_T ? 64 : 0;   // step t fetches step t + 2
        const int adv1 = t + 4 < n_T ? 64 : 0;
        PKV_STEP(0, adv0)
        PKV_STEP(1, adv1)
    }
#undef PKV_STEP
#undef PKV_QUARTER
    wait_vm<0>();                 // the ring's trailing fills must not land in the staging
    acc_settle();

    TileCtx ctx;
    ctx.lane = lane; ctx.wave = wave; ctx.g4 = g4; ctx.l16 = l16; ctx.wt = wt; ctx.wf = wf;
    ctx.split = split; ctx.ft = ft; ctx.mat = mat; ctx.feat0 = feat0; ctx.row0 = row0;
    ctx.heads_out = heads_out; ctx.out = out;
    tile_epilogue<MODE, EXTRA, NQ>(p, acc, ctx, smem);
}

// tile number -> (token tile, feature tile) of a run of n_tok token tiles, kGroup deep
__device__ __forceinline__ void tile_of(int logical, int n_tok, int n_feat, int* tok, int* ft) {
    const int per_group = kGroup * n_feat;
    const int group = logical / per_group;
    const int first_tok = group * kGroup;
    const int rows_in_group = min(kGroup, n_tok - first_tok);
    const int within = logical - group * per_group;
    *tok = first_tok + within % rows_in_group;
    *ft = within / rows_in_group;
}

template <int MODE, bool EXTRA, int NQ>
__global__ __launch_bounds__(256) void proj_slab_kernel(ProjParams p, int n_tok_tiles,
                                                        int n_tiles, int per_xcd) {
    extern __shared__ __align__(16) unsigned char smem[];
    int logical = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (logical >= n_tiles * p.n_ksplit) return;
    const int split = logical / n_tiles;
    int tok, ft;
    tile_of(logical - split * n_tiles, n_tok_tiles, p.tile_begin[3], &tok, &ft);
    slab_tile<MODE, EXTRA, NQ>(p, smem, tok * (64 * NQ), ft, split);
}

// Both heights in one launch: n_hi token tiles of 256 rows, which fill whole rounds of the CUs,
// then n_lo of 192 for the last, partly filled round: the tail ends sooner than with a round of
// full tiles of which a part of the CUs has none.  No splits of the contraction.
template <int MODE, bool EXTRA>
__global__ __launch_bounds__(256) void proj_slab_mix_kernel(ProjParams p, int n_hi, int n_lo,
                                                            int per_xcd_hi, int per_xcd_lo) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int xcd = (int)(blockIdx.x & 7), nth = (int)(blockIdx.x >> 3);
    const int nf = p.tile_begin[3];
    int tok, ft;
    if (nth < per_xcd_hi) {
        const int logical = xcd * per_xcd_hi + nth;
        if (logical >= n_hi * nf) return;
        tile_of(logical, n_hi, nf, &tok, &ft);
        slab_tile<MODE, EXTRA, 4>(p, smem, tok * 256, ft, 0);
    } else {
        const int logical = xcd * per_xcd_lo + nth - per_xcd_hi;
        if (logical >= n_lo * nf) return;
        tile_of(logical, n_lo, nf, &tok, &ft);
        slab_tile<MODE, EXTRA, 3>(p, smem, n_hi * 256 + tok * 192, ft, 0);
    }
}

// adds the splits of the contraction in a fixed order, rotates, rounds once, stores.
// Sixteen lanes per (row, head), four pairs per lane: elements i .. i + 3 and i + 64 .. of the
// head, 16 bytes per load.  The lane works out the sines and cosines of its pairs itself and
// then walks over every gridDim.y-th head slot, so that no table has to be made and read
// (883 rows x 6144 outputs in two splits: 18 us and 5 for the table -> 12; with one
// pair per lane the sums alone moved 3 TB/s).
__global__ __launch_bounds__(256) void proj_splitk_finish_kernel(ProjParams p,
                                                                 const int32_t* __restrict__ row_pos,
                                                                 RopeTable tab) {
    const int f_total = T * p.tile_begin[3];
    const int idx = blockIdx.x * 256 + threadIdx.x;
    const int row = idx >> 4;
    if (row >= p.m) return;                     // a row's lanes leave together
    const int i = (idx & 15) * 4;
    float sn[4], cs[4];
    const double pos = (double)row_pos[row];
#pragma unroll
    for (int e = 0; e < 4; ++e) rope_sincos(pos, tab.inv_freq[i + e], &sn[e], &cs[e]);
    for (int hs = blockIdx.y; hs < f_total / D; hs += gridDim.y) {   // head slot over Q | K | V
        const int ft = hs / 2;
        int mat = 0;
        if (ft >= p.tile_begin[1]) mat = 1;
        if (ft >= p.tile_begin[2]) mat = 2;
        bf16_t* out = p.out[mat];
        if (out == nullptr) continue;
        const int head = (ft - p.tile_begin[mat]) * 2 + (hs & 1);
        const int heads_out = mat == 0 ? p.hq : p.hkv;
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
        const float* src = p.partial + (int64_t)row * f_total + hs * D + i;
#pragma unroll 4
        for (int s = 0; s < p.n_ksplit; ++s) {
            a += *reinterpret_cast<const f32x4*>(src);
            b += *reinterpret_cast<const f32x4*>(src + D / 2);
            src += (int64_t)p.m * f_total;
        }
        if (p.bias[mat]) {
            const bf16x4 ba = *reinterpret_cast<const bf16x4*>(p.bias[mat] + head * D + i);
            const bf16x4 bb = *reinterpret_cast<const bf16x4*>(p.bias[mat] + head * D + i + D / 2);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] += (float)ba[e];
                b[e] += (float)bb[e];
            }
        }
        if (mat != 2 && p.norm_w[mat]) {
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) ss += a[e] * a[e] + b[e] * b[e];
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
            const float r = 1.0f / sqrtf(ss * (1.0f / D) + p.norm_eps);
            const bf16x4 ga = *reinterpret_cast<const bf16x4*>(p.norm_w[mat] + i);
            const bf16x4 gb = *reinterpret_cast<const bf16x4*>(p.norm_w[mat] + i + D / 2);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = a[e] * r * (float)ga[e];
                b[e] = b[e] * r * (float)gb[e];
            }
        }
        bf16x4 va, vb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float ra = mat != 2 ? a[e] * cs[e] - b[e] * sn[e] : a[e];
            const float rb = mat != 2 ? b[e] * cs[e] + a[e] * sn[e] : b[e];
            va[e] = (bf16_t)ra;
            vb[e] = (bf16_t)rb;
        }
        const int64_t orow = (mat != 0 && p.dst_row) ? p.dst_row[row] : row;
        bf16_t* o = out + (orow * heads_out + head) * D + i;
        *reinterpret_cast<bf16x4*>(o) = va;
        *reinterpret_cast<bf16x4*>(o + D / 2) = vb;
    }
}

// the same for the plain and the gated linear layers: one thread per (row, 4 outputs)
template <int MODE>
__global__ __launch_bounds__(256) void linear_splitk_finish_kernel(ProjParams p) {
    const int f_total = T * p.tile_begin[3];
    const int quads = p.n_out / 4;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)p.m * quads) return;
    const int row = (int)(idx / quads);
    const int f = (int)(idx % quads) * 4;
    // column of output f in the tile order of the partials
    const int col = MODE == kProjGated ? (f >> 7) * T + ((f >> 6) & 1) * 128 + (f & 63) : f;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int s = 0; s < p.n_ksplit; ++s) {
        const float* src = p.partial + ((int64_t)s * p.m + row) * f_total + col;
        a += *reinterpret_cast<const f32x4*>(src);
        if (MODE == kProjGated) b += *reinterpret_cast<const f32x4*>(src + 64);
    }
    const int64_t o = (int64_t)row * p.n_out + f;
    bf16x4 v;
    if (MODE == kProjGated) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float ar = (float)(bf16_t)a[e], br = (float)(bf16_t)b[e];
            v[e] = (bf16_t)((float)(bf16_t)silu_f32(ar) * br);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16_t)a[e];
        if (p.residual) {
            const bf16x4 r = *reinterpret_cast<const bf16x4*>(p.residual + o);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (bf16_t)((float)v[e] + (float)r[e]);
        }
    }
    *reinterpret_cast<bf16x4*>(p.out[0] + o) = v;
}

// ---- which tile, how many splits ---------------------------------------------------------
// Four tiles: 64 or 128 tokens x 128 features (gather_qkv_proj_tiles.hip), 192 or 256 tokens x
// 256 features (the slab kernel; contractions that are no multiple of 128 take the 32-wide
// ring).  The large ones have the better rate once the chip is full (8192^3: 1467 TFLOP/s), the
// small ones fill it with fewer rows and without splitting the contraction, whose fp32 partial
// tiles cost a round trip through memory and a second launch.  The choice minimises an estimate
// of the launch time:
//     rounds of the CUs x (fixed + step cost x steps)  against  bytes / 7 TB/s  (+ partials)
// where a partly filled round costs between a full one and its share (the CUs that work clock
// higher).  The constants are fitted to 2661 launches (1024 to 14336 inputs, 1024 to 28672
// outputs, 16 to 6681 rows, 1 to 16 splits; rms error 5 %).  Over those 228 shapes the choice is
// within 1 % of the fastest tile on average and 1.46 x faster than 256 x 256 tiles alone were:
// 64 rows x 4096 x 4096 24 -> 15 us, x 28672 gated 64 -> 45; 512 rows x 4096 x 4096 39 -> 30;
// 1702 rows x 6144 x 4096 84 -> 70; 256 rows x 1536 x 1024 21 -> 8.  The present plan's
// 256-token tile is left only for one that is estimated 5 % faster.
struct TileCost {
    float fixed, step;      // us per tile and per 64 of the contraction
    float part;             // share of a full round that an almost empty one costs
    float overlap;          // how badly the loop and the memory traffic overlap
};
constexpr int kTileTokens[4] = {64, 128, 192, 256};
constexpr TileCost kTileCost[4] = {{0.855f, 0.401f, 0.744f, 0.597f},
                                   {2.217f, 0.512f, 0.759f, 0.378f},
                                   {5.207f, 1.044f, 0.742f, 0.253f},
                                   {6.630f, 1.348f, 0.721f, 0.179f}};

struct TilePlan {
    int tokens, ksplit;   // tokens 256 with n_hi > 0: that many tiles of 256, the rest of 192
    int n_hi;
};

// features of a launch x splits of its contraction that the fp32 partials have room for
// (256 tiles' worth of 256 x 256; nothing for launches of more than 128 token tiles)
int64_t partial_features(int64_t m) {
    const int64_t n_tok_tiles = ceil_div(m, T);
    return n_tok_tiles > 128 ? 0 : (int64_t)T * 256 / n_tok_tiles;
}

float estimate_us(int kind, int64_t m, int64_t features, int64_t k_in, int ks) {
    const TileCost& c = kTileCost[kind];
    const int64_t tiles =
        ceil_div(m, kTileTokens[kind]) * (features / (kind < 2 ? 128 : 256)) * ks;
    const float steps = (float)k_in / (64.f * ks);
    const float r = (float)tiles / 256.f;
    const float full = (float)(tiles / 256), up = (float)ceil_div(tiles, 256);
    float loop;
    if (kind == 0) {
        // two workgroups share a CU: a second tile costs 0.84 of a first one's steps
        const float more = r <= 1.f ? 0.f : 0.564f * (up - 1.f) + 0.436f * (r - 1.f);
        const float rounds = r <= 1.f ? c.part + (1.f - c.part) * r : 1.f + 0.844f * more;
        loop = c.step * steps * rounds + c.fixed * (1.f + 0.603f * more);
    } else {
        const float rounds = full + (up > full ? c.part + (1.f - c.part) * (r - full) : 0.f);
        loop = c.step * steps * rounds + c.fixed * up;
    }
    const float mb = 2e-6f * ((float)features * k_in + (float)m * k_in + (float)m * features);
    const float mem = mb / 7.094f;
    const float hi = loop > mem ? loop : mem, lo = loop > mem ? mem : loop;
    float t = 1.671f + hi + c.overlap * lo * lo / hi;
    if (ks > 1) t += 3.956f + 8e-6f * (float)ks * (float)m * (float)features / 6.419f;
    return t;
}

// `rounds` full rounds of 256-token tiles and `left` 192-token tiles behind them
float estimate_mix_us(int64_t m, int64_t features, int64_t k_in, int64_t rounds, int64_t left) {
    const TileCost &h = kTileCost[3], &l = kTileCost[2];
    const float steps = (float)k_in / 64.f;
    float loop = (float)rounds * (h.step * steps + h.fixed);
    if (left > 0) {
        const float full = (float)(left / 256), up = (float)ceil_div(left, 256);
        const float part = up > full ? l.part + (1.f - l.part) * ((float)left / 256.f - full) : 0.f;
        loop += l.step * steps * (full + part) + l.fixed * up;
    }
    const float mem =
        2e-6f * ((float)features * k_in + (float)m * k_in + (float)m * features) / 7.094f;
    const float hi = loop > mem ? loop : mem, lo = loop > mem ? mem : loop;
    return 1.671f + hi + h.overlap * lo * lo / hi;
}

// what 256 x 256 tiles take: the largest power of two that keeps the launch within 256
// workgroups and a split >= NS stages
int plan_ksplit(int64_t n_tiles, int n_k) {
    int ks = 1;
    while (ks < 16 && n_tiles * (ks * 2) <= 256 && n_k % (ks * 2) == 0 && n_k / (ks * 2) >= NS)
        ks *= 2;
    return ks;
}

TilePlan plan_tiles(int64_t m, int64_t features, int64_t k_in) {
    const int64_t n_tiles = ceil_div(m, T) * (features / T);
    TilePlan best = {256, plan_ksplit(n_tiles, (int)(k_in / BK)), 0};
    const float now = estimate_us(3, m, features, k_in, best.ksplit);
    float t_best = 0.95f * now;
    const int64_t room = partial_features(m);
    for (int kind = n_tiles <= 2048 ? 0 : 2; kind < 4; ++kind)
        for (int ks = 1; ks <= 16; ks *= 2) {
            if (ks > 1 && ks * features > room) break;
            if (k_in < 256 * ks || k_in % ((kind < 2 ? 64 : 128) * ks)) break;
            const float t = estimate_us(kind, m, features, k_in, ks);
            if (t < t_best) {
                t_best = t;
                best.tokens = kTileTokens[kind];
                best.ksplit = ks;
            }
        }
    // whole rounds of 256-token tiles, what is left of the rows on 192-token ones
    const int64_t nf = features / T;
    const int64_t rounds = n_tiles / 256, hi = 256 * rounds / nf;
    if (rounds >= 1 && n_tiles % 256 != 0 && hi >= 1 && k_in % 128 == 0) {
        const int64_t left = ceil_div(m - hi * T, 192) * nf - (256 * rounds - hi * nf);
        const float t = estimate_mix_us(m, features, k_in, rounds, left);
        if (t < 0.97f * (best.tokens == 256 ? now : t_best)) {
            best.tokens = 256;
            best.ksplit = 1;
            best.n_hi = (int)hi;
        }
    }
    return best;
}

}  // namespace

size_t proj_dma128_partial_bytes(const pkv_layer_cfg& cfg, int64_t m) {
    (void)cfg;
    return (size_t)m * (size_t)partial_features(m) * sizeof(float);
}

bool proj_dma128_supported(const pkv_layer_cfg& cfg, int64_t m) {
    return cfg.dtype == PKV_BF16 && cfg.head_dim == D && cfg.hidden % BK == 0 &&
           cfg.hidden / BK >= NS && cfg.n_q_heads % 2 == 0 && cfg.n_kv_heads % 2 == 0 &&
           m > 0 && m < (1 << 30);
}

namespace {

// row_pos, tab: the angles of a Q | K | V launch (p.cs: room for their table, or the table)
template <int MODE, bool EXTRA = false>
pkv_status launch_tiles(const ProjParams& p, const int32_t* row_pos, const RopeTable& tab,
                        hipStream_t st, bool angles_ready = false) {
    static std::atomic<bool> configured{false};   // set twice at worst: the calls are idempotent
    if (!configured.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(proj_dma_kernel<MODE, EXTRA>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(proj_slab_kernel<MODE, EXTRA, 4>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kSlabLdsBytes<4>) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(proj_slab_mix_kernel<MODE, EXTRA>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kSlabLdsBytes<4>) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(proj_slab_kernel<MODE, EXTRA, 3>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kSlabLdsBytes<3>) != hipSuccess)
            return PKV_ERR_LAUNCH;
        configured.store(true, std::memory_order_release);
    }
    if (p.tile_begin[3] == 0) return PKV_OK;
    if (ceil_div(p.m, T) * p.tile_begin[3] > (1 << 29)) return PKV_ERR_SHAPE;
    const TilePlan plan = plan_tiles(p.m, (int64_t)p.tile_begin[3] * T, p.hid);
    ProjParams q = p;
    q.n_ksplit = plan.ksplit;
    if (q.n_ksplit > 1 && q.partial == nullptr) return PKV_ERR_WORKSPACE;
    // a split launch's finishing kernel works the angles out by itself
    if (MODE == kProjRope && q.n_ksplit == 1 && !angles_ready)
        launch_rope_table(row_pos, p.m, D / 2, tab, const_cast<float2*>(p.cs), st);
    if (plan.tokens < 192) {
        const pkv_status rc = launch_proj_small<MODE, EXTRA>(plan.tokens, q, st);
        if (rc != PKV_OK) return rc;
    } else {
        const int n_tok_tiles = (int)ceil_div(p.m, plan.tokens);
        const int n_tiles = n_tok_tiles * p.tile_begin[3];
        const int per_xcd = (int)ceil_div((int64_t)n_tiles * q.n_ksplit, 8);
        const dim3 grid((unsigned)(per_xcd * 8)), block(256);
        // contraction in slabs of 64 when every split has an even number of them
        if (plan.n_hi > 0) {
            const int n_lo = (int)ceil_div(p.m - plan.n_hi * T, 192);
            const int px_hi = (int)ceil_div((int64_t)plan.n_hi * p.tile_begin[3], 8);
            const int px_lo = (int)ceil_div((int64_t)n_lo * p.tile_begin[3], 8);
            hipLaunchKernelGGL((proj_slab_mix_kernel<MODE, EXTRA>),
                               dim3((unsigned)(8 * (px_hi + px_lo))), block, kSlabLdsBytes<4>, st,
                               q, plan.n_hi, n_lo, px_hi, px_lo);
        } else if (plan.tokens == 192)
            hipLaunchKernelGGL((proj_slab_kernel<MODE, EXTRA, 3>), grid, block, kSlabLdsBytes<3>,
                               st, q, n_tok_tiles, n_tiles, per_xcd);
        else if (p.hid % (128 * q.n_ksplit) == 0)
            hipLaunchKernelGGL((proj_slab_kernel<MODE, EXTRA, 4>), grid, block, kSlabLdsBytes<4>,
                               st, q, n_tok_tiles, n_tiles, per_xcd);
        else
            hipLaunchKernelGGL((proj_dma_kernel<MODE, EXTRA>), grid, block, kLdsBytes, st, q,
                               n_tok_tiles, n_tiles, per_xcd);
    }
    if (q.n_ksplit > 1) {
        if (MODE == kProjRope) {
            // enough workgroups to hide the loads, as few head groups as that allows
            const int64_t blocks = ceil_div((int64_t)p.m * 16, 256);
            const int64_t heads = 2 * p.tile_begin[3];
            int64_t groups = ceil_div(1024, blocks);
            if (groups > heads) groups = heads;
            hipLaunchKernelGGL(proj_splitk_finish_kernel,
                               dim3((unsigned)blocks, (unsigned)groups), dim3(256), 0, st, q,
                               row_pos, tab);
        } else {
            const int64_t total = (int64_t)p.m * (p.n_out / 4);
            hipLaunchKernelGGL(linear_splitk_finish_kernel<MODE>,
                               dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, st, q);
        }
    }
    return launch_status();
}

}  // namespace

bool proj_dma128_reads_angles(int64_t m, int64_t features, int64_t k_in) {
    return features > 0 && plan_tiles(m, features, k_in).ksplit == 1;
}

pkv_status launch_proj_dma128(const ProjParams& p, const int32_t* row_pos, const RopeTable& tab,
                              hipStream_t st, bool angles_ready) {
    const bool extra = p.bias[0] || p.bias[1] || p.bias[2] || p.norm_w[0] || p.norm_w[1] ||
                       p.dst_row;
    return extra ? launch_tiles<kProjRope, true>(p, row_pos, tab, st, angles_ready)
                 : launch_tiles<kProjRope, false>(p, row_pos, tab, st, angles_ready);
}

bool linear_dma_supported(int mode, int64_t m, int64_t k_in, int64_t n_out) {
    const int64_t per_tile = mode == kProjGated ? T / 2 : T;
    return m > 0 && m < (1 << 30) && k_in % BK == 0 && k_in / BK >= NS && k_in < (1 << 30) &&
           n_out > 0 && n_out % per_tile == 0 && n_out < (1 << 30);
}

size_t linear_dma_partial_bytes(int64_t m) {
    return m <= 0 ? 0 : (size_t)m * (size_t)partial_features(m) * sizeof(float);
}

pkv_status launch_linear_dma(int mode, const bf16_t* x, const bf16_t* w0, const bf16_t* w1,
                             const bf16_t* residual, bf16_t* y, int64_t m, int64_t k_in,
                             int64_t n_out, float* partial, hipStream_t st) {
    ProjParams p = {};
    p.hidden = x;
    p.row_idx = nullptr;
    p.w[0] = w0;
    p.w[1] = w1;
    p.out[0] = y;
    p.cs = nullptr;
    p.m = (int)m;
    p.hid = (int)k_in;
    const int nft = (int)(n_out / (mode == kProjGated ? T / 2 : T));
    p.tile_begin[0] = 0;
    p.tile_begin[1] = p.tile_begin[2] = p.tile_begin[3] = nft;
    p.partial = partial;
    p.n_ksplit = 1;
    p.residual = residual;
    p.n_out = (int)n_out;
    return mode == kProjGated ? launch_tiles<kProjGated>(p, nullptr, RopeTable{}, st)
                              : launch_tiles<kProjPlain>(p, nullptr, RopeTable{}, st);
}

}  // namespace pkv
