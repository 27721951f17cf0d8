// Step 5, head_dim 128, bf16, for contexts of a few thousand keys and the rows selected from them: up to
// two and a half jobs of 128 columns per CU, from a fifth of one on where the keys are few.
// (Paper: Sec. 4.3 Stage II - complete recomputation, but only for the selected
// tokens; Sec. 5.3 - this attention over the long cache dominates the cost.)
//
// Arithmetic, operand layouts and the three-deep pipeline of a sub-step of 32 keys are those of
// attn_w8_kernel (sparse_row_attn_w8.hip).  There a workgroup owns 256 (row, head) columns, and a
// launch with so few rows that some jobs would outlast the others cuts the keys into ranges, whose
// fp32 partial results go through memory to a merge launch; with more jobs than CUs it also needs a
// queue, and a launch that clears its counters: 15 us beside 60 to 130 of arithmetic.  Here a job
// is 128 columns, as in attn_short_kernel: its two groups of four waves take every other block of 32
// keys and meet in LDS.  Jobs are half as long without a partial result in memory, and the hardware
// deals them out, heavier ones first: one launch.
//
// Whole call, ranges and queue -> this (us; rows spread over the keys): 637 rows over 4k keys, 40 / 8
// heads, 63 -> 58, 870 over 4k 80 -> 62; 32 / 8 heads, 900 over 2k 47 -> 40, 1400 over 3.5k 80 -> 59,
// 1702 over 8k 135 -> 129, 2200 over 8k 191 -> 167; the rule is with attn_pair_applies.
//
// A group has rings of its own: four stages of 8 KB for keys and four for values, 128 KB for both.  At
// its sub-step u the keys of u + 6 and the values of u + 3 are requested into the stages that u - 1
// read, and one barrier per sub-step keeps the waves that far apart.
#include <algorithm>
#include <atomic>

#include "attn_common.h"
#include "attn_tile.h"

namespace pkv {

namespace {

constexpr int D = 128;
constexpr int KC = D / 16;             // contraction chunks of S^T
constexpr int DB = D / 32;             // 32-row blocks of O^T
constexpr int kSub = 32;               // keys of a sub-step
constexpr int kStage = kSub * D * 2;   // 8 KB: 32 keys of K or V
constexpr int kCols = 128;             // columns of a workgroup
constexpr int G = 2;                   // groups of four waves that share the keys
constexpr int kThreads = G * 256;
constexpr int kRing = 8 * kStage;      // a group's four stages of keys and four of values
constexpr int kLdsBytes = G * kRing;

__global__ __launch_bounds__(kThreads, 2) void attn_pair_kernel(AttnParams p) {
    extern __shared__ __align__(16) unsigned char smem_all[];
    __shared__ int s_red[4 * G];
    __shared__ float s_ml[2][kCols];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave_all >> 2, wave = wave_all & 3;   // group, wave in it
    unsigned char* const smem = smem_all + half * kRing;
    const int hh = lane >> 5;
    const int l32 = lane & 31;

    // one (kv head, row tile) job per workgroup, the heavier ones first; the kv head is the fastest
    // index, so that with eight of them a head's K/V stays in one XCD's L2
    const int g = (int)(blockIdx.x % p.hkv);
    const int tile = p.n_tiles - 1 - (int)(blockIdx.x / p.hkv);

    // ---- global -> LDS: wave w fills rows 8 w .. + 8 of every stage, two instructions ------------
    // Key row r of a stage at byte r*256, 16-byte chunk c at c ^ (r & 15); value row r likewise at
    // c ^ (4 (r & 3)).
    const uint32_t row_bytes = (uint32_t)p.hkv * D * 2;
    uint32_t voff_k[2], voff_v[2], kofs_last[2], vofs_last[2];
    {
        const int last = (p.n_keys - 1) % kSub;   // last row of the (possibly ragged) last block
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 8 * wave + 4 * i + (lane >> 4);
            const uint32_t chunk = (uint32_t)(((lane & 15) ^ (r & 15)) * 16);
            const uint32_t vchunk = (uint32_t)(((lane & 15) ^ (4 * (r & 3))) * 16);
            voff_k[i] = (uint32_t)r * row_bytes + chunk;
            voff_v[i] = (uint32_t)r * row_bytes + vchunk;
            kofs_last[i] = (uint32_t)min(r, last) * row_bytes + chunk;
            vofs_last[i] = (uint32_t)min(r, last) * row_bytes + vchunk;
        }
    }
    const uint32_t lds_wave =
        __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * 8 * 256);
    const bf16_t* const k_head = p.k + g * D;
    const bf16_t* const v_head = p.v + g * D;
    // the group's block U of the keys or values (clamped to the last one) into its stage
    int last_block = (p.n_keys - 1) / kSub;
#define PAIR_DMA_K(U, STAGE)                                                             \
    {                                                                                    \
        const int u_ = min((U) * G + half, last_block);                                  \
        const bf16_t* gb_ = k_head + (int64_t)u_ * kSub * p.hkv * D;                     \
        const bool full_ = u_ * kSub + kSub <= p.n_keys;   /* wave-uniform */            \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                    \
            dma16(gb_, full_ ? voff_k[i] : kofs_last[i],                                 \
                  lds_wave + (STAGE) * kStage + i * 1024);                               \
    }
#define PAIR_DMA_V(U, STAGE)                                                             \
    {                                                                                    \
        const int u_ = min((U) * G + half, last_block);                                  \
        const bf16_t* gb_ = v_head + (int64_t)u_ * kSub * p.hkv * D;                     \
        const bool full_ = u_ * kSub + kSub <= p.n_keys;                                 \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                    \
            dma16(gb_, full_ ? voff_v[i] : vofs_last[i],                                 \
                  lds_wave + (4 + (STAGE)) * kStage + i * 1024);                         \
    }
#define PAIR_DMA_FIRST                                                                   \
    PAIR_DMA_K(0, 0) PAIR_DMA_K(1, 1) PAIR_DMA_K(2, 2) PAIR_DMA_K(3, 3) PAIR_DMA_V(0, 0)
    PAIR_DMA_FIRST   // in bounds whatever the rows see

    // ---- this lane's column ---------------------------------------------------------------
    const int col = wave * 32 + l32;
    const int rl = col / p.group;
    const int row = tile * p.bm + rl;
    const int head = g * p.group + col % p.group;
    const bool valid = rl < p.bm && row < p.m;
    const int limit = valid ? min(p.row_pos[row], p.n_keys - 1) : -1;   // last key it sees
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
    if (lane == 0) s_red[wave_all] = lmax;
    wait_vm<0>();
    __syncthreads();
    int tile_max = -1;
#pragma unroll
    for (int w = 0; w < 4; ++w) tile_max = max(tile_max, s_red[w]);   // (the groups' are alike)
    // blocks of this job, and of a group (the second's last one may be one too many: masked)
    const int n_sub = __builtin_amdgcn_readfirstlane((tile_max + kSub) / kSub);
    if (n_sub <= 0) return;   // block-uniform: no valid row
    last_block = n_sub - 1;   // nothing behind it is asked for any more
    const int n_grp = (n_sub + G - 1) / G;
    // the group's blocks [0, u_unm) lie entirely at or below every limit of this wave; a wave
    // without a valid column has nothing to mask
    const int u_unm = __builtin_amdgcn_readfirstlane(
        lmin == 0x7fffffff ? 0x3fffffff : ((lmin + 1) / kSub - half + G - 1) / G);

    // ---- LDS -> register operand addresses (sparse_row_attn_w8.hip) -------------------------------
    const int prow = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
    uint32_t kaddr[KC], vaddr[4];
    {
        const uint32_t a0 = prow * 256 + (((prow & 15) ^ hh) * 16);
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kaddr[kc] = a0 ^ (kc << 5);
        const int e = (lane >> 2) & 3, j = lane & 3, gh = (lane >> 4) & 1;
#pragma unroll
        for (int db = 0; db < 4; ++db)
            vaddr[db] = (uint32_t)(4 * kStage + (8 * hh + e) * 256 +
                                   (((db ^ e) * 4 + gh * 2 + (j >> 1)) * 16) + (j & 1) * 8);
    }
    const float c2 = p.scale_log2;

    float m_run = -INFINITY, l_run;
    f32x16 o_acc[DB];
    f32x16 s_a, s_b;          // S^T of even / odd sub-steps
    bf16x8 pb_a[2], pb_b[2];  // P^T of even / odd sub-steps: [16-key half]
    bf16x8 ka[KC], va[2][DB];
    float rs;                 // this lane's sum of the probabilities being produced
    float msc;                // reference maximum times c2 (0 while it is -inf)
    constexpr float kGrow = 1.0e24f;   // ~2^80
    float rs_max;
    float e_half;
    float x_next;

#define PAIR_LOAD_KA1(ST, KCI)                                                           \
    ka[KCI] = *reinterpret_cast<const bf16x8*>(smem + (ST) * kStage + kaddr[KCI]);
#define PAIR_LOAD_KA(ST)                                                                 \
    _Pragma("unroll") for (int kc = 0; kc < KC; ++kc) { PAIR_LOAD_KA1(ST, kc) }
#define PAIR_LOAD_VA1(ST, KK, DBI)                                                       \
    {                                                                                    \
        const unsigned char* a_ = smem + (ST) * kStage + 16 * (KK) * 256 + vaddr[DBI];   \
        const bf16x4 lo_ = lds_read_tr(a_), hi_ = lds_read_tr(a_ + 4 * 256);             \
        va[KK][DBI] = __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7);         \
    }

    // exponent of element R of score buffer S whose first key is T0
#define PAIR_SM_PREP(S, R, T0, MASK)                                                     \
    {                                                                                    \
        float x_ = S[R];                                                                 \
        if (MASK) {                                                                      \
            const int key_ = (T0) + 16 * ((R) / 8) + 8 * hh + (R) % 8;                   \
            if (key_ > limit) x_ = -INFINITY;                                            \
        }                                                                                \
        x_next = x_ * c2 - msc;                                                          \
    }
    // probability of element R (exponent prepared one step earlier) into PB; prepares the
    // exponent of element RN of SN (first key T0N) in between
#define PAIR_SM_STEP(PB, R, SN, RN, T0N, MASK)                                           \
    {                                                                                    \
        const float e_ = __builtin_amdgcn_exp2f(x_next);                                 \
        PAIR_SM_PREP(SN, RN, T0N, MASK)                                                  \
        rs += e_;                                                                        \
        if ((R) % 2 == 0) {                                                              \
            e_half = e_;                                                                 \
            asm volatile("" : "+v"(rs), "+v"(e_half), "+v"(x_next));                     \
        } else {                                                                         \
            PB[(R) / 8][(R) % 8 - 1] = (bf16_t)e_half;                                   \
            PB[(R) / 8][(R) % 8] = (bf16_t)e_;                                           \
            asm volatile("" : "+v"(rs), "+v"(PB[(R) / 8]), "+v"(x_next));                \
        }                                                                                \
    }

    // One sub-step U.  SCUR = S^T(u+1) (complete), SNXT receives S^T(u+2) from the operands in ka;
    // PCUR = P(u) (complete), PNXT receives P(u+1).  ST = u mod 4: the values of u are read from
    // that stage and the keys of u + 3 from the one before it, which the barrier then frees.
#define PAIR_SUBSTEP(SCUR, SNXT, PCUR, PNXT, U, ST, MASK)                                \
    {                                                                                    \
        const int t0n_ = (((U) + 1) * G + half) * kSub;                                  \
        __builtin_amdgcn_sched_barrier(0);                                               \
        PAIR_DMA_K((U) + 6, ((ST) + 2) & 3)                                              \
        __builtin_amdgcn_sched_barrier(0);                                               \
        _Pragma("unroll") for (int i_ = 0; i_ < 8; ++i_) {                               \
            const f32x16 z_ = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,                   \
                               0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};                  \
            SNXT = mfma32(ka[i_], qreg[i_], i_ == 0 ? z_ : SNXT);                        \
            PAIR_LOAD_VA1(ST, i_ >> 2, i_ & 3)                                           \
            PAIR_SM_STEP(PNXT, i_, SCUR, i_ + 1, t0n_, MASK)                             \
            __builtin_amdgcn_sched_barrier(0);                                           \
        }                                                                                \
        PAIR_DMA_V((U) + 3, ((ST) + 3) & 3)                                              \
        __builtin_amdgcn_sched_barrier(0);                                               \
        _Pragma("unroll") for (int i_ = 0; i_ < 8; ++i_) {                               \
            const int kk_ = i_ >> 2, db_ = i_ & 3;                                       \
            mfma32_acc(va[kk_][db_], PCUR[kk_], o_acc[db_]);                             \
            PAIR_LOAD_KA1(((ST) + 3) & 3, i_)                                            \
            if (i_ < 7) { PAIR_SM_STEP(PNXT, 8 + i_, SCUR, 9 + i_, t0n_, MASK) }         \
            else { PAIR_SM_STEP(PNXT, 15, SNXT, 0, t0n_ + G * kSub, MASK) }              \
            __builtin_amdgcn_sched_barrier(0);                                           \
        }                                                                                \
        l_run += rs;                                                                     \
        rs_max = fmaxf(rs_max, rs);                                                      \
        rs = 0.f;                                                                        \
        wait_vm<8>();   /* K(u+4), V(u+1) have landed; the 8 newest loads stay in flight */ \
        __syncthreads();                                                                 \
    }

    // Two attempts at most, as in attn_w8_kernel: the softmax reference of a column is the maximum of
    // its first 32 keys; where the sums leave the safe range the workgroup finds the true maxima of
    // its columns and goes over its keys once more with those.
    bool exact = false;
    float l_tot;
    for (;;) {
        l_run = rs = rs_max = e_half = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o_acc[db][r] = 0.f;
        // ---- prologue -------------------------------------------------------------------------
        if (exact) {
            PAIR_DMA_FIRST
            wait_vm<0>();
            __syncthreads();
        }
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                             0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        PAIR_LOAD_KA(0)
        s_a = mfma32(ka[0], qreg[0], zero);
#pragma unroll
        for (int kc = 1; kc < KC; ++kc) s_a = mfma32(ka[kc], qreg[kc], s_a);
        PAIR_LOAD_KA(1)
        s_b = mfma32(ka[0], qreg[0], zero);
#pragma unroll
        for (int kc = 1; kc < KC; ++kc) s_b = mfma32(ka[kc], qreg[kc], s_b);
        PAIR_LOAD_KA(2)            // operands of S^T(2)
        if (!exact) {
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = half * kSub + 16 * (r / 8) + 8 * hh + (r % 8);
                if (key <= limit) mx = fmaxf(mx, s_a[r]);
            }
            m_run = fmaxf(mx, __shfl_xor(mx, 32, 64));
        }
        msc = (m_run == -INFINITY ? 0.f : m_run) * c2;
        // P(0) in full
        const int t0 = half * kSub;
        PAIR_SM_PREP(s_a, 0, t0, true)
#pragma unroll
        for (int r = 0; r < 15; ++r) PAIR_SM_STEP(pb_a, r, s_a, r + 1, t0, true)
        PAIR_SM_STEP(pb_a, 15, s_b, 0, t0 + G * kSub, true)
        l_run += rs;
        rs_max = fmaxf(rs_max, rs);
        rs = 0.f;
        // the keys of blocks 4 to 6 go where those of 0 to 2 are: every wave must be done reading
        __syncthreads();
        // what sub-steps -2 and -1 would have requested, in their order
        PAIR_DMA_K(4, 0)
        PAIR_DMA_V(1, 1)
        PAIR_DMA_K(5, 1)
        PAIR_DMA_V(2, 2)

        // ---- main loop: four sub-steps per trip so that every LDS stage is a constant ----------------
        // sub-step u is mask free when every score it turns into a probability (of block u + 1 and
        // the first of u + 2) lies at or below every limit of the wave
        const int n_loop = (n_grp + 1) & ~1;   // (what is one too many has probability 0)
        const int n_unm = min(n_loop, max(0, u_unm - 2)) & ~3;
        int u = 0;
        for (; u < n_unm; u += 4) {
            PAIR_SUBSTEP(s_b, s_a, pb_a, pb_b, u, 0, false)
            PAIR_SUBSTEP(s_a, s_b, pb_b, pb_a, u + 1, 1, false)
            PAIR_SUBSTEP(s_b, s_a, pb_a, pb_b, u + 2, 2, false)
            PAIR_SUBSTEP(s_a, s_b, pb_b, pb_a, u + 3, 3, false)
        }
        for (; u < n_loop; u += 2) {
            const int st = u & 3;
            PAIR_SUBSTEP(s_b, s_a, pb_a, pb_b, u, st, true)
            PAIR_SUBSTEP(s_a, s_b, pb_b, pb_a, u + 1, st + 1, true)
        }
        wait_vm<0>();   // nothing may still be writing LDS when the workgroup moves on
        // the last O^T MFMAs were issued behind the compiler's back: let them retire before the
        // accumulators are read (which the statements behind the wait keep behind it)
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
        for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(o_acc[db]));

        l_tot = l_run + __shfl_xor(l_run, 32, 64);
        const bool bad = !(rs_max < kGrow) || !(l_tot < 3.0e38f);
        const int wave_bad = __any(bad) ? 1 : 0;   // over all lanes, before the branch
        __syncthreads();                       // s_red held the tile limits so far
        if (lane == 0) s_red[wave_all] = wave_bad;
        __syncthreads();
        int marked = 0;
#pragma unroll
        for (int w = 0; w < 4 * G; ++w) marked |= s_red[w];
        if (exact || !marked) break;           // block-uniform
        exact = true;
        float mx = -INFINITY;
        for (int t = 0; t < n_grp; ++t) {
            __syncthreads();      // nobody reads the stage that is about to be filled
            PAIR_DMA_K(t, 0)
            wait_vm<0>();
            __syncthreads();
            PAIR_LOAD_KA(0)
            f32x16 s = zero;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) s = mfma32(ka[kc], qreg[kc], s);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((t * G + half) * kSub + 16 * (r / 8) + 8 * hh + (r % 8) <= limit)
                    mx = fmaxf(mx, s[r]);
        }
        m_run = fmaxf(mx, __shfl_xor(mx, 32, 64));
        __syncthreads();
    }

#undef PAIR_DMA_K
#undef PAIR_DMA_V
#undef PAIR_DMA_FIRST
#undef PAIR_LOAD_KA
#undef PAIR_LOAD_KA1
#undef PAIR_LOAD_VA1
#undef PAIR_SM_PREP
#undef PAIR_SM_STEP
#undef PAIR_SUBSTEP

    // ---- epilogue ------------------------------------------------------------------------------
    // the groups meet in LDS, where the rings were
    float* const ex = reinterpret_cast<float*>(smem_all) + wave * (DB * 16 * 64) + lane;
    __syncthreads();
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
    if (half == 1 || !valid) return;
    const float m1 = s_ml[0][col], m = fmaxf(m_run, m1);   // finite: the row sees a key
    const float w0 = __builtin_amdgcn_exp2f((m_run - m) * c2);
    const float w1 = __builtin_amdgcn_exp2f((m1 - m) * c2);
    l_tot = l_tot * w0 + s_ml[1][col] * w1;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            o_acc[db][r] = o_acc[db][r] * w0 + ex[(db * 16 + r) * 64] * w1;
    const float inv = 1.f / l_tot;
    const int64_t colg = (int64_t)row * p.hq + head;
    bf16_t* op = p.out + colg * D + 4 * hh;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (bf16_t)(o_acc[db][4 * r4 + e] * inv);
            *reinterpret_cast<bf16x4*>(op + db * 32 + r4 * 8) = v;
        }
    if (hh == 0 && p.lse) p.lse[colg] = m * p.scale + logf(l_tot);
}

}  // namespace

// Against ranges and queue at 400 sizes, heads 8 / 1 to 96 / 8, each with rows spread over the
// keys, as a selection has them, and with all rows at the end of the cache (us, spread / end).
// Up to one job per CU: the launch lasts as long as its longest job, 0.6 us per 64 keys and 15
// besides, so jobs have to be many or short: n_keys <= 20 jobs (40 / 8, 56 jobs over 1118 keys
// 24 -> 20 / 27 -> 21, 32 / 8, 192 over 3411 50 -> 44 / 57 -> 49; 256 over 8k 93 -> 96).
// Up to two and a half: a CU's later, lighter jobs fill up what its first one leaves (40 / 8, 280
// jobs over 2.3k 51 -> 36 / 51 -> 58, 32 / 8, 448 over 4.8k 102 -> 80 / 120 -> 122, 600 over 10k
// 235 -> 216 / 400 -> 369); beyond, the wider tiles read the keys less often (832 over 8k: 205 -> 221), and
// beyond 12k keys the two are level (1702 rows over 16.5k: 220 and 224).  Rows at the end, all
// of one weight, lose where one more job per CU is begun for a few of them, so the gain with
// spread rows has to be worth it.  It is not
// - for a third job per CU where the wide tiles are one per CU (40 / 8, 520 over 4.8k 105 -> 100
//   / 130 -> 172; 96 / 8, 536 over 10.7k 201 -> 199 / 336 -> 418),
// - for groups that leave more than a twentieth of the 128 columns empty (96 / 8, 264 over 4k 57
//   -> 54 / 75 -> 108, 400 over 1.1k 32 -> 32 / 34 -> 39),
// - for large groups, whose jobs have few rows, over few keys (64 / 8, 480 over 1.1k 35 -> 37 /
//   35 -> 37).
bool attn_pair_applies(const pkv_layer_cfg& cfg, int64_t n_keys, int64_t m) {
    const int group = cfg.n_q_heads / cfg.n_kv_heads;
    if (group > kCols || n_keys > 12288) return false;
    const int rows = kCols / group;
    const int64_t jobs = ceil_div(m, rows) * cfg.n_kv_heads;
    if (jobs <= kPlanCus) return n_keys <= 20 * jobs;
    const int64_t wide = ceil_div(m, 2 * kCols / group) * cfg.n_kv_heads;
    return 2 * jobs <= 5 * kPlanCus && !(jobs > 2 * kPlanCus && wide <= kPlanCus) &&
           20 * rows * group >= 19 * kCols &&
           (group <= 5 || 2 * jobs <= 3 * kPlanCus || n_keys >= 1536);
}

pkv_status launch_attn_pair(AttnParams p, hipStream_t st) {
    static std::atomic<bool> configured{false};   // set twice at worst: the calls are idempotent
    if (!configured.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(attn_pair_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLdsBytes) != hipSuccess)
            return PKV_ERR_LAUNCH;
        configured.store(true, std::memory_order_release);
    }
    p.bm = kCols / p.group;
    p.n_tiles = (int)ceil_div(p.m, p.bm);
    hipLaunchKernelGGL(attn_pair_kernel, dim3((unsigned)(p.n_tiles * p.hkv)), dim3(kThreads),
                       kLdsBytes, st, p);
    return launch_status();
}

}  // namespace pkv
