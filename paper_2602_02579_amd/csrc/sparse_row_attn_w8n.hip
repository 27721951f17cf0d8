// Step 5, head_dim 128, bf16, eight waves per workgroup, for launches with more jobs than CUs.
// (Paper: Sec. 4.3 Stage II - complete recomputation, but only for the selected
// tokens; Sec. 5.3 - this attention over the long cache dominates the cost.)
//
// The job, its columns, the LDS ring, the three-deep pipeline and the second attempt are those
// of attn_w8_kernel (sparse_row_attn_w8.hip).  What differs is the matrix instruction,
// v_mfma_f32_16x16x32_bf16 instead of 32x32x16, and with it the register layouts and the
// instruction order.
//
// Why: a launch that keeps every CU busy is held by the power limit, and the smaller tile moves
// half the accumulator bytes per product through the register file (in registers alone, Gaussian
// operands, 256 CUs sustain 2044 against 1757 TFLOP/s).  It also takes twice the issue slots:
// an MFMA occupies its wave's vector issue for 8 clocks whichever its size, so per 32 clocks of
// matrix work 16 instead of 24 are left for the 18 of the softmax.  The change therefore pays
// only under the power limit, and only with the softmax arithmetic laid out by hand between
// the two MFMAs of a pair: a wave that reaches the second one while the pipe is busy issues
// nothing else.  6681 rows over 32k keys, whole call: 32x32x16 1513 us (72.5 % of the matrix
// pipe at ~1.64 GHz); 16x16x32 in the compiler's order 1522 us (61 %); laid out 1455 us (65
// to 68 % at ~1.9 GHz).  1766 rows over 16k 260 -> 249 us, 26470 over 131k 21.9 -> 21.2 ms.  With one
// job per CU, where the clock is not limited, it is the slower one (637 rows over 4k keys
// in one range 84 -> 92 us): those launches keep attn_w8_kernel.
//
// Two instantiations: <false> reads V^T tiles from a transposed copy of the value cache
// that a pre-pass makes; <true> fills LDS with the value rows as the cache holds them and
// transposes them on the way out (ds_read_b64_tr_b16).  The launcher picks by problem size.
#include <algorithm>
#include <atomic>

#include "attn_common.h"
#include "attn_tile.h"

namespace pkv {

namespace {

constexpr int D = 128;
constexpr int KC = D / 32;             // contraction chunks of S^T
constexpr int DB = D / 16;             // 16-row blocks of O^T
constexpr int NS = 4;                  // LDS stages per operand
constexpr int NW = 8;                  // waves per workgroup
constexpr int kThreads = NW * 64;
constexpr int kStageK = kBN * D * 2;   // bytes: 64 keys x 256 B
constexpr int kStageV = D * kBN * 2;   // bytes: 128 d-rows x 128 B
constexpr int kLdsBytes = NS * (kStageK + kStageV);
constexpr int kStealLag = 2;   // tiles another kv head must be behind before a workgroup helps it

// O^T accumulators pinned to their registers (never touched by the VALU inside the loop)
__device__ __forceinline__ void mfma16_acc(bf16x8 a, bf16x8 b, f32x4& c) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ f32x4 mfma16_zero(bf16x8 a, bf16x8 b) {
    f32x4 c;
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
    return c;
}
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The softmax arithmetic of the main loop, written out so that each instruction stays between
// the two MFMAs it was put between (the compiler otherwise gathers them behind a pair of
// MFMAs, and a wave that waits for the matrix pipe at the second one issues nothing).  The
// result of the exponential is consumed at least one MFMA later, as the hardware requires.
__device__ __forceinline__ float vexp2(float x) {
    float y;
    asm volatile("v_exp_f32 %0, %1" : "=v"(y) : "v"(x));
    return y;
}
__device__ __forceinline__ float vfma_sub(float a, float b, float c) {   // a * b - c
    float y;
    asm volatile("v_fma_f32 %0, %1, %2, -%3" : "=v"(y) : "v"(a), "s"(b), "v"(c));
    return y;
}
__device__ __forceinline__ float vadd(float a, float b) {
    float y;
    asm volatile("v_add_f32 %0, %1, %2" : "=v"(y) : "v"(a), "v"(b));
    return y;
}
__device__ __forceinline__ uint32_t vpack(float lo, float hi) {
    uint32_t y;
    asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(y) : "v"(lo), "v"(hi));
    return y;
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// kNatV: the values are read from the cache as it is (key-major) and transposed on their
// way out of LDS; otherwise from a V^T copy made by a pre-pass.
template <bool kNatV>
__global__ __launch_bounds__(kThreads) void attn_w8n_kernel(AttnParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_red[NW];
    __shared__ int s_job;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4;    // key octet of a 32-key sub-step this lane holds scores of
    const int l16 = lane & 15;   // its column in each of the wave's two 16-column blocks

    // Work distribution: one workgroup per CU takes (kv head, row tile[, key range]) jobs, heaviest
    // first (tiles from the last one on, or by p.order), claimed from one counter per kv head; it
    // prefers its home head (whose K/V its XCD's L2 holds) unless another head is kStealLag or more
    // jobs behind.  The first p.dealt jobs (one per workgroup, or none) go by the workgroup's number
    // instead (deal_first_jobs).
    const int home = blockIdx.x % p.hkv;
    const int jobs_per_head = p.n_tiles * p.dma_splits;
    // jobs of head h that went by number, and with those claimed (a division here, eight times a
    // claim, took 1.4 us of every job)
    const int dealt_each = p.dealt / p.hkv, dealt_rest = p.dealt % p.hkv;
    auto dealt = [&](int h) { return dealt_each + (h < dealt_rest ? 1 : 0); };
    auto taken = [&](int h) {
        return dealt(h) +
               __hip_atomic_load(&p.queue[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
  for (bool first = p.dealt > 0;; first = false) {
    if (tid == 0) {
        // (the grid is no larger than the number of jobs, so there is a first one)
        int head = home, j = first ? (int)(blockIdx.x / p.hkv) : jobs_per_head;
        // at most hkv failed claims: each one finds a head exhausted for good
        for (int attempt = 0; attempt <= p.hkv && j >= jobs_per_head; ++attempt) {
            int best = home;
            int best_c = taken(home);
            if (best_c < jobs_per_head) best_c -= kStealLag;
            for (int q = 1; q < p.hkv; ++q) {
                int y = home + q;
                if (y >= p.hkv) y -= p.hkv;
                const int c = taken(y);
                if (c < best_c) {
                    best_c = c;
                    best = y;
                }
            }
            if (best_c >= jobs_per_head) break;   // nothing left anywhere
            head = best;
            j = dealt(best) + atomicAdd(&p.queue[best], 1);
        }
        int job = -1;
        if (j < jobs_per_head) job = head * jobs_per_head + (p.order ? p.order[j] : j);
        s_job = job;
    }
    __syncthreads();
    const int job = __builtin_amdgcn_readfirstlane(s_job);
    if (job < 0) break;   // block-uniform: every head is exhausted
    const int g = job / jobs_per_head;
    const int within = job - g * jobs_per_head;
    const int tile = p.n_tiles - 1 - within / p.dma_splits;
    const int split = within % p.dma_splits;
    const int kb = split * p.dma_split_len;                      // a multiple of kBN
    const int n_keys_job = min(p.n_keys - kb, p.dma_split_len);  // keys the job may touch

    // ---- this lane's two columns ----------------------------------------------------------
    int row[2], head[2], limit[2];
    bool valid[2];
    int lmax = -1, lmin = 0x7fffffff;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const int col = wave * 32 + ct * 16 + l16;
        const int rl = col / p.group;
        row[ct] = tile * p.bm + rl;
        head[ct] = g * p.group + col % p.group;
        valid[ct] = rl < p.bm && row[ct] < p.m;
        // last key of this job's range that the column sees (negative: none).  Clamped to the
        // range: the pipeline forms the probabilities of one sub-step beyond the last tile and
        // adds them to the sum, so whatever lies behind the range has to be masked like the
        // keys behind the row's own position.
        limit[ct] = valid[ct] ? min(p.row_pos[row[ct]] - kb, n_keys_job - 1) : -1;
        lmax = max(lmax, limit[ct]);
        if (valid[ct]) lmin = min(lmin, limit[ct]);
    }
    for (int o = 8; o > 0; o >>= 1) {
        lmax = max(lmax, __shfl_xor(lmax, o, 64));
        lmin = min(lmin, __shfl_xor(lmin, o, 64));
    }
    if (lane == 0) s_red[wave] = lmax;
    __syncthreads();
    int tile_max = -1;
#pragma unroll
    for (int w = 0; w < NW; ++w) tile_max = max(tile_max, s_red[w]);
    const int key_end = min(tile_max + 1, n_keys_job);
    const int n_iter = __builtin_amdgcn_readfirstlane((key_end + kBN - 1) / kBN);
    if (n_iter <= 0) continue;   // block-uniform: no valid row, or no row reaches this range
    // sub-steps [0, u_unm) lie entirely at or below every limit of this wave; a wave without
    // a valid column has nothing to mask
    const int u_unm = __builtin_amdgcn_readfirstlane(lmin == 0x7fffffff ? 0x3fffffff
                                                                        : (lmin + 1) / 32);

    // ---- Q as B operands ---------------------------------------------------------------------
    bf16x8 qreg[2][KC];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const bf16_t* qp = p.q + ((int64_t)row[ct] * p.hq + head[ct]) * D + g4 * 8;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            if (valid[ct]) {
                qreg[ct][kc] = *reinterpret_cast<const bf16x8*>(qp + kc * 32);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) qreg[ct][kc][e] = (bf16_t)0.0f;
            }
        }
    }

    float m_run[2], l_run[2];
    f32x4 o_acc[DB][2];

    // ---- global -> LDS ------------------------------------------------------------------------
    // K stage: key row r at byte r*256, 16-byte chunk c at c ^ fk(r), fk(r) = 4 ((r >> 3) & 3) +
    // (r & 3): the sixteen rows of one operand read differ in just those bits.  V^T stage: row d
    // at byte d*128, chunk c at c ^ ((d >> 1) & 7).  A wave instruction fills 1 KB; wave w owns K
    // rows [8w, 8w+8) and V^T rows [16w, 16w+16) of every tile: two instructions each.
    // Key-major V stage (kNatV): key row r at byte r*256, chunk c at c ^ 2 fv(r), fv(r) =
    // (r & 3) + 4 ((r >> 3) & 1), so that the eight rows x 32 bytes a half wave reads in one
    // transposing instruction cover all 64 banks once; wave w owns rows [8w, 8w+8).
    const uint32_t lds_k = (uint32_t)(uintptr_t)smem;
    const uint32_t lds_v = lds_k + NS * kStageK;
    const uint32_t k_row_bytes = (uint32_t)p.hkv * D * 2;
    uint32_t voff_k[2], voff_v[2], kofs_last[2], vofs_last[2];
    {
        const int last = (n_keys_job - 1) % kBN;   // last row of the (possibly ragged) last tile
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 8 * wave + 4 * i + (lane >> 4);
            const uint32_t chunk = (uint32_t)(((lane & 15) ^ (((r >> 1) & 12) | (r & 3))) * 16);
            voff_k[i] = (uint32_t)r * k_row_bytes + chunk;
            kofs_last[i] = (uint32_t)min(r, last) * k_row_bytes + chunk;
            if (kNatV) {
                const uint32_t vchunk = (uint32_t)(((lane & 15) ^ (2 * (r & 3) + (r & 8))) * 16);
                voff_v[i] = (uint32_t)r * k_row_bytes + vchunk;
                vofs_last[i] = (uint32_t)min(r, last) * k_row_bytes + vchunk;
            } else {
                const int d = 16 * wave + 8 * i + (lane >> 3);
                voff_v[i] =
                    (uint32_t)d * (uint32_t)p.n_pad * 2u + (((lane & 7) ^ ((d >> 1) & 7)) * 16);
                vofs_last[i] = voff_v[i];
            }
        }
    }
    const uint32_t lds_k_wave = __builtin_amdgcn_readfirstlane(lds_k + wave * 8 * 256);
    const uint32_t lds_v_wave = __builtin_amdgcn_readfirstlane(lds_v + wave * 16 * 128);
    const bf16_t* const k_head = p.k + ((int64_t)kb * p.hkv + g) * D;
    const bf16_t* const v_head = kNatV ? p.v + ((int64_t)kb * p.hkv + g) * D
                                       : p.vt + (int64_t)g * D * p.n_pad + kb;

    // K tile T / V^T tile T (clamped to the last tile) into their ring slots, both instructions
#define W8_DMA_K(T)                                                                      \
    {                                                                                    \
        const int t_ = min((T), n_iter - 1);                                             \
        const bf16_t* gb_ = k_head + (int64_t)t_ * kBN * p.hkv * D;                      \
        const bool full_ = t_ * kBN + kBN <= n_keys_job;                                 \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                    \
            dma16(gb_, full_ ? voff_k[i] : kofs_last[i],                                 \
                  lds_k_wave + ((T) & 3) * kStageK + i * 1024);                          \
    }
#define W8_DMA_V(T)                                                                      \
    {                                                                                    \
        const int t_ = min((T), n_iter - 1);                                             \
        const bf16_t* gb_ = kNatV ? v_head + (int64_t)t_ * kBN * p.hkv * D               \
                                  : v_head + t_ * kBN;                                   \
        const bool full_ = t_ * kBN + kBN <= n_keys_job;                                 \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                    \
            dma16(gb_, full_ ? voff_v[i] : vofs_last[i],                                 \
                  lds_v_wave + ((T) & 3) * kStageV + i * 1024);                          \
    }
    // the four fill instructions of a tile body (K tile J+4, V^T tile J+2), one pair per
    // sub-step, prepared once per tile
    const bf16_t* gbk_;
    const bf16_t* gbv_;
    bool k_full_, v_full_;
#define W8_DMA_PREP(J)                                                                   \
    {                                                                                    \
        const int tk_ = min((J) + 4, n_iter - 1);                                        \
        gbk_ = k_head + (int64_t)tk_ * kBN * p.hkv * D;                                  \
        k_full_ = tk_ * kBN + kBN <= n_keys_job;   /* wave-uniform */                    \
        const int tv_ = min((J) + 2, n_iter - 1);                                        \
        gbv_ = kNatV ? v_head + (int64_t)tv_ * kBN * p.hkv * D : v_head + tv_ * kBN;     \
        v_full_ = tv_ * kBN + kBN <= n_keys_job;                                         \
    }
#define W8_DMA_ONE_K(I, SDK)                                                             \
    dma16(gbk_, k_full_ ? voff_k[I] : kofs_last[I], lds_k_wave + (SDK) * kStageK + (I) * 1024);
#define W8_DMA_ONE_V(I, SDV)                                                             \
    dma16(gbv_, v_full_ ? voff_v[I] : vofs_last[I], lds_v_wave + (SDV) * kStageV + (I) * 1024);

    // ---- LDS -> register operand addresses (bytes inside a stage) -----------------------------
    // Of a 32-key sub-step, A-row 4 a + i of key block kt reads key 8 a + 4 kt + i, so that a
    // lane's accumulator registers of the two blocks hold keys 8 g4 .. 8 g4 + 7 of its column:
    // the B operand of the second contraction.  Key block 1 is 4 rows (1 KB) behind block 0.
    uint32_t kaddr[KC], vaddr[8];
    {
        const int a = l16 >> 2, i = l16 & 3;
        const uint32_t a0 = (8 * a + i) * 256 + ((g4 ^ (4 * a + i)) * 16);
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kaddr[kc] = a0 ^ (kc << 6);
        if (kNatV) {
            // vaddr[db]: the 8 bytes this lane addresses for the d-block db of a sub-step
            // (row 8 g4 + e, d = 16 db + 4 j .. + 3; four rows further for the second half)
            const int e = l16 >> 2, j = l16 & 3;
#pragma unroll
            for (int db = 0; db < 8; ++db)
                vaddr[db] = (uint32_t)((8 * g4 + e) * 256 + ((db ^ (e + 4 * (g4 & 1))) * 32) +
                                       j * 8);
        } else {
            // vaddr[h]: row l16 of a d-block (2 KB apart), keys 8 g4 .. of sub-step h
#pragma unroll
            for (int h = 0; h < 2; ++h)
                vaddr[h] = l16 * 128 + (((4 * h + g4) ^ (l16 >> 1)) * 16);
        }
        // the value stages lie behind the 64 KB of key stages: with that base inside the lane's
        // address every stage and block offset of a value read fits the 16-bit immediate of
        // the LDS instruction, and no address arithmetic is left in the loop
#pragma unroll
        for (int q = 0; q < (kNatV ? 8 : 2); ++q) vaddr[q] += NS * kStageK;
    }
    const float c2 = p.scale_log2;

    f32x4 s_a[2][2], s_b[2][2];   // S^T of even / odd sub-steps: [key block][column block]
    u32x4 pb_a[2], pb_b[2];       // P^T (bf16 pairs) of even / odd sub-steps: [column block]
    bf16x8 ka[2 * KC], va[DB];    // ka[2 kc + key block]
    // sums of the probabilities being produced: of the last pair, of a column's eight
    float t_sum, rs;
    float msc[2];                 // reference maximum times c2 (0 while it is -inf)
    constexpr float kGrow = 1.0e24f;   // ~2^80
    float e0, e1, e2;                     // the last probabilities, the newest first
    float x_next;                         // exponent of the next one

    // operand i = 2 kc + key block of the K half tile (ST, H); d-block DBI of the value half
    // tile (ST, H)
#define W8_LOAD_KA1(ST, H, I_)                                                           \
    ka[I_] = *reinterpret_cast<const bf16x8*>(                                           \
        smem + (ST) * kStageK + (H) * 32 * 256 + ((I_) & 1) * 1024 + kaddr[(I_) >> 1]);
#define W8_LOAD_KA(ST, H)                                                                \
    _Pragma("unroll") for (int i_ = 0; i_ < 2 * KC; ++i_) { W8_LOAD_KA1(ST, H, i_) }
#define W8_LOAD_VA1(ST, H, DBI)                                                          \
    if (kNatV) {                                                                         \
        const unsigned char* a_ = smem + (ST) * kStageV + (H) * 32 * 256 + vaddr[DBI];   \
        const bf16x4 lo_ = lds_read_tr(a_), hi_ = lds_read_tr(a_ + 4 * 256);             \
        va[DBI] = __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7);             \
    } else {                                                                             \
        va[DBI] = *reinterpret_cast<const bf16x8*>(                                      \
            smem + (ST) * kStageV + (DBI) * 16 * 128 + vaddr[H]);                        \
    }

    // Scores are taken in the order R = 8 * column block + key of the octet.
    // exponent of score R of score buffer S whose first key is T0
#define W8_SM_PREP(S, R, T0, MASK)                                                       \
    {                                                                                    \
        float x_ = S[((R) & 7) >> 2][(R) >> 3][(R) & 3];                                 \
        if (MASK) {                                                                      \
            const int key_ = (T0) + 8 * g4 + ((R) & 7);                                  \
            if (key_ > limit[(R) >> 3]) x_ = -INFINITY;                                  \
        }                                                                                \
        x_next = vfma_sub(x_, c2, msc[(R) >> 3]);                                        \
    }
    // A softmax step is split over the two MFMAs of a pair.  First half: the probability of
    // score R from the exponent prepared one step earlier.
#define W8_SM_EXP                                                                        \
    e2 = e1;                                                                             \
    e1 = e0;                                                                             \
    e0 = vexp2(x_next);
    // Second half: the exponent of score RN of SN (first key T0N), and, when R is even, the
    // pair of scores (R - 2, R - 1) is packed into the B operand and summed; when R is odd that
    // sum goes to its column's.  At R = 0, 1 the pair is the last one of the previous
    // sub-step, whose probabilities are PCUR.
#define W8_SM_REST(PCUR, PNXT, R, SN, RN, T0N, MASK)                                     \
    W8_SM_PREP(SN, RN, T0N, MASK)                                                        \
    if ((R) % 2 == 0) {                                                                  \
        if ((R) == 0) PCUR[1][3] = vpack(e2, e1);                               \
        else PNXT[((R) - 2) >> 3][(((R) - 2) & 7) >> 1] = vpack(e2, e1);        \
        t_sum = vadd(e2, e1);                                                   \
    } else {                                                                             \
        rs = (R) == 3 || (R) == 11 ? t_sum : vadd(rs, t_sum);                            \
        if ((R) == 9) l_run[0] = vadd(l_run[0], rs);                                     \
        if ((R) == 1) l_run[1] = vadd(l_run[1], rs);                                     \
    }

    // One 32-key sub-step u.  SCUR = S^T(u+1) (complete), SNXT receives S^T(u+2) from the
    // operands in ka; PCUR = P(u) (complete), PNXT receives P(u+1); (KST, KH) name the K
    // half tile of sub-step u+3, (VST, VH) the V^T half tile of sub-step u; T0N is the first
    // key of sub-step u+1.  I = which of the tile's two fill pairs goes out here.
#define W8_SUBSTEP(SCUR, SNXT, PCUR, PNXT, KST, KH, VST, VH, T0N, MASK, I, SDK, SDV)     \
    {                                                                                    \
        __builtin_amdgcn_sched_barrier(0);                                               \
        W8_DMA_ONE_K(I, SDK)                                                             \
        __builtin_amdgcn_sched_barrier(0);                                               \
        /* every MFMA pair frees one operand; the operand that the other group needs     \
           eight pairs later is requested into its place, so K and V^T operands together \
           never hold more than nine registers' worth of tiles */                        \
        _Pragma("unroll") for (int i_ = 0; i_ < 8; ++i_) {                               \
            if (i_ < 2) SNXT[i_ & 1][0] = mfma16_zero(ka[i_], qreg[0][i_ >> 1]);         \
            else mfma16_acc(ka[i_], qreg[0][i_ >> 1], SNXT[i_ & 1][0]);                  \
            W8_SM_EXP                                                                    \
            __builtin_amdgcn_sched_barrier(0);                                           \
            if (i_ < 2) SNXT[i_ & 1][1] = mfma16_zero(ka[i_], qreg[1][i_ >> 1]);         \
            else mfma16_acc(ka[i_], qreg[1][i_ >> 1], SNXT[i_ & 1][1]);                  \
            W8_LOAD_VA1(VST, VH, i_)                                                     \
            W8_SM_REST(PCUR, PNXT, i_, SCUR, i_ + 1, T0N, MASK)                          \
            __builtin_amdgcn_sched_barrier(0);                                           \
        }                                                                                \
        W8_DMA_ONE_V(I, SDV)                                                             \
        __builtin_amdgcn_sched_barrier(0);                                               \
        _Pragma("unroll") for (int i_ = 0; i_ < 8; ++i_) {                               \
            mfma16_acc(va[i_], __builtin_bit_cast(bf16x8, PCUR[0]), o_acc[i_][0]);       \
            W8_SM_EXP                                                                    \
            __builtin_amdgcn_sched_barrier(0);                                           \
            mfma16_acc(va[i_], __builtin_bit_cast(bf16x8, PCUR[1]), o_acc[i_][1]);       \
            W8_LOAD_KA1(KST, KH, i_)                                                     \
            if (i_ < 7) { W8_SM_REST(PCUR, PNXT, 8 + i_, SCUR, 9 + i_, T0N, MASK) }      \
            else { W8_SM_REST(PCUR, PNXT, 15, SNXT, 0, (T0N) + 32, MASK) }               \
            __builtin_amdgcn_sched_barrier(0);                                           \
        }                                                                                \
    }

    // one 64-key tile J: sub-steps 2J, 2J+1.  K halves read: tile J+1 half 1 (stage SK1) and
    // tile J+2 half 0 (stage SK2); V^T tile J in stage SV0; K(J+4) -> stage SV0's index (the
    // slot of K(J)), V^T(J+2) -> stage SK2's index.
#define W8_TILE(J, SK1, SK2, SV0, MASK)                                                  \
    {                                                                                    \
        const int t0_tile_ = (J) * kBN;                                                  \
        W8_DMA_PREP(J)                                                                   \
        W8_SUBSTEP(s_b, s_a, pb_a, pb_b, SK1, 1, SV0, 0, t0_tile_ + 32, MASK, 0, SV0, SK2) \
        W8_SUBSTEP(s_a, s_b, pb_b, pb_a, SK2, 0, SV0, 1, t0_tile_ + 64, MASK, 1, SV0, SK2) \
        wait_vm<4>();   /* K(J+3), V^T(J+1) have landed; the 4 newest loads stay in flight */ \
        __syncthreads();                                                                 \
    }

    // Two attempts at most.  The first takes the maximum of a column's first 32 keys as its
    // softmax reference; where probabilities leave the safe range because later scores lie far
    // above it, the workgroup finds the true maxima of its columns and goes over its keys once
    // more with those (cold: one 64-key tile at a time).
    bool exact = false;
    float l_tot[2];
    for (;;) {
        l_run[0] = l_run[1] = t_sum = rs = e0 = e1 = e2 = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                for (int r = 0; r < 4; ++r) o_acc[db][ct][r] = 0.f;
    // ---- prologue -------------------------------------------------------------------------
    W8_DMA_K(0)
    W8_DMA_V(0)
    W8_DMA_K(1)
    W8_DMA_K(2)
    wait_vm<0>();
    __syncthreads();
    W8_DMA_K(3)
    W8_DMA_V(1)
#define W8_FIRST_S(S)                                                                    \
    _Pragma("unroll") for (int i_ = 0; i_ < 8; ++i_) {                                   \
        const f32x4 z_ = {0.f, 0.f, 0.f, 0.f};                                           \
        _Pragma("unroll") for (int ct_ = 0; ct_ < 2; ++ct_)                              \
            S[i_ & 1][ct_] = mfma16(ka[i_], qreg[ct_][i_ >> 1],                          \
                                    i_ < 2 ? z_ : S[i_ & 1][ct_]);                       \
    }
    W8_LOAD_KA(0, 0)
    W8_FIRST_S(s_a)
    W8_LOAD_KA(0, 1)
    W8_FIRST_S(s_b)
    W8_LOAD_KA(1, 0)            // operands of S^T(2)
    // the reference of a column: the maximum of its first 32 keys, fixed from here on
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        if (!exact) {
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (8 * g4 + e <= limit[ct]) mx = fmaxf(mx, s_a[e >> 2][ct][e & 3]);
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            m_run[ct] = fmaxf(mx, __shfl_xor(mx, 32, 64));
        }
        msc[ct] = (m_run[ct] == -INFINITY ? 0.f : m_run[ct]) * c2;
    }
    // the scores are read by statements of our own: made before this wait, read behind it
    asm volatile("s_nop 15"
                 : "+v"(s_a[0][0]), "+v"(s_a[0][1]), "+v"(s_a[1][0]), "+v"(s_a[1][1]),
                   "+v"(s_b[0][0]), "+v"(s_b[0][1]), "+v"(s_b[1][0]), "+v"(s_b[1][1]));
    // P(0); its last pair is packed and summed by the first sub-step
    W8_SM_PREP(s_a, 0, 0, true)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        W8_SM_EXP
        asm volatile("s_nop 1");
        if (r < 2) {
            W8_SM_PREP(s_a, r + 1, 0, true)
        } else if (r < 15) {
            W8_SM_REST(pb_b, pb_a, r, s_a, r + 1, 0, true)
        } else {
            W8_SM_REST(pb_b, pb_a, 15, s_b, 0, 32, true)
        }
    }
    // tile 0 already requests K(4) into the slot of K(0): every wave must be done reading it
    __syncthreads();

    // ---- main loop: four tiles per trip so that every LDS stage is a constant ----------------
    // tile j is mask free when every score it turns into a probability (sub-steps 2j+1, 2j+2
    // and the first element of 2j+3) lies at or below every limit of the wave: 2j + 3 < u_unm
    int n_unm = min(n_iter, max(0, (u_unm - 2) / 2));
    n_unm &= ~3;
    int j = 0;
    for (; j < n_unm; j += 4) {
        W8_TILE(j, 1, 2, 0, false)
        W8_TILE(j + 1, 2, 3, 1, false)
        W8_TILE(j + 2, 3, 0, 2, false)
        W8_TILE(j + 3, 0, 1, 3, false)
    }
    for (; j < n_iter; ++j) {
        W8_TILE(j, (j + 1) & 3, (j + 2) & 3, j & 3, true)
    }
    wait_vm<0>();   // nothing may still be writing LDS when the workgroup moves on
    // the last O^T MFMAs were issued behind the compiler's back: let them retire before the
    // accumulators are read (which the statements behind the wait keep behind it)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) asm volatile("" : "+v"(o_acc[db][ct]));

#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        l_tot[ct] = l_run[ct] + __shfl_xor(l_run[ct], 16, 64);
        l_tot[ct] += __shfl_xor(l_tot[ct], 32, 64);
    }
    {
        // (every partial sum is at most the total: all terms are positive)
        const bool bad = !(l_tot[0] < kGrow) || !(l_tot[1] < kGrow);
        const int wave_bad = __any(bad) ? 1 : 0;   // over all lanes, before the branch
        __syncthreads();                       // s_red held the tile limits so far
        if (lane == 0) s_red[wave] = wave_bad;
        __syncthreads();
        int marked = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) marked |= s_red[w];
        if (exact || !marked) break;           // block-uniform
        exact = true;
        float mx[2] = {-INFINITY, -INFINITY};
        for (int t = 0; t < n_iter; ++t) {
            __syncthreads();      // nobody reads the stage that is about to be filled
            W8_DMA_K(t)
            wait_vm<0>();
            __syncthreads();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                W8_LOAD_KA(t & 3, h)
                f32x4 s[2][2];
                W8_FIRST_S(s)
#pragma unroll
                for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (t * kBN + h * 32 + 8 * g4 + e <= limit[ct])
                            mx[ct] = fmaxf(mx[ct], s[e >> 2][ct][e & 3]);
            }
        }
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
            mx[ct] = fmaxf(mx[ct], __shfl_xor(mx[ct], 16, 64));
            m_run[ct] = fmaxf(mx[ct], __shfl_xor(mx[ct], 32, 64));
        }
        __syncthreads();
    }
    }   // second attempt

#undef W8_DMA_K
#undef W8_DMA_V
#undef W8_DMA_PREP
#undef W8_DMA_ONE_K
#undef W8_DMA_ONE_V
#undef W8_LOAD_KA
#undef W8_LOAD_KA1
#undef W8_LOAD_VA1
#undef W8_SM_PREP
#undef W8_SM_EXP
#undef W8_SM_REST
#undef W8_FIRST_S
#undef W8_SUBSTEP
#undef W8_TILE

    // ---- epilogue ------------------------------------------------------------------------------
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        if (!valid[ct]) continue;
        const float inv = 1.f / l_tot[ct];
        // A row whose keys all lie in the first range has its whole result in that range's
        // job: it is written as the final output there and never merged.  Every other row
        // leaves a normalised fp32 partial result per range it reaches.
        const int pos = min(p.row_pos[row[ct]], p.n_keys - 1);
        const bool direct = p.dma_splits == 1 || pos < p.dma_split_len;
        if (!direct) {
            if (pos >= kb) {   // else the row sees nothing of this range
                const int64_t colg = ((int64_t)split * p.m + row[ct]) * p.hq + head[ct];
                float* op = p.part_o + colg * D + 4 * g4;
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    *reinterpret_cast<f32x4*>(op + db * 16) = o_acc[db][ct] * inv;
                if (g4 == 0) p.part_lse[colg] = m_run[ct] * p.scale + logf(l_tot[ct]);
            }
        } else if (split == 0) {
            const int64_t colg = (int64_t)row[ct] * p.hq + head[ct];
            bf16_t* op = p.out + colg * D + 4 * g4;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (bf16_t)(o_acc[db][ct][e] * inv);
                *reinterpret_cast<bf16x4*>(op + db * 16) = v;
            }
            if (g4 == 0) {
                const float lse = m_run[ct] * p.scale + logf(l_tot[ct]);
                if (p.lse) p.lse[colg] = lse;
                // asked for only when every key the row sees is a context key: unsplit
                // launches whose keys are all context keys, and first-range rows (a range
                // boundary lies at the end of the context)
                if (p.lse_ctx) p.lse_ctx[colg] = lse;
            }
        }
    }
  }   // next job
}

}  // namespace

// Whether a workgroup's first job goes by its number.  256 workgroups at the counters take 4 to
// 5 us to claim theirs (claimed -> by number, us, spread rows: 128 / 8 heads, 559 rows over 1.2k
// keys 49 -> 44, 32 / 32, 1141 over 13k in two ranges 184 -> 170, 28 / 4, 762 over 9.8k in four
// 84 -> 79).  Workgroups of one number modulo eight share an XCD, and with kv heads that divide
// eight their first jobs lie 8 / hkv apart: with two or four ranges some XCDs then begin with
// the fuller ranges only (8 / 2, 5614 over 19.6k in two 231 -> 252, 16 / 2, 1459 over 17k in
// four 124 -> 131, 28 / 4, 1839 over 21k in two 259 -> 273).  Fewer kv heads than XCDs and more
// than two jobs per CU: level or 2 % slower (28 / 4, 5096 over 11.6k 366 -> 374).
static bool deal_first_jobs(int hkv, int n_splits, int64_t jobs, int n_cu) {
    if (hkv % 8 == 0) return true;
    return jobs <= 2 * (int64_t)n_cu && !(hkv % 2 == 0 && (n_splits == 2 || n_splits == 4));
}

pkv_status launch_attn_w8n_main(AttnParams p, int n_cu, hipStream_t st) {
    static std::atomic<bool> configured{false};   // set twice at worst: the calls are idempotent
    if (!configured.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(attn_w8n_kernel<false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(attn_w8n_kernel<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLdsBytes) != hipSuccess)
            return PKV_ERR_LAUNCH;
        configured.store(true, std::memory_order_release);
    }
    // one workgroup per CU (its LDS admits no second one), or per job if there are fewer
    const int64_t grid = std::min<int64_t>((int64_t)p.n_tiles * p.dma_splits * p.hkv, n_cu);
    p.dealt = deal_first_jobs(p.hkv, p.dma_splits, (int64_t)p.n_tiles * p.dma_splits * p.hkv, n_cu)
                  ? (int)grid : 0;
    if (p.v)   // the values as the cache holds them; p.vt is then not used
        hipLaunchKernelGGL(attn_w8n_kernel<true>, dim3((unsigned)grid), dim3(kThreads), kLdsBytes,
                           st, p);
    else
        hipLaunchKernelGGL(attn_w8n_kernel<false>, dim3((unsigned)grid), dim3(kThreads),
                           kLdsBytes, st, p);
    return launch_status();
}

}  // namespace pkv
