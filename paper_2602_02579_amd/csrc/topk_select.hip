// Step 3: top-p selection - indices of the k largest fused scores, ties to
// the lower index, returned in ascending index order.
// (Paper: Eq. 4, TOP_p of the value function; Algorithm 1, "Select token
// indices"; Sec. 4.3: the set is chosen once and used by every layer.)
//
// One workgroup of 1024 lanes (16 waves).  The score vector is small (128 KB
// at 32k context) and stays in L2, so the kernel is latency-bound.
//
// Up to 64 scores per lane (n <= 65536) the keys live in registers (topk_radix_kernel):
//   1. the smallest and the largest key; 2048 bins of equal width between them are counted
//      with LDS atomics and searched from the top for the k-th largest key, then the bin that
//      holds it is divided again, until the whole bin is wanted or it is one key wide (two or
//      three times; keys are spread over the bins by the span of the actual scores, so the
//      few binades that real scores occupy do not meet in a few bins);
//   2. an index-ordered compaction by ballots; of keys equal to the threshold those at the
//      lowest indices are taken - the lower-index tie rule.
// Built bit by bit instead, with a count over all keys and a barrier per bit, the threshold
// took up to 32 rounds.
// Longer vectors use the radix kernel below:
//   1. radix select, 4 passes of 8 bits over order-preserving uint32 keys,
//      finds the key tau of the k-th largest score and how many scores equal
//      to tau are still needed;
//   2. an index-ordered compaction: every wave owns a contiguous segment,
//      counts its (> tau, == tau) elements with ballots, a 16-entry scan
//      gives each wave its output offset, and a second walk writes the
//      selected indices.  An element equal to tau is taken only while the
//      number of equal elements at lower indices is below the need, which is
//      exactly the lower-index tie rule.
#include "pkv_common.h"

namespace pkv {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

// larger float <=> larger key; -0.0 is folded onto +0.0 first
__device__ __forceinline__ uint32_t order_key(float x) {
    uint32_t u = __float_as_uint(x + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

__global__ __launch_bounds__(kThreads) void topk_select_kernel(
    const float* __restrict__ score, int n, int k, int32_t* __restrict__ idx_out) {
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_prefix, s_remaining;
    __shared__ uint32_t wave_gt[kWaves], wave_eq[kWaves], wave_off[kWaves],
        wave_eq_before[kWaves];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    // ---- 1. radix select of the k-th largest key --------------------------
    if (tid == 0) {
        s_prefix = 0;
        s_remaining = (uint32_t)k;
    }
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        const uint32_t prefix = s_prefix;
        const uint32_t himask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
        for (int i = tid; i < n; i += kThreads) {
            const uint32_t key = order_key(score[i]);
            if ((key & himask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (wave == 0) {
            // lane l owns digits 4l .. 4l+3; suffix sums from the top digit
            uint32_t c[4];
            uint32_t mine = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                c[j] = hist[4 * lane + j];
                mine += c[j];
            }
            // inclusive suffix scan over lanes (higher lanes = larger digits)
            uint32_t suf = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = __shfl_down(suf, d, 64);
                if (lane + d < 64) suf += o;
            }
            uint32_t above = suf - mine;  // elements with digits above my four
            const uint32_t remaining = s_remaining;
            // digits from high to low inside my four
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                if (above < remaining && remaining <= above + c[j]) {
                    s_prefix = prefix | ((uint32_t)(4 * lane + j) << shift);
                    s_remaining = remaining - above;
                }
                above += c[j];
            }
        }
        __syncthreads();
    }
    const uint32_t tau = s_prefix;
    const uint32_t need = s_remaining;  // elements == tau still to take (>= 1 if k > 0)

    // ---- 2. index-ordered compaction ---------------------------------------
    int seg = (n + kWaves - 1) / kWaves;
    seg = (seg + 63) & ~63;
    const int begin = wave * seg < n ? wave * seg : n;
    const int end = begin + seg < n ? begin + seg : n;

    uint32_t gt = 0, eq = 0;
    for (int i = begin + lane; i - lane < end; i += 64) {
        const bool in = i < end;
        const uint32_t key = in ? order_key(score[i]) : 0u;
        gt += __popcll(__ballot(in && key > tau));
        eq += __popcll(__ballot(in && key == tau));
    }
    if (lane == 0) {
        wave_gt[wave] = gt;
        wave_eq[wave] = eq;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t off = 0, eqb = 0;
        for (int w = 0; w < kWaves; ++w) {
            wave_off[w] = off;
            wave_eq_before[w] = eqb;
            const uint32_t room = eqb < need ? need - eqb : 0u;
            off += wave_gt[w] + (wave_eq[w] < room ? wave_eq[w] : room);
            eqb += wave_eq[w];
        }
    }
    __syncthreads();
    if (k == 0) return;
    uint32_t out = wave_off[wave];
    uint32_t eq_run = wave_eq_before[wave];
    const uint64_t lt = lanemask_lt();
    for (int i = begin + lane; i - lane < end; i += 64) {
        const bool in = i < end;
        const uint32_t key = in ? order_key(score[i]) : 0u;
        const uint64_t beq = __ballot(in && key == tau);
        const bool is_eq = in && key == tau;
        const bool take = in && (key > tau ||
                                 (is_eq && eq_run + __popcll(beq & lt) < need));
        const uint64_t bsel = __ballot(take);
        if (take) idx_out[out + __popcll(bsel & lt)] = i;
        out += __popcll(bsel);
        eq_run += __popcll(beq);
    }
}

// Keys of the kernel below: past the end of the vector 0, of scores order_key, one higher below
// zero: no score has the key that is free between the two halves, -0.0 being folded.
__device__ __forceinline__ uint32_t inner_key(float x) {
    const uint32_t u = __float_as_uint(x + 0.0f);
    return (u & 0x80000000u) ? 0u - u : (u | 0x80000000u);
}

// Updates of one LDS counter by c lanes of an instruction take about 6 c cycles, so a key that many
// scores share (zeros of an underflow, masks, ties) is kept out of the bins: every wave looks
// whether kOften of 64 of its keys are one, the block takes two such keys, and their number goes
// to the bin they belong to in one update per wave.  And a bin that holds a sixteenth of all keys
// is divided by the span of the keys in it, not by its width: often it is one key, and done.
// Vectors of kOftenMin or fewer scores do without the former.
constexpr int kOften = 4, kOftenMin = 2048;

// One workgroup, the keys in registers: wave w owns scores [64 ITEMS w, 64 ITEMS (w + 1)),
// a lane four consecutive ones of every 256.
template <int ITEMS, bool OFTEN>
__global__ __launch_bounds__(kThreads) void topk_radix_kernel(
    const float* __restrict__ score, int n, int k, int32_t* __restrict__ idx_out) {
    constexpr int kBins = 2048, kBits = 11;
    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t s_a[kWaves], s_b[kWaves], s_res[3];
    __shared__ uint32_t s_often[2 * kWaves];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int base = wave * 64 * ITEMS + lane * 4;   // + 256 (j / 4) + j % 4 for element j

    uint32_t key[ITEMS];
    uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
    for (int j = 0; j < ITEMS; j += 4) {
        const int i0 = base + j * 64;
        if (i0 + 3 < n) {
            const float4 v = *reinterpret_cast<const float4*>(score + i0);
            key[j] = inner_key(v.x);
            key[j + 1] = inner_key(v.y);
            key[j + 2] = inner_key(v.z);
            key[j + 3] = inner_key(v.w);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) key[j + e] = i0 + e < n ? inner_key(score[i0 + e]) : 0u;
        }
    }
    // ---- 1. the span of the keys: mn + 1 to mx ---------------------------------------------
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        mn = min(mn, key[j] - 1u);   // no score: wraps to the largest
        mx = max(mx, key[j]);
    }
    // up to two keys that kOften or more of 64 of the wave's keys are (0: none)
    uint32_t often[2] = {0u, 0u};
    if (OFTEN) {
        uint64_t left = __ballot(key[0] != 0u);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (left == 0) break;
            const uint32_t k0 = __builtin_amdgcn_readlane(key[0], (int)__builtin_ctzll(left));
            const uint64_t same = __ballot(key[0] == k0) & left;
            left &= ~same;
            if (__popcll(same) >= kOften) often[r] = k0;
        }
    }
    if (OFTEN && lane == 0) {
        s_often[2 * wave] = often[0];
        s_often[2 * wave + 1] = often[1];
    }
    hist[tid] = 0u;
    hist[tid + kThreads] = 0u;
    // smallest and largest of the block's values; a barrier inside
    auto block_span = [&](uint32_t& lo_, uint32_t& hi_) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo_ = min(lo_, __shfl_xor(lo_, o, 64));
            hi_ = max(hi_, __shfl_xor(hi_, o, 64));
        }
        if (lane == 0) {
            s_a[wave] = lo_;
            s_b[wave] = hi_;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            lo_ = min(lo_, s_a[w]);
            hi_ = max(hi_, s_b[w]);
        }
    };
    block_span(mn, mx);
    // the block's two, the same in every wave
    bool crowded = false;
    if (OFTEN) {
        const uint32_t v = s_often[lane & (2 * kWaves - 1)];
        const uint64_t some = __ballot(v != 0u);
        crowded = some != 0;
        often[0] = often[1] = 0u;
        if (crowded) {
            often[0] = __builtin_amdgcn_readlane(v, (int)__builtin_ctzll(some));
            const uint64_t more = __ballot(v != 0u && v != often[0]);
            if (more) often[1] = __builtin_amdgcn_readlane(v, (int)__builtin_ctzll(more));
        }
    }
    // how many of the wave's keys are those
    uint32_t own[2] = {0u, 0u};
    if (crowded) {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            own[0] += __popcll(__ballot(key[j] == often[0]));
            own[1] += __popcll(__ballot(key[j] == often[1]));
        }
    }

    // ---- 2. lo = lower end of the bin with the k-th largest key, ever finer ----------------
    // keys [lo, lo + span] are counted; no bin reaches beyond the largest key, so that a key of 0,
    // which wraps to the far end too, lies in none
    const uint32_t top = mx;
    uint32_t lo = mn + 1u, span = top - lo;
    uint32_t rest = (uint32_t)k, cnt = 0u;
    int shift = span ? max(0, 32 - __clz(span) - kBits) : 0;
    for (;;) {
        if (!crowded) {
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t d = key[j] - lo;   // wraps to the far end below lo
                if (d <= span) atomicAdd(&hist[d >> shift], 1u);
            }
        } else {
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t d = key[j] - lo;
                if (d <= span && key[j] != often[0] && key[j] != often[1])
                    atomicAdd(&hist[d >> shift], 1u);
            }
            const uint32_t d = (lane == 0 ? often[0] : often[1]) - lo;
            if (lane < 2 && d <= span) atomicAdd(&hist[d >> shift], lane == 0 ? own[0] : own[1]);
        }
        __syncthreads();
        // thread t owns the bins 2047 - 2 t and 2046 - 2 t; counts above them
        const uint32_t c0 = hist[kBins - 1 - 2 * tid], c1 = hist[kBins - 2 - 2 * tid];
        uint32_t inc = c0 + c1;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        if (lane == 63) s_a[wave] = inc;
        __syncthreads();
        uint32_t above = inc - c0 - c1;
        for (int w = 0; w < wave; ++w) above += s_a[w];
        if (above < rest && rest <= above + c0) {
            s_res[0] = kBins - 1 - 2 * tid;
            s_res[1] = rest - above;
            s_res[2] = c0;
        } else if (above + c0 < rest && rest <= above + c0 + c1) {
            s_res[0] = kBins - 2 - 2 * tid;
            s_res[1] = rest - above - c0;
            s_res[2] = c1;
        }
        hist[kBins - 1 - 2 * tid] = 0u;
        hist[kBins - 2 - 2 * tid] = 0u;
        __syncthreads();
        lo += s_res[0] << shift;
        rest = s_res[1];
        cnt = s_res[2];
        // the whole bin is wanted: the selection is everything from lo on; or the bin is one
        // key wide and `rest` of its equals are wanted
        if (rest == cnt || shift == 0) break;
        span = min((1u << shift) - 1u, top - lo);
        if (cnt <= (uint32_t)n / 16u) {
            shift = max(0, shift - kBits);
            continue;
        }
        // the span that the bin's keys really take
        mn = 0xffffffffu;
        mx = 0u;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint32_t d = key[j] - lo;
            mn = min(mn, d <= span ? d : 0xffffffffu);
            mx = max(mx, d <= span ? d : 0u);
        }
        block_span(mn, mx);
        lo += mn;
        span = mx - mn;
        if (span == 0u) {
            __syncthreads();   // s_a and s_b are written again below
            break;
        }
        shift = max(0, 32 - __clz(span) - kBits);
    }

    // ---- 3. compaction in index order -------------------------------------------------------
    const uint64_t lt = lanemask_lt();
    if (rest == cnt) {
        uint32_t mine = 0;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) mine += __popcll(__ballot(key[j] >= lo));
        if (lane == 0) s_b[wave] = mine;
        __syncthreads();
        uint32_t out = 0;
        for (int w = 0; w < wave; ++w) out += s_b[w];
#pragma unroll
        for (int j = 0; j < ITEMS; j += 4) {
            uint32_t at = out;
            bool take[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                take[e] = key[j + e] >= lo;
                const uint64_t b = __ballot(take[e]);
                at += __popcll(b & lt);
                out += __popcll(b);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (take[e]) idx_out[at++] = base + j * 64 + e;
        }
        return;
    }
    // `rest` of the cnt keys equal to lo, those at the lowest indices
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        gt += __popcll(__ballot(key[j] > lo));
        eq += __popcll(__ballot(key[j] == lo));
    }
    if (lane == 0) {
        s_a[wave] = gt;
        s_b[wave] = eq;
    }
    __syncthreads();
    gt = eq = 0;       // of the waves before mine, then of the groups as well
    for (int w = 0; w < wave; ++w) {
        gt += s_a[w];
        eq += s_b[w];
    }
#pragma unroll
    for (int j = 0; j < ITEMS; j += 4) {
        uint32_t g_at = gt, e_at = eq;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t bg = __ballot(key[j + e] > lo);
            const uint64_t be = __ballot(key[j + e] == lo);
            g_at += __popcll(bg & lt);
            e_at += __popcll(be & lt);
            gt += __popcll(bg);
            eq += __popcll(be);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool is_gt = key[j + e] > lo, is_eq = key[j + e] == lo;
            if (is_gt || (is_eq && e_at < rest)) idx_out[g_at + min(e_at, rest)] = base + j * 64 + e;
            g_at += is_gt ? 1u : 0u;
            e_at += is_eq ? 1u : 0u;
        }
    }
}


// ---------------------------------------------------------------------------
// Longer vectors with a workspace: a radix select spread over many
// workgroups, so that the counting runs at the bandwidth of the whole chip instead of one
// CU's.  A workgroup of 256 lanes owns 2048 consecutive scores (8 per lane, in registers).
//   hist<0>  histogram of the top 11 key bits              -> hist0[2048]
//   hist<1>  (bin0, rest0) from hist0; next 11 bits of the keys in bin0 -> hist1[2048]
//   hist<2>  (bin1, rest1) from hist1; last 10 bits of the keys in (bin0, bin1) -> hist2[1024]
//   count    (bin2, need) from hist2 gives tau; per workgroup (keys > tau, keys == tau)
//   write    exclusive sums over the workgroups before mine give my output offset; equal
//            keys are taken in index order until `need` of them are - the lower-index rule
// Each kernel scans only the newest histogram: workgroup 0 leaves the (bin, rest) pair it
// found in the workspace for the kernels behind it.  Histogram updates are integer
// atomics, so the result does not depend on their order.
// Workspace (uint32 words): hist0[2048] hist1[2048] hist2[1024] sel[8] counts[2 * n_wg].
// ---------------------------------------------------------------------------
constexpr int kSeg = 2048;          // scores per workgroup
constexpr int kSegThreads = 256;
constexpr int kHistWords = 2048 + 2048 + 1024;

__global__ __launch_bounds__(256) void topk_ws_zero_kernel(uint32_t* __restrict__ ws) {
    for (int i = threadIdx.x; i < kHistWords + 8; i += 256) ws[i] = 0u;
}

// The bin b (counted from the top) with count(bins > b) < rest <= count(bins >= b), and what
// is left of rest inside it.  All 256 lanes call it; the result is block-uniform.
__device__ __forceinline__ void topk_find_bin(const uint32_t* __restrict__ hist, int nbins,
                                              uint32_t rest, uint32_t* bin_out,
                                              uint32_t* rest_out) {
    __shared__ uint32_t s_wsum[4];
    __shared__ uint32_t s_res[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = nbins / kSegThreads;          // 8 or 4
    uint32_t c[8];
    uint32_t mine = 0;
    // lane t owns bins [nbins - (t + 1) per, nbins - t per): the top bins belong to lane 0
    const int hi = nbins - tid * per;
    for (int j = 0; j < per; ++j) {
        c[j] = hist[hi - 1 - j];                  // descending
        mine += c[j];
    }
    uint32_t inc = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) s_wsum[wave] = inc;
    __syncthreads();
    uint32_t above = inc - mine;                  // keys in bins above mine
    for (int w = 0; w < wave; ++w) above += s_wsum[w];
    for (int j = 0; j < per; ++j) {
        if (above < rest && rest <= above + c[j]) {
            s_res[0] = (uint32_t)(hi - 1 - j);
            s_res[1] = rest - above;
        }
        above += c[j];
    }
    __syncthreads();
    *bin_out = s_res[0];
    *rest_out = s_res[1];
    __syncthreads();                              // s_res / s_wsum may be reused
}

__device__ __forceinline__ void topk_load_keys(const float* __restrict__ score, int n, int base,
                                               bool aligned, uint32_t* key) {
#pragma unroll
    for (int j = 0; j < 8; j += 4) {
        if (aligned && base + j + 3 < n) {
            const float4 v = *reinterpret_cast<const float4*>(score + base + j);
            key[j] = order_key(v.x);
            key[j + 1] = order_key(v.y);
            key[j + 2] = order_key(v.z);
            key[j + 3] = order_key(v.w);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)   // indices >= n: key 0, below every float's key
                key[j + e] = base + j + e < n ? order_key(score[base + j + e]) : 0u;
        }
    }
}

template <int PASS>
__global__ __launch_bounds__(256) void topk_ws_hist_kernel(const float* __restrict__ score, int n,
                                                           int k, uint32_t* __restrict__ ws,
                                                           int aligned) {
    __shared__ uint32_t s_hist[2048];
    uint32_t* hist0 = ws;
    uint32_t* hist1 = ws + 2048;
    uint32_t* hist2 = ws + 4096;
    uint32_t* sel = ws + kHistWords;
    const int tid = threadIdx.x;
    constexpr int nbins = PASS == 2 ? 1024 : 2048;
    for (int i = tid; i < nbins; i += 256) s_hist[i] = 0u;
    uint32_t prefix = 0;        // the key bits fixed so far, right-aligned
    if (PASS == 1) {
        uint32_t b, r;
        topk_find_bin(hist0, 2048, (uint32_t)k, &b, &r);
        if (blockIdx.x == 0 && tid == 0) { sel[0] = b; sel[1] = r; }
        prefix = b;
    } else if (PASS == 2) {
        uint32_t b, r;
        topk_find_bin(hist1, 2048, sel[1], &b, &r);
        if (blockIdx.x == 0 && tid == 0) { sel[2] = b; sel[3] = r; }
        prefix = (sel[0] << 11) | b;
    } else {
        __syncthreads();
    }
    uint32_t key[8];
    const int base = blockIdx.x * kSeg + tid * 8;
    topk_load_keys(score, n, base, aligned != 0, key);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (base + j >= n) continue;
        if (PASS == 0) atomicAdd(&s_hist[key[j] >> 21], 1u);
        else if (PASS == 1) { if ((key[j] >> 21) == prefix) atomicAdd(&s_hist[(key[j] >> 10) & 2047u], 1u); }
        else { if ((key[j] >> 10) == prefix) atomicAdd(&s_hist[key[j] & 1023u], 1u); }
    }
    __syncthreads();
    uint32_t* out = PASS == 0 ? hist0 : PASS == 1 ? hist1 : hist2;
    for (int i = tid; i < nbins; i += 256)
        if (s_hist[i]) atomicAdd(&out[i], s_hist[i]);
}

__global__ __launch_bounds__(256) void topk_ws_count_kernel(const float* __restrict__ score, int n,
                                                            uint32_t* __restrict__ ws, int aligned) {
    __shared__ uint32_t s_g[4], s_e[4];
    uint32_t* hist2 = ws + 4096;
    uint32_t* sel = ws + kHistWords;
    uint32_t* counts = sel + 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t b, need;
    topk_find_bin(hist2, 1024, sel[3], &b, &need);
    if (blockIdx.x == 0 && tid == 0) { sel[4] = b; sel[5] = need; }
    const uint32_t tau = (sel[0] << 21) | (sel[2] << 10) | b;
    uint32_t key[8];
    const int base = blockIdx.x * kSeg + tid * 8;
    topk_load_keys(score, n, base, aligned != 0, key);
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        gt += key[j] > tau ? 1u : 0u;
        eq += (key[j] == tau && base + j < n) ? 1u : 0u;
    }
    for (int o = 32; o > 0; o >>= 1) {
        gt += __shfl_xor(gt, o, 64);
        eq += __shfl_xor(eq, o, 64);
    }
    if (lane == 0) { s_g[wave] = gt; s_e[wave] = eq; }
    __syncthreads();
    if (tid == 0) {
        counts[2 * blockIdx.x] = s_g[0] + s_g[1] + s_g[2] + s_g[3];
        counts[2 * blockIdx.x + 1] = s_e[0] + s_e[1] + s_e[2] + s_e[3];
    }
}

__global__ __launch_bounds__(256) void topk_ws_write_kernel(const float* __restrict__ score, int n,
                                                            const uint32_t* __restrict__ ws,
                                                            int32_t* __restrict__ idx_out,
                                                            int aligned) {
    __shared__ uint32_t s_g[4], s_e[4];
    const uint32_t* sel = ws + kHistWords;
    const uint32_t* counts = sel + 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t tau = (sel[0] << 21) | (sel[2] << 10) | sel[4];
    const uint32_t need = sel[5];
    // keys > tau and keys == tau in the workgroups before mine
    uint32_t gb = 0, eb = 0;
    for (int w = tid; w < (int)blockIdx.x; w += 256) {
        gb += counts[2 * w];
        eb += counts[2 * w + 1];
    }
    for (int o = 32; o > 0; o >>= 1) {
        gb += __shfl_xor(gb, o, 64);
        eb += __shfl_xor(eb, o, 64);
    }
    if (lane == 0) { s_g[wave] = gb; s_e[wave] = eb; }
    __syncthreads();
    const uint32_t gt_wg = s_g[0] + s_g[1] + s_g[2] + s_g[3];
    const uint32_t eq_wg = s_e[0] + s_e[1] + s_e[2] + s_e[3];
    __syncthreads();
    uint32_t key[8];
    const int base = blockIdx.x * kSeg + tid * 8;
    topk_load_keys(score, n, base, aligned != 0, key);
    uint32_t my_gt = 0, my_eq = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        my_gt += key[j] > tau ? 1u : 0u;
        my_eq += (key[j] == tau && base + j < n) ? 1u : 0u;
    }
    uint32_t in_gt = my_gt, in_eq = my_eq;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t og = __shfl_up(in_gt, d, 64), oe = __shfl_up(in_eq, d, 64);
        if (lane >= d) { in_gt += og; in_eq += oe; }
    }
    if (lane == 63) { s_g[wave] = in_gt; s_e[wave] = in_eq; }
    __syncthreads();
    uint32_t gt_before = gt_wg + in_gt - my_gt, eq_before = eq_wg + in_eq - my_eq;
    for (int w = 0; w < wave; ++w) {
        gt_before += s_g[w];
        eq_before += s_e[w];
    }
    // equal keys at lower indices are taken first, until `need` of them are
    uint32_t out = gt_before + (eq_before < need ? eq_before : need);
    uint32_t eq_seen = eq_before;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool is_eq = key[j] == tau && base + j < n;
        const bool take = key[j] > tau || (is_eq && eq_seen < need);
        if (take) idx_out[out++] = base + j;
        eq_seen += is_eq ? 1u : 0u;
    }
}

}  // namespace

// Shortest vector that takes the many-workgroup kernels when a workspace is given (and, up to
// 32768 scores, only if its address is not a multiple of 16): their six launches cost a flat
// 17.5 us, one workgroup without register keys 43 us at 24k.
constexpr int64_t kWsMin = 24 * 1024 + 1;

size_t topk_select_ws_bytes(int64_t n) {
    if (n < kWsMin || n > ((int64_t)1 << 22)) return 0;   // other kernels, no scratch
    return (size_t)(kHistWords + 8 + 2 * ceil_div(n, kSeg)) * sizeof(uint32_t);
}

pkv_status launch_topk_select(const float* score, int64_t n, int64_t k,
                              int32_t* idx_out, void* ws, size_t ws_bytes, hipStream_t st) {
    if (n == 0 || k == 0) return PKV_OK;
    // the register kernels read 16 bytes at a time
    const bool aligned = (reinterpret_cast<uintptr_t>(score) & 15) == 0;
    // every pass walks over all register keys, so short vectors take the instantiation with
    // the fewest keys per lane that holds them.  From 1000 to 32768 scores 4.9, 6.7 (4k), 7.1
    // (8k), 9.1 (16k) and 13.9 us; the many-workgroup kernels take 17.5 at any length (with the
    // threshold built bit by bit 9, 10, 14, 15 and 26).  Scores that share a few values: 98 %
    // zeros 7.6, 7.8, 8.0, 10.7 and 18.8 (many workgroups 21.5), 25 values 6.9, 7.8, 8.7, 12.2 and
    // 21.5 (17.1; bit by bit 16, 16, 16, 22 and 33)
    if (aligned && n <= kOftenMin) {
        hipLaunchKernelGGL((topk_radix_kernel<8, false>), dim3(1), dim3(kThreads), 0, st, score,
                           (int)n, (int)k, idx_out);
        return launch_status();
    }
    if (aligned && n <= 8 * kThreads) {
        hipLaunchKernelGGL((topk_radix_kernel<8, true>), dim3(1), dim3(kThreads), 0, st, score,
                           (int)n, (int)k, idx_out);
        return launch_status();
    }
    if (aligned && n <= 16 * kThreads) {
        hipLaunchKernelGGL((topk_radix_kernel<16, true>), dim3(1), dim3(kThreads), 0, st, score,
                           (int)n, (int)k, idx_out);
        return launch_status();
    }
    if (aligned && n <= 32 * kThreads) {
        hipLaunchKernelGGL((topk_radix_kernel<32, true>), dim3(1), dim3(kThreads), 0, st, score,
                           (int)n, (int)k, idx_out);
        return launch_status();
    }
    const size_t need = topk_select_ws_bytes(n);
    if (need && ws && ws_bytes >= need && (reinterpret_cast<uintptr_t>(ws) & 3) == 0) {
        uint32_t* w = (uint32_t*)ws;
        const dim3 grid((unsigned)ceil_div(n, kSeg)), block(kSegThreads);
        const int al = aligned ? 1 : 0;
        hipLaunchKernelGGL(topk_ws_zero_kernel, dim3(1), block, 0, st, w);
        hipLaunchKernelGGL(topk_ws_hist_kernel<0>, grid, block, 0, st, score, (int)n, (int)k, w, al);
        hipLaunchKernelGGL(topk_ws_hist_kernel<1>, grid, block, 0, st, score, (int)n, (int)k, w, al);
        hipLaunchKernelGGL(topk_ws_hist_kernel<2>, grid, block, 0, st, score, (int)n, (int)k, w, al);
        hipLaunchKernelGGL(topk_ws_count_kernel, grid, block, 0, st, score, (int)n, w, al);
        hipLaunchKernelGGL(topk_ws_write_kernel, grid, block, 0, st, score, (int)n, w, idx_out, al);
        return launch_status();
    }
    if (aligned && n <= 64 * kThreads) {
        hipLaunchKernelGGL((topk_radix_kernel<64, true>), dim3(1), dim3(kThreads), 0, st, score,
                           (int)n, (int)k, idx_out);
        return launch_status();
    }
    // no (or too small a) workspace: one workgroup does it all
    hipLaunchKernelGGL(topk_select_kernel, dim3(1), dim3(kThreads), 0, st, score,
                       (int)n, (int)k, idx_out);
    return launch_status();
}

}  // namespace pkv
