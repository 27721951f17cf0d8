// Single precision on the matrix cores: projection and linear layers, query score, attention.
// (The same steps as the bf16 kernels: Algorithm 1, both stages; Appendix E.)
//
// v_mfma_f32_16x16x4_f32 multiplies and adds in fp32, so nothing is given up against plain
// FMA kernels that sum in one chain (against the linear layers', which summed in parts, it is:
// those take the fp64 instruction, see below); what is gained is that one instruction does 1024
// multiply-adds without moving operands.  fp32 problems here are small (a 1k-token request is
// 0.2 GFLOP, 2 us of the fp32 matrix rate), so all of these kernels are bound by latency: the
// launch, and the chain of memory round trips inside it.  Each is therefore cut so that a wave
// makes few round trips, all operands of one requested together, and enough waves run at once to
// cover the chip.
//
// Operand layout of the instruction: A lane l holds row l % 16, contraction index l / 16; B
// likewise with columns; the accumulator of lane l holds column l % 16, rows 4 (l / 16) + r.
// The contraction may run in any order as long as A and B agree, so lane group g = l / 16 takes
// indices 4 g .. 4 g + 3 of every 16 (one 16-byte load) and step j uses element j of all.
//
// Measured, 1024 context tokens, 16 query tokens, 4 heads of 64 (us, plain kernels -> these):
// attention of 220 rows 105 -> 19, column sums 158 -> 5.7, normalisers 13 -> 4.3,
// projection of 220 rows 34 -> 6.7; linear layers of 151 rows, 256 -> 512 gated 21 -> 5.9,
// 512 -> 256 10.3 -> 6.5.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "f32_kernels.h"

#include "attn_common.h"

namespace pkv {

namespace {

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4 mfma_f64(float a, float b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64((double)a, (double)b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// ---- projection and linear layers ----------------------------------------------------------
// A workgroup (4 waves) computes 64 rows x 32 output columns, a wave 16 rows x 32 columns as
// two accumulators.  The 32 columns are two sets of 16 whose members meet in one lane and
// register: rotary partners (i, i + D/2), gate and up of one output, or simply the next 16
// outputs.  The contraction runs in chunks of 128 through LDS; the next chunk is on its way in
// registers while one is multiplied.  Rows of LDS are 132 floats apart: the 16 rows of an
// operand read start 4 banks apart and cover all 64 once.
constexpr int kTM = 64, kTN = 32, kTK = 128;
constexpr int kRow = kTK + 4;

// Sums.  The projection sums in fp32, one product behind the other in each of its KS parts of
// the contraction (3e-7 off the fp64 result at 256 inputs with one, 1.5e-7 with four).  The
// plain linear layers summed 64 interleaved parts and then these in a tree: 0.6 to 1.2e-7 off
// the fp64 result (2-norm, 64 to 4096 inputs), where one chain is 0.9 to 8.4e-7 off.  So they
// sum in fp64 here (v_mfma_f64_16x16x4_f64, at half the rate; products of fp32 are exact in it)
// and round once: 0.3e-7 at any length.  Its accumulator register r of lane group g is row g + 4
// r, not 4 g + r, so the weight rows go in permuted and the outputs come out alike.
//
// KS = 4, where all tiles then run at once: a tile of 16 rows whose four waves share the
// contraction and meet in LDS - four times the workgroups, a quarter of the chain (linear layers,
// 151 rows, 256 -> 512: 8.5 us with KS = 1, 4.4 with 4; 400 rows, 512 -> 1024: 14.8 and 14.1;
// projection, 4 heads of 64, 256 inputs: 16 rows 6.4 and 4.4, 220 rows 6.7 and 5.3; 8 heads of 64,
// 1024 inputs, 64 rows: 16.5 and 8.3; with more tiles the higher ones' better use of the weights
// wins, gemm_f32_low).
template <int KS>
constexpr int kTileRows = kTM / KS;

// NORM: the rows are RMS-normalised on their way into LDS.  The workgroup first goes over its rows for
// the sums of squares; for short rows that costs less than a launch of its own for the rows and
// their round trip (norm_f32_pays).
template <int MODE, int KS, bool NORM>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32GemmParams p, RopeTable tab) {
    constexpr int TM = kTileRows<KS>, kLoads = (TM + kTN) / 8;
    constexpr bool kWide = MODE != kF32Rope;
    typedef typename std::conditional<kWide, f64x4, f32x4>::type acc_t;
    __shared__ __align__(32) float lds[(TM + kTN) * kRow];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int g4 = lane >> 4, l16 = lane & 15;
    const int row0 = blockIdx.y * TM;

    // weight row of column c of this tile (c < 16: first set, else its partner)
    int mat = 0, ct = blockIdx.x;
    if (MODE == kF32Rope) {
        if (ct >= p.tile_begin[1]) mat = 1;
        if (ct >= p.tile_begin[2]) mat = 2;
        ct -= p.tile_begin[mat];
    }
    const int half = p.d / 2;
    // index of the first set's column c: pair index, output index
    auto col_of = [&](int c) { return ct * (MODE == kF32Plain ? 32 : 16) + c; };
    const int n_cols = MODE == kF32Rope ? (mat == 0 ? p.hq : p.hkv) * half : p.n_out;
    auto w_row = [&](int c) -> const float* {
        int j = col_of(c & 15);
        if (MODE == kF32Plain) {
            j = min(j + (c & 16), n_cols - 1);
            return p.w[0] + (int64_t)j * p.k;
        }
        j = min(j, n_cols - 1);
        if (MODE == kF32Gated) return (c & 16 ? p.w[1] : p.w[0]) + (int64_t)j * p.k;
        const int head = j / half, i = j % half;
        return p.w[mat] + (int64_t)(head * p.d + i + (c & 16 ? half : 0)) * p.k;
    };

    // loader: TM + 32 rows of 32 16-byte pieces; thread t takes piece t % 32 of rows t / 32 + 8 n
    const int piece = tid & 31, r0 = tid >> 5;
    const float* src[kLoads];
#pragma unroll
    for (int n = 0; n < kLoads; ++n) {
        const int r = r0 + 8 * n;
        if (r < TM) {
            const int row = min(row0 + r, p.m - 1);
            src[n] = p.x + (int64_t)(p.row_idx ? p.row_idx[row] : row) * p.k;
        } else {
            src[n] = w_row(r - TM);
        }
    }
    f32x4 st[kLoads], gain;
    auto load = [&](int k0) {
        const int k = k0 + piece * 4;
#pragma unroll
        for (int n = 0; n < kLoads; ++n)
            st[n] = k < p.k ? ld4(src[n] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
        if (NORM) gain = k < p.k ? ld4(p.norm_w + k) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    acc_t acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    const int w16 = kWide ? 4 * (l16 & 3) + (l16 >> 2) : l16;
    load(0);
    float rnorm[TM / 8];   // of rows r0 + 8 n
    if (NORM) {
#pragma unroll
        for (int n = 0; n < TM / 8; ++n) {
            float ss = 0.f;
            for (int k = piece * 4; k < p.k; k += kTK) {
                const f32x4 v = ld4(src[n] + k);
                ss += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
            }
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);   // a row's 32 threads
            rnorm[n] = 1.0f / sqrtf(ss / (float)p.k + p.norm_eps);
        }
    }
    for (int k0 = 0; k0 < p.k; k0 += kTK) {
        if (NORM) {
#pragma unroll
            for (int n = 0; n < TM / 8; ++n) st[n] = st[n] * rnorm[n] * gain;
        }
        __syncthreads();
#pragma unroll
        for (int n = 0; n < kLoads; ++n)
            *reinterpret_cast<f32x4*>(lds + (r0 + 8 * n) * kRow + piece * 4) = st[n];
        __syncthreads();
        if (k0 + kTK < p.k) load(k0 + kTK);
        const int part = KS == 1 ? 0 : wave * (kTK / KS);   // of the chunk
        const float* xb = lds + ((KS == 1 ? wave * 16 : 0) + l16) * kRow + g4 * 4 + part;
        const float* wb = lds + (TM + w16) * kRow + g4 * 4 + part;
#pragma unroll
        for (int c = 0; c < kTK / KS / 16; ++c) {
            const f32x4 b = ld4(xb + c * 16), a0 = ld4(wb + c * 16),
                        a1 = ld4(wb + 16 * kRow + c * 16);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (kWide) {
                    acc[0] = mfma_f64(a0[j], b[j], acc[0]);
                    acc[1] = mfma_f64(a1[j], b[j], acc[1]);
                } else {
                    acc[0] = mfma_f32(a0[j], b[j], acc[0]);
                    acc[1] = mfma_f32(a1[j], b[j], acc[1]);
                }
            }
        }
    }

    if constexpr (KS > 1) {
        acc_t* const ex = reinterpret_cast<acc_t*>(lds);   // [wave - 1][set][lane]
        static_assert((KS - 1) * 2 * 64 * sizeof(acc_t) <= sizeof(lds), "");
        __syncthreads();
        if (wave > 0) {
            ex[(wave * 2 - 2) * 64 + lane] = acc[0];
            ex[(wave * 2 - 1) * 64 + lane] = acc[1];
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int w = 0; w < 2 * (KS - 1); ++w) acc[w & 1] += ex[w * 64 + lane];
    }
    // a lane holds row l16 of the wave, columns 4 g4 + r of both sets
    const int row = row0 + (KS == 1 ? wave * 16 : 0) + l16;
    if (row >= p.m) return;
    const int c0 = col_of(4 * g4);
    f32x4 sum[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[s][r] = (float)acc[s][r];
    if (MODE == kF32Plain) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int f = c0 + 16 * s;
            if (f >= n_cols) continue;             // n_out is a multiple of 8
            const int64_t o = (int64_t)row * p.n_out + f;
            f32x4 v = sum[s];
            if (p.residual) v += ld4(p.residual + o);
            *reinterpret_cast<f32x4*>(p.out[0] + o) = v;
        }
    } else if (MODE == kF32Gated) {
        if (c0 >= n_cols) return;
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = sum[0][r] / (1.f + expf(-sum[0][r])) * sum[1][r];
        *reinterpret_cast<f32x4*>(p.out[0] + (int64_t)row * p.n_out + c0) = v;
    } else {
        if (c0 >= n_cols) return;                  // half is a multiple of 8
        const int head = c0 / half, i0 = c0 % half;
        const int heads = mat == 0 ? p.hq : p.hkv;
        const int64_t orow = mat != 0 && p.dst_row ? p.dst_row[row] : row;
        float* o = p.out[mat] + (orow * heads + head) * p.d + i0;
        f32x4 a = sum[0], b = sum[1];
        if (p.bias[mat]) {
            a += ld4(p.bias[mat] + head * p.d + i0);
            b += ld4(p.bias[mat] + head * p.d + i0 + half);
        }
        if (mat != 2) {
            const double pos = (double)p.row_pos[row];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float sn, cs;
                rope_sincos(pos, tab.inv_freq[i0 + r], &sn, &cs);
                const float ra = a[r] * cs - b[r] * sn, rb = b[r] * cs + a[r] * sn;
                a[r] = ra;
                b[r] = rb;
            }
        }
        *reinterpret_cast<f32x4*>(o) = a;
        *reinterpret_cast<f32x4*>(o + half) = b;
    }
}

// ---- shared by score and attention -----------------------------------------------------------
// S of 16 keys x 16 columns: k4[c] = key (lane % 16), elements 16 c + 4 g4 ..; q4 likewise
template <int D>
__device__ __forceinline__ f32x4 dot_tile(const f32x4 (&k4)[D / 16], const f32x4 (&q4)[D / 16]) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / 16; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (c & 1) s2 = mfma_f32(k4[c][j], q4[c][j], s2);   // two chains: half the latency
            else s = mfma_f32(k4[c][j], q4[c][j], s);
        }
    return s + s2;
}
template <int D>
__device__ __forceinline__ void load_row(f32x4 (&dst)[D / 16], const float* row, int g4) {
#pragma unroll
    for (int c = 0; c < D / 16; ++c) dst[c] = ld4(row + c * 16 + 4 * g4);
}
__device__ __forceinline__ float col_max(float v) {   // over the lane groups of a column
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float col_sum(float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// ---- attention ---------------------------------------------------------------------------------
// A workgroup owns 16 (row, head) columns of one kv head; its NW waves take every NW-th tile of
// 16 keys, each with a running maximum of its own, and meet in LDS at the end.  The scores of a
// lane (keys 4 g4 + r of its column) are the B operand of the second product as they are: step
// j multiplies key 4 g4 + j of every lane group.  Row i of output block e is element C i + e of
// the head, so that a lane's piece of a value row is C = D / 16 consecutive floats (one element
// per load instead took 16 loads per tile and as long as the multiplications).  K and V of the
// next tile are requested before the current one is used.
//
// S > 1, where all of them still have a CU of their own: S workgroups per tile of columns, each with its
// C / S elements of every value row and all of the scores.  The two products, alike in size, are what
// a workgroup spends its time on, so four take towards 5/8 of it, with the same bits and no parts to be
// merged (us, 220 rows: 4 heads of 64, 1040 keys 19.4 -> 17.7, 4096 57.7 -> 50.8; 8 / 2 heads of 128,
// where two share, 1040 keys 33.7 -> 26.5; 64 rows of them, four, 33.2 -> 24.1; 4 / 2 of 32 13.2 -> 12.0).
constexpr int kColRow = 17;   // the merge reads down the columns: 16 would be 16 lanes to a bank
template <int D, int NW, int S>
__global__ __launch_bounds__(NW * 64) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
    const int32_t* __restrict__ row_pos, float* __restrict__ out, float* __restrict__ lse_out,
    int m_all, int hq, int hkv, float scale, int chunk_len) {
    constexpr int C = D / 16, CS = C / S, DS = D / S;
    extern __shared__ __align__(16) float smem[];      // [NW][DS][16] partial outputs, rows of 17
    __shared__ float s_m[NW][16], s_l[NW][16], s_f[NW][16], s_top[16];
    __shared__ int s_out[16];   // (row, head) of a column, -1: none
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int g4 = lane >> 4, l16 = lane & 15;
    const int g = blockIdx.y, group = hq / hkv;
    const int part = blockIdx.x % S;
    const int tile = (gridDim.x - 1 - blockIdx.x) / S; // rows in position order: heavy ones first
    // rows and keys of chunk blockIdx.z start at row0 (one chunk: the keys are a cache of their own)
    const int row0 = (int)blockIdx.z * chunk_len;
    const int m = min(m_all, row0 + chunk_len);
    const int col = tile * 16 + l16;
    const int row = row0 + col / group, head = g * group + col % group;
    const bool valid = row < m;
    const int limit = valid ? row_pos[row] : -1;
    int last = limit;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o, 64));

    f32x4 q4[C];
    load_row<D>(q4, q + ((int64_t)(valid ? row : 0) * hq + head) * D, g4);
    const int64_t krow = (int64_t)hkv * D;
    const float* kb = kc + row0 * krow + (int64_t)g * D;
    const float* vb = vc + row0 * krow + (int64_t)g * D + C * l16 + CS * part;
    typedef float vrow_t __attribute__((ext_vector_type(CS)));
    f32x4 k4[C], kn[C], o_acc[CS];
    vrow_t v4[4], vn[4];
#pragma unroll
    for (int c = 0; c < CS; ++c) o_acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, sum = 0.f;
    // keys beyond the tile's last visible one are never needed: re-read that one instead
    auto load_kv = [&](int t0) {
        load_row<D>(kn, kb + (int64_t)min(t0 + l16, last) * krow, g4);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            vn[j] = *reinterpret_cast<const vrow_t*>(vb + (int64_t)min(t0 + 4 * g4 + j, last) * krow);
    };
    int t0 = wave * 16;
    if (t0 <= last) load_kv(t0);
    for (; t0 <= last; t0 += NW * 16) {
#pragma unroll
        for (int c = 0; c < C; ++c) k4[c] = kn[c];
#pragma unroll
        for (int j = 0; j < 4; ++j) v4[j] = vn[j];
        if (t0 + NW * 16 <= last) load_kv(t0 + NW * 16);
        f32x4 s = dot_tile<D>(k4, q4);
        float tm = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = t0 + 4 * g4 + r <= limit ? s[r] * scale : -INFINITY;
            tm = fmaxf(tm, s[r]);
        }
        const float mn = fmaxf(mx, col_max(tm));
        const float ref = mn == -INFINITY ? 0.f : mn;
        const float corr = expf(mx - ref);
        float ts = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = expf(s[r] - ref);
            ts += s[r];
        }
        sum = sum * corr + ts;       // this lane group's keys only
        mx = mn;
#pragma unroll
        for (int c = 0; c < CS; ++c) o_acc[c] *= corr;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < CS; ++c) o_acc[c] = mfma_f32(v4[j][c], s[j], o_acc[c]);
    }
    sum = col_sum(sum);
    if (g4 == 0) {
        s_m[wave][l16] = mx;
        s_l[wave][l16] = sum;
    }
#pragma unroll
    for (int c = 0; c < CS; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            smem[(wave * DS + CS * (4 * g4 + r) + c) * kColRow + l16] = o_acc[c][r];
    __syncthreads();
    if (tid < NW * 16) {        // the weight of every wave's part
        const int w = tid >> 4, cc = tid & 15;
        float mm = -INFINITY;
#pragma unroll
        for (int v = 0; v < NW; ++v) mm = fmaxf(mm, s_m[v][cc]);
        s_f[w][cc] = expf(s_m[w][cc] - mm);
        if (w == 0) {                                   // (this lane's own column: cc = l16)
            s_top[cc] = mm;
            s_out[cc] = valid ? row * hq + head : -1;
        }
    }
    __syncthreads();
#pragma unroll
    for (int e0 = 0; e0 < DS * 16; e0 += NW * 64) {
        const int e = e0 + tid;
        if (DS * 16 % (NW * 64) && e >= DS * 16) break;   // few elements on 16 waves
        const int cc = e / DS, es = e % DS;
        const int dd = es / CS * C + CS * part + es % CS;   // element of the head
        const int64_t oc = s_out[cc];
        if (oc < 0) continue;
        float acc = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = s_f[w][cc];
            acc += f * smem[(w * DS + es) * kColRow + cc];
            l += f * s_l[w][cc];
        }
        out[oc * D + dd] = acc / l;
        if (lse_out && dd == 0) lse_out[oc] = s_top[cc] + logf(l);
    }
}

// ---- query score ---------------------------------------------------------------------------------
// Columns of a kv head are numbered (query token, head of the group), in tiles of 16.
// Pass 1: per column the (maximum, sum) over a range of keys; four waves per workgroup take
// every fourth tile of 16 keys and meet in LDS.  With one range that is the column's normaliser,
// and it goes out as such (lse, then part is not used).
template <int D>
__global__ __launch_bounds__(256) void score_part_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, float2* __restrict__ part,
    float* __restrict__ lse, int nq,
    int n_ctx, int hq, int hkv, int split_len, float scale) {
    constexpr int C = D / 16;
    __shared__ float s_m[4][16], s_l[4][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g4 = lane >> 4, l16 = lane & 15;
    const int g = blockIdx.y, group = hq / hkv;
    const int col = blockIdx.x * 16 + l16;
    const int n_col = nq * group;
    const int cc = min(col, n_col - 1);
    const int64_t qcol = (int64_t)(cc / group) * hq + g * group + cc % group;
    const int begin = blockIdx.z * split_len, end = min(n_ctx, begin + split_len);
    f32x4 q4[C], k4[C];
    load_row<D>(q4, q + qcol * D, g4);
    const float* kb = k + (int64_t)g * D;
    const int64_t krow = (int64_t)hkv * D;
    float mx = -INFINITY, sum = 0.f;
    int t0 = begin + wave * 16;
    if (t0 < end) load_row<D>(k4, kb + (int64_t)min(t0 + l16, end - 1) * krow, g4);
    for (; t0 < end; t0 += 64) {
        f32x4 s = dot_tile<D>(k4, q4);
        if (t0 + 64 < end)
            load_row<D>(k4, kb + (int64_t)min(t0 + 64 + l16, end - 1) * krow, g4);
        float mn = mx;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = t0 + 4 * g4 + r < end ? s[r] * scale : -INFINITY;
            mn = fmaxf(mn, s[r]);
        }
        const float ref = mn == -INFINITY ? 0.f : mn;   // this lane's own reference
        float ts = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) ts += expf(s[r] - ref);
        sum = sum * expf(mx - ref) + ts;
        mx = mn;
    }
    const float m = col_max(mx);
    sum = col_sum(m == -INFINITY ? 0.f : sum * expf(mx - m));
    if (g4 == 0) {
        s_m[wave][l16] = m;
        s_l[wave][l16] = sum;
    }
    __syncthreads();
    if (threadIdx.x < 16 && col < n_col) {
        float mm = -INFINITY, l = 0.f;
        for (int w = 0; w < 4; ++w) mm = fmaxf(mm, s_m[w][l16]);   // finite: the range has keys
        for (int w = 0; w < 4; ++w) l += s_l[w][l16] * expf(s_m[w][l16] - mm);
        if (lse) lse[qcol] = mm + logf(l);
        else part[(int64_t)blockIdx.z * nq * hq + qcol] = make_float2(mm, l);
    }
}

// Pass 2: the sum over all columns per key.  A workgroup owns 16 keys; its four waves take every
// fourth tile of columns and meet in LDS.  Columns come in blocks of 256 whose normalisers the
// workgroup folds (part) or reads (lse) into LDS first.  Fixed order, no atomics.
// With row_pos a query row counts for the keys up to row_pos[row] only.
template <int D>
__global__ __launch_bounds__(256) void score_sum_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float2* __restrict__ part,
    int n_splits, const float* __restrict__ lse, const int32_t* __restrict__ row_pos,
    float* __restrict__ score, int nq, int n_ctx, int hq, int hkv, float scale, int accumulate) {
    constexpr int C = D / 16;
    __shared__ float s_lse[256];
    __shared__ float s_sum[4][16];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int g4 = lane >> 4, l16 = lane & 15;
    const int group = hq / hkv, n_col = nq * group, ncol = nq * hq;
    const int tiles_g = (n_col + 15) / 16, tiles = tiles_g * hkv;
    const int t0 = blockIdx.x * 16;
    auto qcol_of = [&](int tile, int c) -> int {      // -1 past the last column of the kv head
        const int cc = (tile % tiles_g) * 16 + c;
        return cc < n_col ? (cc / group) * hq + (tile / tiles_g) * group + cc % group : -1;
    };
    const float* krow = k + (int64_t)min(t0 + l16, n_ctx - 1) * hkv * D;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    f32x4 k4[C], q4[C];
    for (int tb = 0; tb < tiles; tb += 16) {
        if (tb) __syncthreads();
        // operands of the wave's first tile, requested before the fold below
        const bool any = tb + wave < tiles;
        if (any) {
            load_row<D>(k4, krow + (int64_t)((tb + wave) / tiles_g) * D, g4);
            load_row<D>(q4, q + (int64_t)max(qcol_of(tb + wave, l16), 0) * D, g4);
        }
        {
            const int tile = tb + (tid >> 4);
            const int qc = tile < tiles ? qcol_of(tile, tid & 15) : -1;
            float v = INFINITY;                       // switches the column off
            if (qc >= 0) {
                if (lse) {
                    v = lse[qc];
                } else {
                    float m = -INFINITY, l = 0.f;
                    for (int s = 0; s < n_splits; s += 8) {
                        float2 ml[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e)   // past the end: the last one, weight 0
                            ml[e] = part[(int64_t)min(s + e, n_splits - 1) * ncol + qc];
                        float mn = m;
#pragma unroll
                        for (int e = 0; e < 8; ++e) mn = fmaxf(mn, ml[e].x);
                        l *= expf(m - mn);
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            l += s + e < n_splits ? ml[e].y * expf(ml[e].x - mn) : 0.f;
                        m = mn;
                    }
                    v = m + logf(l);
                }
            }
            s_lse[tid] = v;
        }
        __syncthreads();
        const int te = min(tiles, tb + 16);
        for (int tile = tb + wave; tile < te; tile += 4) {
            const f32x4 s = dot_tile<D>(k4, q4);
            const float norm = s_lse[(tile - tb) * 16 + l16];
            const int lim = row_pos ? row_pos[max(qcol_of(tile, l16), 0) / hq] : n_ctx;
            if (tile + 4 < te) {
                if ((tile + 4) / tiles_g != tile / tiles_g)
                    load_row<D>(k4, krow + (int64_t)((tile + 4) / tiles_g) * D, g4);
                load_row<D>(q4, q + (int64_t)max(qcol_of(tile + 4, l16), 0) * D, g4);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + 4 * g4 + r <= lim) acc[r] += expf(s[r] * scale - norm);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float v = acc[r];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
        if (l16 == 0) s_sum[wave][4 * g4 + r] = v;
    }
    __syncthreads();
    const int t = t0 + tid;
    if (tid < 16 && t < n_ctx) {
        const float v = ((s_sum[0][tid] + s_sum[1][tid]) + (s_sum[2][tid] + s_sum[3][tid])) /
                        (float)ncol;
        score[t] = accumulate ? score[t] + v : v;
    }
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <int D, int NW, int S>
pkv_status attn_f32_launch(dim3 grid, const float* q, const float* k, const float* v,
                           const int32_t* row_pos, float* out, float* lse, int64_t m, int hq,
                           int hkv, float scale, int chunk_len, hipStream_t st) {
    constexpr size_t kBytes = (size_t)NW * (D / S) * kColRow * sizeof(float);
    grid.x *= S;
    static std::atomic<bool> configured{false};   // set twice at worst: the calls are idempotent
    if (!configured.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_f32_kernel<D, NW, S>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kBytes) != hipSuccess)
            return PKV_ERR_LAUNCH;
        configured.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((attn_f32_kernel<D, NW, S>), grid, dim3(NW * 64), kBytes, st, q, k, v, row_pos,
                       out, lse, (int)m, hq, hkv, scale, chunk_len);
    return launch_status();
}

}  // namespace

bool f32_tiles_supported(const pkv_layer_cfg& cfg) {
    return cfg.dtype == PKV_F32 &&
           (cfg.head_dim == 32 || cfg.head_dim == 64 || cfg.head_dim == 128);
}

namespace {

int gemm_f32_column_tiles(int mode, const F32GemmParams& p) {
    return mode == kF32Rope ? p.tile_begin[3]
                            : (int)ceil_div(p.n_out, mode == kF32Plain ? 32 : 16);
}
// Tiles of 16 rows, where they all run at once (four workgroups per CU).  The projection, whose fp32
// products are half as long as the linear layers' fp64 ones, takes a fourth one per CU only where its
// tiles of 64 rows would be more than one per CU (64 rows -> 16, us: 1024 inputs, 768 tiles 16.8 -> 14.7,
// 832 16.8 -> 18.0, 864 in place of 288 25.1 -> 18.1; 256 inputs, 768 6.9 -> 6.6, 864 7.0 -> 7.5; 4096,
// 768 56.8 -> 46.8, 960 56.5 -> 59.0).
bool gemm_f32_low(int mode, const F32GemmParams& p) {
    const int64_t columns = gemm_f32_column_tiles(mode, p);
    const int64_t tiles = ceil_div(p.m, kTileRows<4>) * columns;
    return tiles <= 768 ||
           (tiles <= 1024 && (mode != kF32Rope || ceil_div(p.m, kTM) * columns > 256));
}

}  // namespace

// Every tile of columns goes over the rows again for their sums of squares.  On tiles of 16 rows that is
// two chains of k / 128 loads per thread, against 3 us for a launch of its own (normalisation and
// products apart -> together, us, a projection of K and V / of Q, K and V in a layer call: 256
// inputs, 209 rows 15.6 -> 13.1 / 18.7 -> 17.6, 768 inputs, 65 rows 15.5 -> 13.1 / 18.8 -> 17.2; 1024,
// 25 rows 15.7 -> 13.2 / 20.1 -> 22.3; 2048, 13 rows 17.0 -> 19.1 / 23.4 -> 28.5).  Tiles of 64 rows make
// eight such chains (256 inputs, 1261 rows 41 -> 45; 2048, 761 rows, K and V 54 -> 89).  The gated layer
// has twice the weights to come behind the chain: whole layers of 256 inputs, 26 rows 27.6 -> 25.6, 145
// rows 32.5 -> 31.5, of 384, 36 rows 34.3 -> 33.5, of 512 31 -> 32 at 2 rows and level at 3 to 51.
bool norm_f32_pays(int mode, const F32GemmParams& p) {
    return p.k <= (mode == kF32Rope ? 768 : 384) && gemm_f32_low(mode, p);
}

pkv_status launch_gemm_f32(int mode, const F32GemmParams& p, const RopeTable& tab, hipStream_t st) {
    const bool low = gemm_f32_low(mode, p);
    const int64_t rows = ceil_div(p.m, low ? kTileRows<4> : kTM);
    if (rows > 65535) return PKV_ERR_SHAPE;
    if (p.norm_w && (!low || mode == kF32Plain)) return PKV_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)gemm_f32_column_tiles(mode, p), (unsigned)rows);
#define PKV_GEMM_F32(MODE, KS, NORM)                                                             \
    hipLaunchKernelGGL((gemm_f32_kernel<MODE, KS, NORM>), grid, dim3(256), 0, st, p, tab)
    if (mode == kF32Rope && p.norm_w) PKV_GEMM_F32(kF32Rope, 4, true);
    else if (mode == kF32Rope && low) PKV_GEMM_F32(kF32Rope, 4, false);
    else if (mode == kF32Rope) PKV_GEMM_F32(kF32Rope, 1, false);
    else if (mode == kF32Plain && low) PKV_GEMM_F32(kF32Plain, 4, false);
    else if (mode == kF32Plain) PKV_GEMM_F32(kF32Plain, 1, false);
    else if (p.norm_w) PKV_GEMM_F32(kF32Gated, 4, true);
    else if (low) PKV_GEMM_F32(kF32Gated, 4, false);
    else PKV_GEMM_F32(kF32Gated, 1, false);
#undef PKV_GEMM_F32
    return launch_status();
}

bool linear_f32_supported(const void* x, const void* w0, const void* w1, const void* residual,
                          const void* y, int64_t m) {
    return ceil_div(m, kTM) <= 65535 && aligned16(x) && aligned16(w0) && aligned16(w1) &&
           aligned16(residual) && aligned16(y);
}

// us of a launch: a wave per output takes about 1e-4 + 2.2e-7 k_in per output (and, where the
// weights no longer stay in a cache, 0.004 per input beyond 1024), the tiles 0.0083 per input
// while they run at once.  Measured, wave per output against tiles of 16 rows: 256 x 512, 16 rows 3.5
// / 4.4, 64 rows 7.4 / 4.4; 512 x 256, 64 rows 5.6 / 6.5, 110 rows 8.2 / 6.5; 1024 x 4096, 4 rows
// 7.4 / 11.1, 16 rows 23 / 11; 4096 x 1024, 7 rows 21 / 36, 32 rows 74 / 36.
bool linear_f32_pays(bool gated, int64_t m, int64_t k_in, int64_t n_out) {
    const double k = (double)k_in;
    const double per_output = (double)m * (double)n_out * (1.0e-4 + 2.2e-7 * k) +
                              0.004 * std::max(0.0, k - 1024.0);
    return per_output * (gated ? 2.0 : 1.0) >= 0.45 + 0.0083 * k;
}

pkv_status launch_attn_f32(const pkv_layer_cfg& cfg, const float* q, const float* k,
                           const float* v, const int32_t* row_pos, float* out, float* lse,
                           int64_t m, int64_t n_keys, float scale, hipStream_t st,
                           int64_t chunk_len) {
    const int hq = cfg.n_q_heads, hkv = cfg.n_kv_heads;
    if (chunk_len <= 0) chunk_len = m;
    const dim3 grid((unsigned)ceil_div(chunk_len * (hq / hkv), 16), (unsigned)hkv,
                    (unsigned)ceil_div(m, chunk_len));
    // as many waves as their registers allow: 16 up to head_dim 64, 8 with 128; four where that
    // is a tile or two of keys each (head_dim 128: a tile), so that fewer parts have to be merged
    const bool few = n_keys <= (cfg.head_dim == 128 ? 64 : 128);
    // workgroups that share a tile of columns: as many as leave each a CU of its own (beyond, the scores
    // made again would take the time that the shorter products save).  One where the results replace
    // q: the others would still read the rows that the first one has written.
    const int64_t tiles = (int64_t)grid.x * grid.y * grid.z, n_cu = attn_cu_count();
    const int most = few || out == q ? 1 : 4 * tiles <= n_cu ? 4 : 2 * tiles <= n_cu ? 2 : 1;
#define PKV_ATTN_F32(D, NW, S)                                                                   \
    attn_f32_launch<D, NW, S>(grid, q, k, v, row_pos, out, lse, m, hq, hkv, scale, (int)chunk_len, st)
#define PKV_ATTN_F32_SHARED(D, NW)                                                               \
    (most == 4 && D > 32 ? PKV_ATTN_F32(D, NW, (D > 32 ? 4 : 2))                                 \
                         : most > 1 ? PKV_ATTN_F32(D, NW, 2) : PKV_ATTN_F32(D, NW, 1))
    if (cfg.head_dim == 32) return few ? PKV_ATTN_F32(32, 4, 1) : PKV_ATTN_F32_SHARED(32, 16);
    if (cfg.head_dim == 64) return few ? PKV_ATTN_F32(64, 4, 1) : PKV_ATTN_F32_SHARED(64, 16);
    return few ? PKV_ATTN_F32(128, 4, 1) : PKV_ATTN_F32_SHARED(128, 8);
#undef PKV_ATTN_F32_SHARED
#undef PKV_ATTN_F32
}

F32ScorePlan plan_score_f32(const pkv_layer_cfg& cfg, int64_t n_ctx, int64_t nq) {
    // about one workgroup per CU; every workgroup of pass 2 folds splits x columns partial
    // normalisers, 8192 at most (above that many columns there is one split, and nothing to fold:
    // it reads the normalisers)
    const int group = cfg.n_q_heads / cfg.n_kv_heads;
    const int64_t tiles = ceil_div(nq * group, 16) * cfg.n_kv_heads;
    int64_t want = std::min(ceil_div(256, tiles), ceil_div(n_ctx, 64));
    want = std::max<int64_t>(1, std::min(want, 8192 / std::max<int64_t>(1, nq * cfg.n_q_heads)));
    const int64_t len = ceil_div(ceil_div(n_ctx, want), 64) * 64;
    F32ScorePlan p;
    p.split_len = (int)len;
    p.n_splits = (int)ceil_div(n_ctx, len);
    return p;
}

size_t score_f32_ws_bytes(const pkv_layer_cfg& cfg, int64_t n_ctx, int64_t nq) {
    const int n_splits = plan_score_f32(cfg, n_ctx, nq).n_splits;
    return (size_t)(nq * cfg.n_q_heads) * sizeof(float) * (n_splits == 1 ? 1 : 2 * n_splits);
}

pkv_status launch_score_f32(const pkv_layer_cfg& cfg, const float* q, const float* k,
                            const float* lse, const int32_t* row_pos, float* score, int64_t nq,
                            int64_t n_ctx, float scale, int accumulate, void* ws,
                            hipStream_t st) {
    const int hq = cfg.n_q_heads, hkv = cfg.n_kv_heads, d = cfg.head_dim;
    const F32ScorePlan p = plan_score_f32(cfg, n_ctx, nq);
    float2* part = (float2*)ws;
    float* one = p.n_splits == 1 ? (float*)ws : nullptr;
    const dim3 g1((unsigned)ceil_div(nq * (hq / hkv), 16), (unsigned)hkv, (unsigned)p.n_splits);
    const dim3 g2((unsigned)ceil_div(n_ctx, 16));
#define PKV_SCORE_F32(DD)                                                                   \
    {                                                                                       \
        if (!lse)                                                                           \
            hipLaunchKernelGGL(score_part_f32_kernel<DD>, g1, dim3(256), 0, st, q, k, part, \
                               one, (int)nq, (int)n_ctx, hq, hkv, p.split_len, scale);      \
        hipLaunchKernelGGL(score_sum_f32_kernel<DD>, g2, dim3(256), 0, st, q, k, part,      \
                           p.n_splits, lse ? lse : one, row_pos, score, (int)nq,            \
                           (int)n_ctx, hq, hkv, scale, accumulate);                         \
    }
    if (d == 32) PKV_SCORE_F32(32)
    else if (d == 64) PKV_SCORE_F32(64)
    else PKV_SCORE_F32(128)
#undef PKV_SCORE_F32
    return launch_status();
}

}  // namespace pkv
