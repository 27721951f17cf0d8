// The rest of a pre-norm decoder layer for the rows that are carried through the model
// (paper: Sec. 4.2, the user query against the imprecise cache; Sec. 4.3 and Appendix E,
// the selected and the query rows through every layer): RMS normalisation of gathered
// rows, a linear layer with an optional residual, and the gated up-projection of the
// MLP.  The block is the public Llama one; the paper does not restate it.
//
// bf16 linear layers of MFMA-friendly sizes run on the 256 x 256 tile kernel of the
// Q/K/V projection with a different epilogue (gather_qkv_proj_dma.hip), fp32 ones on the fp32
// matrix-core kernel (f32_kernels.hip); everything else (odd bf16 sizes, unaligned pointers)
// takes the simple kernels below, one wave per output element.
#include <cmath>

#include "f32_kernels.h"
#include "proj_common.h"

namespace pkv {

namespace {

__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// ---- RMS normalisation: one wave per row, 16 bytes per lane and step ---------------
// The row is read twice (sum of squares, then scaling); the second read comes out of
// the cache.  Rows of up to 8 steps per lane (8 KB: hidden 4096 in bf16) stay in
// registers instead.
// A = RowAngles: also the row's line of the table of angles that the projection of the normalised rows
// reads, one (cos, sin) per lane, worked out under the latency of the row.  A launch of its own is
// 4.6 us for 512 rows of 64 angles and 3.0 for 2000; here it adds 3.0 and 1.3 to the row kernels.
struct NoAngles {};
__device__ __forceinline__ void row_angles(const NoAngles&, int, int, int) {}
__device__ __forceinline__ void row_angles(const RowAngles& a, int row, int first, int step) {
    for (int i = first; i < a.half; i += step) {
        float sn, c;
        rope_sincos((double)a.row_pos[row], a.tab.inv_freq[i], &sn, &c);
        a.cs[(int64_t)row * a.half + i] = make_float2(c, sn);
    }
}

template <typename T, bool IN_REGS, typename A>
__global__ __launch_bounds__(256) void rmsnorm_rows_kernel(const T* __restrict__ h,
                                                           const int32_t* __restrict__ row_idx,
                                                           const T* __restrict__ weight,
                                                           float eps, T* __restrict__ y,
                                                           int m, int hidden, A angles) {
    typedef typename Vec16<T>::type vec_t;
    constexpr int N = Vec16<T>::N;
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= m) return;
    const int64_t src = row_idx ? row_idx[row] : row;
    const vec_t* hp = reinterpret_cast<const vec_t*>(h + src * hidden);
    const vec_t* wp = reinterpret_cast<const vec_t*>(weight);
    vec_t* yp = reinterpret_cast<vec_t*>(y + (int64_t)row * hidden);
    const int n_chunks = hidden / N;
    float ss = 0.f;
    if (IN_REGS) {
        vec_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = i * 64 + lane;
            if (c < n_chunks) {
                v[i] = __builtin_nontemporal_load(hp + c);   // every row is read once
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    const float f = Elem<T>::to_f32(v[i][e]);
                    ss += f * f;
                }
            }
        }
        row_angles(angles, row, lane, 64);
        ss = wave_sum_f32(ss);
        const float r = 1.0f / sqrtf(ss / (float)hidden + eps);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = i * 64 + lane;
            if (c < n_chunks) {
                const vec_t w = wp[c];
                vec_t o;
#pragma unroll
                for (int e = 0; e < N; ++e)
                    o[e] = Elem<T>::from_f32(Elem<T>::to_f32(v[i][e]) * r * Elem<T>::to_f32(w[e]));
                __builtin_nontemporal_store(o, yp + c);
            }
        }
    } else {
        row_angles(angles, row, lane, 64);
        for (int c = lane; c < n_chunks; c += 64) {
            const vec_t v = hp[c];
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const float f = Elem<T>::to_f32(v[e]);
                ss += f * f;
            }
        }
        ss = wave_sum_f32(ss);
        const float r = 1.0f / sqrtf(ss / (float)hidden + eps);
        for (int c = lane; c < n_chunks; c += 64) {
            const vec_t v = hp[c];
            const vec_t w = wp[c];
            vec_t o;
#pragma unroll
            for (int e = 0; e < N; ++e)
                o[e] = Elem<T>::from_f32(Elem<T>::to_f32(v[e]) * r * Elem<T>::to_f32(w[e]));
            yp[c] = o;
        }
    }
}

// The same with a workgroup per row, the row in registers (up to 2048 pieces of 16 bytes): few
// rows are a chain of one load, one sum over the row and one store, and four waves make it a
// quarter as long.
template <typename T, typename A>
__global__ __launch_bounds__(256) void rmsnorm_few_kernel(const T* __restrict__ h,
                                                          const int32_t* __restrict__ row_idx,
                                                          const T* __restrict__ weight, float eps,
                                                          T* __restrict__ y, int hidden,
                                                          A angles) {
    typedef typename Vec16<T>::type vec_t;
    constexpr int N = Vec16<T>::N;
    __shared__ float s_sum[4];
    const int tid = threadIdx.x;
    const int row = blockIdx.x;
    const int64_t src = row_idx ? row_idx[row] : row;
    const vec_t* hp = reinterpret_cast<const vec_t*>(h + src * hidden);
    const vec_t* wp = reinterpret_cast<const vec_t*>(weight);
    vec_t* yp = reinterpret_cast<vec_t*>(y + (int64_t)row * hidden);
    const int n_chunks = hidden / N;
    vec_t v[8], w[8];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = i * 256 + tid;
        if (c < n_chunks) {
            v[i] = hp[c];
            w[i] = wp[c];
        }
    }
    row_angles(angles, row, tid, 256);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (i * 256 + tid < n_chunks) {
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const float f = Elem<T>::to_f32(v[i][e]);
                ss += f * f;
            }
        }
    ss = wave_sum_f32(ss);
    if ((tid & 63) == 0) s_sum[tid >> 6] = ss;
    __syncthreads();
    ss = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
    const float r = 1.0f / sqrtf(ss / (float)hidden + eps);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = i * 256 + tid;
        if (c < n_chunks) {
            vec_t o;
#pragma unroll
            for (int e = 0; e < N; ++e)
                o[e] = Elem<T>::from_f32(Elem<T>::to_f32(v[i][e]) * r * Elem<T>::to_f32(w[i][e]));
            yp[c] = o;
        }
    }
}

// ---- row gather: 16 bytes per lane ------------------------------------------------------
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4* __restrict__ src,
                                                          const int32_t* __restrict__ row_idx,
                                                          uint4* __restrict__ dst, int64_t total,
                                                          int chunks) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int64_t row = i / chunks;
    const int c = (int)(i - row * chunks);
    dst[i] = src[(int64_t)row_idx[row] * chunks + c];
}

// ---- simple linear layers: one wave per output element ----------------------------------
template <typename T>
__device__ __forceinline__ float wave_dot(const T* __restrict__ a, const T* __restrict__ b,
                                          int k, int lane) {
    float s = 0.f;
    for (int i = lane; i < k; i += 64) s += Elem<T>::load(a + i) * Elem<T>::load(b + i);
    return wave_sum_f32(s);
}

__device__ __forceinline__ float silu_ref(float a) { return a / (1.f + expf(-a)); }

template <typename T, bool GATED>
__global__ __launch_bounds__(256) void linear_simple_kernel(const T* __restrict__ x,
                                                            const T* __restrict__ w0,
                                                            const T* __restrict__ w1,
                                                            const T* residual, T* y, int64_t m,
                                                            int k_in, int n_out) {
    const int lane = threadIdx.x & 63;
    const int64_t o = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (o >= m * n_out) return;
    const int64_t row = o / n_out;
    const int f = (int)(o % n_out);
    const T* xr = x + row * k_in;
    const float a = wave_dot(xr, w0 + (int64_t)f * k_in, k_in, lane);
    float out;
    if (GATED) {
        const float b = wave_dot(xr, w1 + (int64_t)f * k_in, k_in, lane);
        const float ar = Elem<T>::to_f32(Elem<T>::from_f32(a));
        const float br = Elem<T>::to_f32(Elem<T>::from_f32(b));
        const float s = Elem<T>::to_f32(Elem<T>::from_f32(silu_ref(ar)));
        out = s * br;
    } else {
        out = a;
        if (residual) out = Elem<T>::to_f32(Elem<T>::from_f32(a)) + Elem<T>::load(residual + o);
    }
    if (lane == 0) y[o] = Elem<T>::from_f32(out);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Whether a workgroup per row is the faster way: the row must give a wave more than one piece
// per lane, and a workgroup more than it has lanes where there are many rows.  Measured, wave per
// row -> workgroup per row (us): 4096 bf16, 64 rows 4.9 -> 2.8, 512 7.4 -> 3.4, 2048 9.6 -> 8.2, 3000
// 11.7 -> 12.4; 5120, 50 rows 5.7 -> 2.9, 870 8.9 -> 5.5; 1024, 256 rows 2.8 -> 2.5, 1500 3.8 -> 4.5; 256
// fp32 (one piece per lane), 883 rows 2.5 -> 2.9.
bool few_rows(int64_t m, int64_t chunks) {
    return chunks <= 2048 && (chunks >= 256 ? m <= 2048 : chunks > 64 && m <= 1024);
}

template <typename T, typename A>
pkv_status rmsnorm_typed(const void* h, const int32_t* row_idx, const void* weight, float eps,
                         void* y, int64_t m, int64_t hidden, const A& angles, hipStream_t st) {
    if (few_rows(m, hidden * (int64_t)sizeof(T) / 16)) {
        hipLaunchKernelGGL((rmsnorm_few_kernel<T, A>), dim3((unsigned)m), dim3(256), 0, st,
                           (const T*)h, row_idx, (const T*)weight, eps, (T*)y, (int)hidden, angles);
        return launch_status();
    }
    const dim3 blocks((unsigned)ceil_div(m, 4));
    const bool in_regs = hidden * (int64_t)sizeof(T) <= 8 * 64 * 16;
    if (in_regs)
        hipLaunchKernelGGL((rmsnorm_rows_kernel<T, true, A>), blocks, dim3(256), 0, st, (const T*)h,
                           row_idx, (const T*)weight, eps, (T*)y, (int)m, (int)hidden, angles);
    else
        hipLaunchKernelGGL((rmsnorm_rows_kernel<T, false, A>), blocks, dim3(256), 0, st, (const T*)h,
                           row_idx, (const T*)weight, eps, (T*)y, (int)m, (int)hidden, angles);
    return launch_status();
}

template <typename T>
pkv_status linear_simple(bool gated, const void* x, const void* w0, const void* w1,
                         const void* residual, void* y, int64_t m, int64_t k_in, int64_t n_out,
                         hipStream_t st) {
    const int64_t blocks = ceil_div(m * n_out, 4);
    if (blocks > 0x7fffffff) return PKV_ERR_SHAPE;
    if (gated)
        hipLaunchKernelGGL((linear_simple_kernel<T, true>), dim3((unsigned)blocks), dim3(256), 0,
                           st, (const T*)x, (const T*)w0, (const T*)w1, (const T*)nullptr, (T*)y,
                           m, (int)k_in, (int)n_out);
    else
        hipLaunchKernelGGL((linear_simple_kernel<T, false>), dim3((unsigned)blocks), dim3(256), 0,
                           st, (const T*)x, (const T*)w0, (const T*)nullptr, (const T*)residual,
                           (T*)y, m, (int)k_in, (int)n_out);
    return launch_status();
}

}  // namespace

pkv_status launch_rmsnorm_rows(int dtype, const void* h, const int32_t* row_idx,
                               const void* weight, float eps, void* y, int64_t m,
                               int64_t hidden, hipStream_t st, const RowAngles* angles) {
    if (!aligned16(h) || !aligned16(weight) || !aligned16(y)) return PKV_ERR_UNSUPPORTED;
    if (dtype == PKV_BF16 && angles)
        return rmsnorm_typed<bf16_t>(h, row_idx, weight, eps, y, m, hidden, *angles, st);
    return dtype == PKV_BF16
               ? rmsnorm_typed<bf16_t>(h, row_idx, weight, eps, y, m, hidden, NoAngles{}, st)
               : rmsnorm_typed<float>(h, row_idx, weight, eps, y, m, hidden, NoAngles{}, st);
}

pkv_status launch_gather_rows(int dtype, const void* src, const int32_t* row_idx, void* dst,
                              int64_t m, int64_t width, hipStream_t st) {
    if (!aligned16(src) || !aligned16(dst)) return PKV_ERR_UNSUPPORTED;
    const int chunks = (int)(width * (dtype == PKV_BF16 ? 2 : 4) / 16);
    const int64_t total = m * chunks;
    const int64_t blocks = ceil_div(total, 256);
    if (blocks > 0x7fffffff) return PKV_ERR_SHAPE;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       (const uint4*)src, row_idx, (uint4*)dst, total, chunks);
    return launch_status();
}

size_t glue_ws_bytes(int dtype, int64_t m, int64_t k_in, int64_t n_out) {
    if (dtype != PKV_BF16) return 0;
    if (!linear_dma_supported(kProjPlain, m, k_in, n_out) &&
        !linear_dma_supported(kProjGated, m, k_in, n_out))
        return 0;
    return linear_dma_partial_bytes(m);
}

pkv_status launch_linear_rows(int dtype, bool gated, const void* x, const void* w0,
                              const void* w1, const void* residual, void* y, int64_t m,
                              int64_t k_in, int64_t n_out, void* ws, hipStream_t st) {
    const int mode = gated ? kProjGated : kProjPlain;
    if (dtype == PKV_BF16 && linear_dma_supported(mode, m, k_in, n_out) && aligned16(x) &&
        aligned16(w0) && aligned16(y) && (!gated || aligned16(w1)) &&
        (!residual || aligned16(residual)))
        return launch_linear_dma(mode, (const bf16_t*)x, (const bf16_t*)w0, (const bf16_t*)w1,
                                 (const bf16_t*)residual, (bf16_t*)y, m, k_in, n_out, (float*)ws,
                                 st);
    if (dtype == PKV_F32 && linear_f32_supported(x, w0, w1, residual, y, m) &&
        linear_f32_pays(gated, m, k_in, n_out)) {
        F32GemmParams p = {};
        p.x = (const float*)x;
        p.w[0] = (const float*)w0; p.w[1] = (const float*)w1;
        p.out[0] = (float*)y;
        p.m = (int)m; p.k = (int)k_in; p.n_out = (int)n_out;
        p.residual = (const float*)residual;
        return launch_gemm_f32(gated ? kF32Gated : kF32Plain, p, RopeTable{}, st);
    }
    return dtype == PKV_BF16
               ? linear_simple<bf16_t>(gated, x, w0, w1, residual, y, m, k_in, n_out, st)
               : linear_simple<float>(gated, x, w0, w1, residual, y, m, k_in, n_out, st);
}

bool norm_swiglu_f32(const void* x, const void* norm_w, float eps, const void* w_gate,
                     const void* w_up, void* y, int64_t m, int64_t k_in, int64_t n_out,
                     hipStream_t st, pkv_status* status) {
    // what the two calls refuse goes to them
    if (m <= 0 || k_in <= 0 || n_out <= 0 || k_in % 8 || n_out % 8 || k_in > 16384 ||
        n_out > (1 << 30) || !(eps >= 0.f) || !std::isfinite(eps) || !x || !norm_w || !w_gate ||
        !w_up || !y || !aligned16(norm_w) || !linear_f32_supported(x, w_gate, w_up, nullptr, y, m))
        return false;
    F32GemmParams p = {};
    p.x = (const float*)x;
    p.w[0] = (const float*)w_gate; p.w[1] = (const float*)w_up;
    p.out[0] = (float*)y;
    p.m = (int)m; p.k = (int)k_in; p.n_out = (int)n_out;
    if (!norm_f32_pays(kF32Gated, p)) return false;
    p.norm_w = (const float*)norm_w;
    p.norm_eps = eps;
    *status = launch_gemm_f32(kF32Gated, p, RopeTable{}, st);
    return true;
}

}  // namespace pkv
