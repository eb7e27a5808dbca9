// LayerNorm of Eqs. (5),(6), Sec. 3.3: one wavefront per token row, the row held in
// registers, mean then variance of the deviations (population variance), fp32 statistics.
// Bound by one read and one write of the row.
#include "common.hpp"

namespace rs {

// Chunk `ch` (8 elements) of a row; zeros past its end.
__device__ __forceinline__ void row_load8(__amdgpu_buffer_rsrc_t row, int ch, const bf16raw*, float (&v)[8]) {
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(row, ch * 16, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void row_load8(__amdgpu_buffer_rsrc_t row, int ch, const float*, float (&v)[8]) {
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(row, ch * 32, 0, 0), b = __builtin_amdgcn_raw_buffer_load_b128(row, ch * 32 + 16, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = __uint_as_float(a[i]);
        v[4 + i] = __uint_as_float(b[i]);
    }
}

// MAXC = 8-element chunks a lane may hold: D <= MAXC * 64 * 8.
template <typename T, int MAXC>
__global__ __launch_bounds__(256) void layernorm_kernel(const T* __restrict__ x,
                                                        const T* __restrict__ gamma,
                                                        const T* __restrict__ beta,
                                                        T* __restrict__ out, int64_t M, int D, float eps,
                                                        int32_t* __restrict__ iota_out, int iota_n) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (row >= M) return;
    const int nchunk = D >> 3, bytes = D * (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t rs_x = row_rsrc(x + row * D, bytes);
    float v[MAXC][8];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) row_load8(rs_x, lane + c * 64, x, v[c]);
    // gamma and beta on the way while the statistics are formed, where the registers allow
    constexpr int EARLY = MAXC <= 2 ? MAXC : 0;
    float g[EARLY ? EARLY : 1][8], b[EARLY ? EARLY : 1][8];
    const __amdgpu_buffer_rsrc_t rs_g = row_rsrc(gamma, gamma ? bytes : 0), rs_b = row_rsrc(beta, beta ? bytes : 0);
#pragma unroll
    for (int c = 0; c < EARLY; ++c) {
        row_load8(rs_g, lane + c * 64, gamma, g[c]);
        row_load8(rs_b, lane + c * 64, beta, b[c]);
    }
    if (iota_out && lane == 0) iota_out[row] = (int32_t)(row % iota_n);
    const float2 st = wave_row_stats<MAXC>(v, nchunk, lane, D, eps);
    T* orow = out + row * D;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int ch = lane + c * 64, e = EARLY ? c : 0;
        if (!EARLY) {
            row_load8(rs_g, ch, gamma, g[0]);
            row_load8(rs_b, ch, beta, b[0]);
        }
        float r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float t = (v[c][i] - st.x) * st.y;
            if (gamma) t *= g[e][i];
            if (beta) t += b[e][i];
            r[i] = t;
        }
        if (ch < nchunk) Elem<T>::store8(orow + ch * 8, r);
    }
}

// Narrow rows (D <= 256): two rows per wave, 32 lanes each, the sums in the same order as above (the lanes
// missing there hold zeros).  12608 x 192 fp32: half of the waves, every lane of a row's first 24 busy.
template <typename T>
__global__ __launch_bounds__(256) void layernorm_narrow_kernel(const T* __restrict__ x, const T* __restrict__ gamma,
                                                               const T* __restrict__ beta, T* __restrict__ out, int64_t M,
                                                               int D, float eps, int32_t* __restrict__ iota_out, int iota_n) {
    const int lane = threadIdx.x & 63, sub = lane & 31;
    const int64_t row = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 2 + (lane >> 5);
    const bool on = row < M && sub < (D >> 3);  // whole waves stay in the shuffles below
    float v[8], g[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) { v[i] = 0.f; g[i] = 1.f; b[i] = 0.f; }
    if (on) {
        Elem<T>::load8(x + row * D + sub * 8, v);
        if (gamma) Elem<T>::load8(gamma + sub * 8, g);
        if (beta) Elem<T>::load8(beta + sub * 8, b);
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += v[i];
    sum = lanes_sum<32>(sum);
    const float mean = sum / (float)D;
    float sq = on ? chunk_sq(v, mean) : 0.f;
    sq = lanes_sum<32>(sq);
    const float inv = rsqrtf(sq / (float)D + eps);
    if (!on) return;
    if (iota_out && sub == 0) iota_out[row] = (int32_t)(row % iota_n);
    float r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float t = (v[i] - mean) * inv;
        if (gamma) t *= g[i];
        if (beta) t += b[i];
        r[i] = t;
    }
    Elem<T>::store8(out + row * D + sub * 8, r);
}

// Row statistics only: stats[row] = (mean, 1 / sqrt(var + eps)), same two-pass arithmetic as above.
// The bf16 block feeds them to the GEMM that follows the LayerNorm, which applies the
// normalisation in its epilogue (the normalised rows are never written).
// Bound by issue and by the wave's one trip to memory rather than by bytes.  All of a row is requested before anything is
// summed, in branch-free loads, and the sums go by DPP: 50432 x 768 23.4 us with a branch and a wait per chunk and sums
// through the LDS pipe, 21.0 with the latter by DPP, 18.1 so (events around it included: about 5.1 TB/s); two or four rows per
// wave 19.6.  16388 x 1024 10.7 / 10.1 / 9.3, 12552 x 768 8.6 / 8.0 / 7.1.
template <typename T, int MAXC>
__global__ __launch_bounds__(256) void rowstats_kernel(const T* __restrict__ x, float2* __restrict__ stats,
                                                       int64_t M, int D, float eps,
                                                       int32_t* __restrict__ iota_out, int iota_n) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (row >= M) return;
    const __amdgpu_buffer_rsrc_t rs_x = row_rsrc(x + row * D, D * (int)sizeof(T));
    float v[MAXC][8];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) row_load8(rs_x, lane + c * 64, x, v[c]);
    const float2 st = wave_row_stats<MAXC>(v, D >> 3, lane, D, eps);
    if (lane == 0) {
        stats[row] = st;
        if (iota_out) iota_out[row] = (int32_t)(row % iota_n);
    }
}

// Narrow rows (D <= 8 G, G = 16 or 32 lanes): 64 / G rows per wave, so that the lanes of a wave
// cover whole 16-byte chunks of consecutive rows instead of leaving most of them idle.  The sums
// run over the same lanes in the same butterfly order as above (the missing partners there
// hold zeros), so the statistics are the same bits.
template <typename T, int G>
__global__ __launch_bounds__(256) void rowstats_narrow_kernel(const T* __restrict__ x, float2* __restrict__ stats,
                                                              int64_t M, int D, float eps,
                                                              int32_t* __restrict__ iota_out, int iota_n) {
    constexpr int RPW = 64 / G;  // rows per wave
    const int lane = threadIdx.x & 63, sub = lane % G;
    const int64_t row = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * RPW + lane / G;
    const bool on = row < M && sub < (D >> 3);  // whole waves stay in the shuffles below
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 0.f;
    if (on) Elem<T>::load8(x + row * D + sub * 8, v);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += v[i];
    sum = lanes_sum<G>(sum);
    const float mean = sum / (float)D;
    float sq = on ? chunk_sq(v, mean) : 0.f;
    sq = lanes_sum<G>(sq);
    if (sub == 0 && row < M) {
        stats[row] = make_float2(mean, rsqrtf(sq / (float)D + eps));
        if (iota_out) iota_out[row] = (int32_t)(row % iota_n);
    }
}

hipError_t launch_rowstats(rs_dtype dt, const void* x, float* stats, int64_t M, int D, float eps,
                           hipStream_t s, int32_t* iota_out, int iota_n) {
    if (M == 0) return hipSuccess;
    dim3 grid((unsigned)((M + 3) / 4)), block(256);
    float2* st = reinterpret_cast<float2*>(stats);
    if (dt == RS_BF16 && D <= 256) {
        const bf16raw* xb = (const bf16raw*)x;
        if (D <= 128) hipLaunchKernelGGL((rowstats_narrow_kernel<bf16raw, 16>), dim3((unsigned)((M + 15) / 16)), block, 0, s, xb, st, M, D, eps, iota_out, iota_n);
        else hipLaunchKernelGGL((rowstats_narrow_kernel<bf16raw, 32>), dim3((unsigned)((M + 7) / 8)), block, 0, s, xb, st, M, D, eps, iota_out, iota_n);
        return hipGetLastError();
    }
#define RS_STATS(T_, MAXC_) \
    hipLaunchKernelGGL((rowstats_kernel<T_, MAXC_>), grid, block, 0, s, (const T_*)x, st, M, D, eps, iota_out, iota_n)
    if (dt == RS_F32) {
        if (D <= 2 * 512) RS_STATS(float, 2);
        else RS_STATS(float, 8);
    } else if (D <= 512) {
        RS_STATS(bf16raw, 1);
    } else if (D <= 2 * 512) {
        RS_STATS(bf16raw, 2);
    } else {
        RS_STATS(bf16raw, 8);
    }
#undef RS_STATS
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_ln_t(const void* x, const void* g, const void* b, void* out, int64_t M,
                              int D, float eps, hipStream_t s, int32_t* iota_out, int iota_n) {
    if (M == 0) return hipSuccess;
    dim3 grid((unsigned)((M + 3) / 4)), block(256);
    const T* xp = (const T*)x;
    const T* gp = (const T*)g;
    const T* bp = (const T*)b;
    T* op = (T*)out;
    if (D <= 256)
        hipLaunchKernelGGL((layernorm_narrow_kernel<T>), dim3((unsigned)((M + 7) / 8)), block, 0, s, xp, gp, bp, op, M, D, eps, iota_out, iota_n);
    else if (D <= 2 * 512)
        hipLaunchKernelGGL((layernorm_kernel<T, 2>), grid, block, 0, s, xp, gp, bp, op, M, D, eps, iota_out, iota_n);
    else
        hipLaunchKernelGGL((layernorm_kernel<T, 8>), grid, block, 0, s, xp, gp, bp, op, M, D, eps, iota_out, iota_n);
    return hipGetLastError();
}

hipError_t launch_layernorm(rs_dtype dt, const void* x, const void* gamma, const void* beta,
                            void* out, int64_t M, int D, float eps, hipStream_t s, int32_t* iota_out, int iota_n) {
    // host-checked by the caller: D % 8 == 0 and D <= 4096
    return dt == RS_F32 ? launch_ln_t<float>(x, gamma, beta, out, M, D, eps, s, iota_out, iota_n)
                        : launch_ln_t<bf16raw>(x, gamma, beta, out, M, D, eps, s, iota_out, iota_n);
}

}  // namespace rs
