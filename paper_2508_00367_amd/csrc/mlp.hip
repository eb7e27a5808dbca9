// The MLP half of the block in one kernel, for narrow tokens (D = 192): LayerNorm statistics, fc1, GELU, fc2,
// residual, shift sums and, where the block keeps every token, the statistics of its output.
//
// As separate launches the hidden activations are written and read once (Dm values per token against 3 D for
// everything else), and at D = 192 that traffic and the two epilogues take twice as long as the matrix work.
// Here they stay in registers: with the weights as the A operand of both products a lane holds, after fc1,
// four consecutive hidden features of ONE token per register quad; one half-wave exchange per pair of
// registers (v_permlane32_swap) turns them into the B operand of fc2, so there is no trip through LDS either.
//
// Measured at 100864 x 192 x 768 inside a block (events on the stream): 114 us against 162 us for the launches it
// replaces (statistics 15, fc1 76, fc2 71).  What bounds it is issue: per step and wave 24 MFMAs and some 230 plain and
// 32 transcendental instructions; the counters show the matrix cores busy 28 % of the cycles, other
// instructions 47 %, both at once 11 % (LDS conflicts 1 %).  Interleaving the two by hand: no change.
#include "gemm_tile.hpp"

namespace rs {

constexpr int kMlpD = 192;         // token width
constexpr int kMlpChunk = 32;      // hidden features per step
constexpr int kMlpMaxDm = 1024;    // the two per-feature vectors of fc1's LayerNorm fold lie in LDS
constexpr int kMlpRows = 128;      // rows per workgroup

// (lo half of a, lo half of b) and (hi half of a, hi half of b): the upper 32 lanes of a change places with the
// lower 32 of b.
__device__ __forceinline__ void half_swap(uint32_t& a, uint32_t& b) {
    const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(a, b, false, false));
    a = r[0];
    b = r[1];
}

// Statistics of a 192-wide row held by lanes l and l + 32, lane half g with the 8-element chunks 2 k + g: the
// additions of wave_row_stats in its order (chunk sums, then partners 16, 8, 4, 2 and 1 chunks apart).
__device__ __forceinline__ float mlp_row_sum(const float (&s)[12]) {
    float t[8], u[4];
#pragma unroll
    for (int k = 0; k < 8; ++k) t[k] = k < 4 ? s[k] + s[k + 8] : s[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = t[k] + t[k + 4];
    const float w = (u[0] + u[2]) + (u[1] + u[3]);
    return half_sum(w);
}
__device__ __forceinline__ float2 mlp_row_stats(const u32x4 (&v)[12], int D, float eps) {
    float s[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        s[k] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[k] += __uint_as_float(v[k][i] << 16);
            s[k] += __uint_as_float(v[k][i] & 0xffff0000u);
        }
    }
    const float mean = mlp_row_sum(s) / (float)D;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        // chunk_sq, element by element: the second square is the rounded one
        float d[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            d[2 * i] = __uint_as_float(v[k][i] << 16) - mean;
            d[2 * i + 1] = __uint_as_float(v[k][i] & 0xffff0000u) - mean;
        }
        s[k] = fmaf(d[0], d[0], d[1] * d[1]);
#pragma unroll
        for (int i = 2; i < 8; ++i) s[k] = fmaf(d[i], d[i], s[k]);
    }
    return make_float2(mean, rsqrtf(mlp_row_sum(s) / (float)D + eps));
}

// Workgroup: 4 waves x 32 rows, two workgroups per CU.  A wave keeps its rows (48 registers) and the 32 x 192
// outputs (96 accumulators) for the whole kernel; weights stream through a ring of three LDS stages, stage
// s = {rows 32 (s + 1) .. of W_fc1, columns 32 s .. of W_fc2}: fc1 runs one step ahead of fc2, so that its matrix
// work stands next to the GELU of the step before it.  One barrier per step of 24 MFMAs per wave.
// The weights come in fragment order: a stage is 12 fragments of W_fc1 (32 features, a row of fragments) and 6 x 2 of W_fc2.
template <int EPI, int DIST>
__global__ __launch_bounds__(256, 2) void mlp192_kernel(
    const bf16raw* __restrict__ x, const bf16raw* __restrict__ w1, const float* __restrict__ colsum,
    const float* __restrict__ bias1, const bf16raw* __restrict__ w2, const bf16raw* __restrict__ b2,
    bf16raw* __restrict__ out, float* __restrict__ partials, const bf16raw* __restrict__ ref, int post, float eps,
    int32_t* __restrict__ iota_out, int iota_n, float2* __restrict__ out_stats, int M, int D, int Dm) {
    constexpr int W1_BYTES = kMlpChunk * kMlpD * 2, STAGE = 2 * W1_BYTES, COPIES = 6;
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGE];
    __shared__ __attribute__((aligned(16))) float s_cs[kMlpMaxDm], s_b[kMlpMaxDm];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int m_base = blockIdx.x * kMlpRows + wave * 32, m = m_base + l32;
    const int T = Dm / kMlpChunk;

    const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(w1, (int64_t)Dm * kMlpD * 2);
    const __amdgpu_buffer_rsrc_t rs2 = make_rsrc(w2, (int64_t)kMlpD * Dm * 2);
    const int voff1 = wave * 1024 + lane * 16, voff2 = frag_off(wave >> 1, wave & 1, Dm) + lane * 16;

#define RS_MLP_DMA(stage_, s_)                                                                             \
    {                                                                                                      \
        const int o1_ = (s_) + 1 < T ? ((s_) + 1) * W1_BYTES : kPastEnd;                                   \
        const bool r2_ = (s_) < T;                                                                         \
        _Pragma("unroll") for (int j = 0; j < 3; ++j) dma16(rs1, (stage_) + (j * 4 + wave) * 1024, voff1, o1_ + j * 4096); \
        _Pragma("unroll") for (int j = 0; j < 3; ++j)                                                      \
            dma16(rs2, (stage_) + W1_BYTES + (j * 4 + wave) * 1024, voff2, r2_ ? frag_off(2 * j, 2 * (s_), Dm) : kPastEnd); \
    }

    // this wave's rows (rows past M are computed on a copy of the last one and never stored) and fc1's first step,
    // whose weights come straight from memory
    u32x4 xr[12], wr[12];
    {
        const bf16raw* xp = x + (int64_t)min(m, M - 1) * kMlpD + g * 8;
        const bf16raw* wp = w1 + lane * 8;
#pragma unroll
        for (int k = 0; k < 12; ++k) xr[k] = *reinterpret_cast<const u32x4*>(xp + k * 16);
#pragma unroll
        for (int k = 0; k < 12; ++k) wr[k] = *reinterpret_cast<const u32x4*>(wp + k * 512);
    }
    for (int f = tid; f < Dm; f += 256) {
        s_cs[f] = colsum[f];
        s_b[f] = bias1[f];
    }
    __builtin_amdgcn_sched_barrier(0);
    RS_MLP_DMA(st0, 0)
    RS_MLP_DMA(st1, 1)
    const float2 st = mlp_row_stats(xr, D, eps);
    f32x16 acc1, acc2[3][2][1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc1[r] = 0.f;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc2[i >> 1][i & 1][0][r] = 0.f;
#pragma unroll
    for (int k = 0; k < 12; ++k)
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wr[k]), __builtin_bit_cast(bf16x8, xr[k]), acc1, 0, 0, 0);

    const int at = lane * 16;

// Step s: GELU of the hidden features 32 s .. (in acc1), fc1 of the next 32, then fc2 over these 32.
#define RS_MLP_STEP(cur_, ahead_, s_)                                                                      \
    {                                                                                                      \
        __builtin_amdgcn_s_waitcnt(COPIES | 0x0070); /* stage s has landed, own LDS reads are done */      \
        __builtin_amdgcn_s_barrier();                                                                      \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");                                             \
        __builtin_amdgcn_sched_barrier(0);                                                                 \
        RS_MLP_DMA(ahead_, (s_) + 2)                                                                       \
        f32x16 nx_;                                                                                        \
        _Pragma("unroll") for (int r = 0; r < 16; ++r) nx_[r] = 0.f;                                       \
        _Pragma("unroll") for (int k = 0; k < 12; ++k) {                                                   \
            const bf16x8 w_ = *reinterpret_cast<const bf16x8*>((cur_) + k * 1024 + at);                    \
            nx_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w_, __builtin_bit_cast(bf16x8, xr[k]), nx_, 0, 0, 0); \
        }                                                                                                  \
        uint32_t h_[8];                                                                                    \
        _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                                    \
            const int f_ = (s_) * kMlpChunk + 8 * q + 4 * g;                                               \
            const f32x4 cs_ = *reinterpret_cast<const f32x4*>(s_cs + f_);                                  \
            const f32x4 bb_ = *reinterpret_cast<const f32x4*>(s_b + f_);                                   \
            float v_[4];                                                                                   \
            _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                  \
                v_[e] = gelu_sp(fmaf(st.y, fmaf(-st.x, cs_[e], acc1[4 * q + e]), bb_[e]));                 \
            h_[2 * q] = pack2bf(v_[0], v_[1]);                                                             \
            h_[2 * q + 1] = pack2bf(v_[2], v_[3]);                                                         \
        }                                                                                                  \
        _Pragma("unroll") for (int k = 0; k < 2; ++k) {                                                    \
            half_swap(h_[4 * k], h_[4 * k + 2]);                                                           \
            half_swap(h_[4 * k + 1], h_[4 * k + 3]);                                                       \
            const bf16x8 b_ = __builtin_bit_cast(bf16x8, (u32x4{h_[4 * k], h_[4 * k + 1], h_[4 * k + 2], h_[4 * k + 3]})); \
            _Pragma("unroll") for (int i = 0; i < 6; ++i) {                                                \
                const bf16x8 w_ = *reinterpret_cast<const bf16x8*>((cur_) + W1_BYTES + (2 * i + k) * 1024 + at); \
                acc2[i >> 1][i & 1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w_, b_, acc2[i >> 1][i & 1][0], 0, 0, 0); \
            }                                                                                              \
        }                                                                                                  \
        acc1 = nx_;                                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                                 \
    }
    for (int s = 0; s < T; s += 3) {  // T % 3 == 0
        RS_MLP_STEP(st0, st2, s)
        RS_MLP_STEP(st1, st0, s + 1)
        RS_MLP_STEP(st2, st1, s + 2)
    }
#undef RS_MLP_DMA
#undef RS_MLP_STEP
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & 0xC07F);  // trailing (empty) copies: the stages get reused
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    // residual rows into the epilogue's regions: the same exchange as above, from the B operand back to the
    // accumulator layout
    EpiRegions<1> reg[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int r0 = (wave * 3 + j) * 4096;
        reg[j].r[0] = r0 < STAGE ? st0 + r0 : st1 + (r0 - STAGE);
    }
    const int sw = epi_swz(l32);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        uint32_t r0 = xr[k][0], r1 = xr[k][1], r2 = xr[k][2], r3 = xr[k][3];
        half_swap(r0, r2);
        half_swap(r1, r3);
        unsigned char* buf = reg[k >> 2].r[0] + l32 * 128 + g * 8;
        const int c = 2 * (k & 3);
        *reinterpret_cast<uint2*>(buf + ((c ^ sw) << 4)) = make_uint2(r0, r1);
        *reinterpret_cast<uint2*>(buf + (((c + 1) ^ sw) << 4)) = make_uint2(r2, r3);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        EpiVecs<1, EPI> vec;
        vec.load(b2, GemmLnFold{}, M, kMlpD, m_base, j * 64, lane);
        gemm_epilogue_acc_layout<1, EPI, DIST>(acc2[j], reg[j], vec, out, partials, ref, post, M, kMlpD, kMlpD, 3, M, m_base,
                                               j * 64, lane);
    }
    if (out_stats) {  // statistics of the rows as stored; both halves of a row's lanes take part
        u32x4 v[12];
#pragma unroll
        for (int k = 0; k < 12; ++k)
            v[k] = *reinterpret_cast<const u32x4*>(reg[k >> 2].r[0] + l32 * 128 + (((2 * (k & 3) + g) ^ sw) << 4));
        const float2 so = mlp_row_stats(v, D, eps);
        if (g == 0 && m < M) out_stats[m] = so;
    }
    if (iota_out && g == 0 && m < M) iota_out[m] = m % iota_n;
}

// The QKV layer behind its LayerNorm for the same narrow tokens: 128 rows per workgroup stay in registers, the weights
// pass by in two LDS stages of 64 features, and every step ends with its 64 columns of the output.  A row is read once
// whatever the output width, nothing is computed for columns that do not exist (576 = 2.25 tiles of 256), and
// the statistics come from the registers when the caller has none.  100864 x 576 x 192 inside a block: 49 us, statistics
// included, against 57 and 15 for theirs (155 MB: 32 us at the copy rate); the wait for a step's stores inside
// the next step costs 3 us.
constexpr int kQkvMaxN = 1024;
__global__ __launch_bounds__(256, 2) void qkv192_kernel(const bf16raw* __restrict__ x, const bf16raw* __restrict__ w, GemmLnFold ln,
                                                        bf16raw* __restrict__ out, float eps, int M, int D, int N) {
    constexpr int STAGE = 64 * kMlpD * 2;
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char s_epi[4 * 4096];
    __shared__ __attribute__((aligned(16))) float s_cs[kQkvMaxN], s_b[kQkvMaxN];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int m_base = blockIdx.x * kMlpRows + wave * 32, m = m_base + l32;
    const int S = N / 64;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(w, (int64_t)N * kMlpD * 2);
    const int voff = wave * 1024 + lane * 16;
#define RS_QKV_DMA(stage_, s_)                                                                             \
    if ((s_) < S) {                                                                                        \
        _Pragma("unroll") for (int j = 0; j < 6; ++j) dma16(rs, (stage_) + (j * 4 + wave) * 1024, voff, (s_) * STAGE + j * 4096); \
    }
    u32x4 xr[12];
    const bf16raw* xp = x + (int64_t)min(m, M - 1) * kMlpD + g * 8;
#pragma unroll
    for (int k = 0; k < 12; ++k) xr[k] = *reinterpret_cast<const u32x4*>(xp + k * 16);
    for (int f = tid; f < N; f += 256) {
        s_cs[f] = ln.colsum[f];
        s_b[f] = ln.bias[f];
    }
    __builtin_amdgcn_sched_barrier(0);
    RS_QKV_DMA(st0, 0)
    EpiVecs<1, EPI_LN_BIAS> vec;
    vec.stats[0] = ln.stats ? reinterpret_cast<const float2*>(ln.stats)[min(m, M - 1)] : mlp_row_stats(xr, D, eps);
    EpiRegions<1> reg;
    reg.r[0] = s_epi + wave * 4096;
    const int at = lane * 16;

// Step s: the barrier says that stage s has landed (every wave has waited for its copies) and that the other stage,
// which the next copies fill, is no longer read.  The wait for these copies comes behind the matrix work and
// before the step's stores, which so have a whole step to complete.
#define RS_QKV_STEP(cur_, other_, s_)                                                                      \
    {                                                                                                      \
        __builtin_amdgcn_s_waitcnt(0xC07F); /* own LDS reads */                                            \
        __builtin_amdgcn_s_barrier();                                                                      \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");                                             \
        __builtin_amdgcn_sched_barrier(0);                                                                 \
        RS_QKV_DMA(other_, (s_) + 1)                                                                       \
        f32x16 acc[2][1];                                                                                  \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                      \
            _Pragma("unroll") for (int r = 0; r < 16; ++r) acc[i][0][r] = 0.f;                             \
        _Pragma("unroll") for (int k = 0; k < 12; ++k) {                                                   \
            _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                  \
                acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                                       \
                    *reinterpret_cast<const bf16x8*>((cur_) + (i * 12 + k) * 1024 + at),                   \
                    __builtin_bit_cast(bf16x8, xr[k]), acc[i][0], 0, 0, 0);                                \
        }                                                                                                  \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                      \
            _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                                \
                const int f_ = (s_) * 64 + i * 32 + q * 8 + g * 4;                                         \
                vec.bv[i][q] = *reinterpret_cast<const f32x4*>(s_b + f_);                                  \
                vec.cs[i][q] = *reinterpret_cast<const f32x4*>(s_cs + f_);                                 \
            }                                                                                              \
        __builtin_amdgcn_sched_barrier(0);                                                                 \
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                                                          \
        __builtin_amdgcn_sched_barrier(0);                                                                 \
        gemm_epilogue_acc_layout<1, EPI_LN_BIAS, 0>(acc, reg, vec, out, nullptr, nullptr, 0, M, N, N, 0, 0, m_base, (s_) * 64, lane); \
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    for (int s = 0; s < S; s += 2) {
        RS_QKV_STEP(st0, st1, s)
        if (s + 1 >= S) break;
        RS_QKV_STEP(st1, st0, s + 1)
    }
#undef RS_QKV_DMA
#undef RS_QKV_STEP
}

// A workgroup's time does not depend on how many there are (30 us at Dm = 768) until every CU has one, that of the
// separate launches does: two blocks in a row (no token dropped) take 127 / 123 us fused / separate at 12608 rows,
// 135 / 136 at 14184, 142 / 146 at 16548, 153 / 178 at 22064, 461 / 583 at 100864.  Below the line a workgroup
// each for half of the CUs.  A forced tile variant runs the separate launches.
static int64_t mlp_min_rows() { return (int64_t)(device_cus() / 2) * kMlpRows; }

bool mlp_fused_fits(rs_dtype dt, int64_t M, int D, int Dm) {
    return dt == RS_BF16 && D == kMlpD && Dm % (3 * kMlpChunk) == 0 && Dm <= kMlpMaxDm && gemm_variant() == 0 && M >= mlp_min_rows();
}

// Two blocks in a row against the tiled GEMM (us): 25216 rows 154 / 157, 50432 241 / 252, 100864 433 / 458, the same at 16548 (143 / 142);
// at 12608 rows, where a workgroup's nine steps are the whole launch, 135 / 124.  The line is that of the MLP kernel.
bool qkv_rows_fits(rs_dtype dt, int64_t M, int D, int N) {
    return dt == RS_BF16 && D == kMlpD && N % 64 == 0 && N <= kQkvMaxN && gemm_variant() == 0 && M >= mlp_min_rows();
}

hipError_t launch_qkv_rows(const void* x, const void* w, GemmLnFold ln, void* out, int64_t M, int N, float eps, hipStream_t s) {
    hipLaunchKernelGGL(qkv192_kernel, dim3((unsigned)((M + kMlpRows - 1) / kMlpRows)), dim3(256), 0, s, (const bf16raw*)x,
                       (const bf16raw*)w, ln, (bf16raw*)out, eps, (int)M, kMlpD, N);
    return hipGetLastError();
}

hipError_t launch_mlp_fused(const MlpArgs& g, rs_dist dist, bool shift, hipStream_t s) {
    const dim3 grid((unsigned)((g.M + kMlpRows - 1) / kMlpRows)), block(256);
#define RS_MLP_GO(EPI_, DIST_)                                                                                    \
    hipLaunchKernelGGL((mlp192_kernel<EPI_, DIST_>), grid, block, 0, s, (const bf16raw*)g.x, (const bf16raw*)g.w1, \
                       g.ln.colsum, g.ln.bias, (const bf16raw*)g.w2, (const bf16raw*)g.b2, (bf16raw*)g.out, g.partials, \
                       (const bf16raw*)g.ref, g.post ? 1 : 0, g.eps, g.iota_out, g.iota_n, (float2*)g.out_stats, (int)g.M, \
                       kMlpD, g.Dm)
    if (!shift) RS_MLP_GO(EPI_BIAS_RES, RS_DIST_L2);
    else if (dist == RS_DIST_L2) RS_MLP_GO(EPI_BIAS_RES_SHIFT, RS_DIST_L2);
    else if (dist == RS_DIST_L1) RS_MLP_GO(EPI_BIAS_RES_SHIFT, RS_DIST_L1);
    else RS_MLP_GO(EPI_BIAS_RES_SHIFT, RS_DIST_COS);
#undef RS_MLP_GO
    return hipGetLastError();
}

}  // namespace rs
