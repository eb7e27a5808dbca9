// fp32 linear layers of the encoder block (parity configuration: fp32 storage, fp32 products and
// sums):  out[m, n] = epi( sum_k a[m, k] * w[k, n] ),  w as the caller gives it ([K, N]).
//
// v_mfma_f32_32x32x2_f32: 256 flops per clock and CU, twice the plain (unpacked) FMA rate, so the
// contraction belongs there.  Weights are the A operand (rows = features), activations the B operand
// (columns = token rows), as in the bf16 kernels.  One k step of the instruction takes k from the low
// half-wave and k' from the high one; which two k these are is free as long as both operands agree, so
// a lane reads four consecutive k of its token row at once (k = 8 h + 4 g + e feeds step (h, e)).
//
// Workgroup tile 32 x 64, four waves that share the tile and split K: of every 64 values of k
// wave w takes 16 w .. 16 w + 15, and the four partial tiles are added through LDS in wave order,
// ((p0 + p1) + (p2 + p3)) per element: one order in both kernels, so results do not depend on
// the grid.  No data is shared between waves inside the loop: every wave streams its own operand
// slices global -> LDS (direct copies) in a ring of its own and waits for nobody, there is no barrier
// before the final sum.  The K split is what fills the chip at the sizes this path is used at: four
// images of 197 tokens make 39 64 x 64 tiles (fc2) on 256 CUs.
// Bound by the matrix cores (132 TFLOP/s at 12608 x 3072 x 768, the library's rate there; 105 at
// 12608 x 768 x 192, where a tile is six slices of 32 long); the plain FMA tiles this replaced ran
// at 60 and took 71 us for the fc2 of a 4 x 197 x 192 block (9.5 us now).
// Two kernels: 32 x 64 tiles with K split over the waves (three stages, 48 KB of LDS in all) for grids that
// leave CUs idle, and 64 x 64 tiles shared by the waves (gemm_f32_wide_kernel) for those that fill the chip.
#include "common.hpp"
#include "gemm_choice.hpp"

namespace rs {

typedef __attribute__((address_space(3))) void* lds_ptr_f;

__device__ __forceinline__ void dma16_f(__amdgpu_buffer_rsrc_t rsrc, unsigned char* lds_base, int voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_f)lds_base, 16, voff, soff, 0, 0);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_f(const void* base, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// Row-major epilogue of a BM x 64 tile, 16 lanes per row, 4 features per lane: load() requests what it needs from
// memory, run() takes the sums (sum(row, group of 4 features)) once they are in LDS.
template <int BM, int EPI, int DIST>
struct F32Epilogue {
    static constexpr bool RES = EPI == EPI_BIAS_RES || EPI == EPI_BIAS_RES_SHIFT;
    int tx, ty, n;
    float bv[4];
    float4 res4[BM / 16];
    __device__ __forceinline__ void load(const float* __restrict__ bias, const float* __restrict__ res, int m0, int n0, int M, int N) {
        tx = threadIdx.x & 15;
        ty = threadIdx.x >> 4;
        n = n0 + tx * 4;
        bv[0] = bv[1] = bv[2] = bv[3] = 0.f;
        if (bias) {
            const float4 b4 = *reinterpret_cast<const float4*>(bias + n);
            bv[0] = b4.x; bv[1] = b4.y; bv[2] = b4.z; bv[3] = b4.w;
        }
        if (RES) {
#pragma unroll
            for (int p = 0; p < BM / 16; ++p) {
                const int m = m0 + p * 16 + ty;
                res4[p] = m < M ? *reinterpret_cast<const float4*>(res + (int64_t)m * N + n) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    }
    template <typename Sum>
    __device__ __forceinline__ void run(const Sum& sum, float* __restrict__ out, float* __restrict__ partials,
                                        const float* __restrict__ ref, int post, int m0, int tn, int slots, int M, int N) {
        const __amdgpu_buffer_rsrc_t rs_out = rsrc_f(out + (int64_t)m0 * N + tn * 64, ((int64_t)(min(M - m0, BM) - 1) * N + 64) * 4);
#pragma unroll
        for (int p = 0; p < BM / 16; ++p) {
            const int r = p * 16 + ty, m = m0 + r;
            const bool m_ok = m < M;
            const f32x4 s4 = sum(r, tx);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = s4[e] + bv[e];
            if (EPI == EPI_BIAS_GELU) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
            }
            float p0 = 0.f, p1 = 0.f, p2 = 0.f;
            if (RES) {
                const float rr[4] = {res4[p].x, res4[p].y, res4[p].z, res4[p].w};
                if (EPI == EPI_BIAS_RES_SHIFT && m_ok) {
                    float fi[4] = {rr[0], rr[1], rr[2], rr[3]};
                    if (ref) {
                        const float4 q = *reinterpret_cast<const float4*>(ref + (int64_t)m * N + n);
                        fi[0] = q.x; fi[1] = q.y; fi[2] = q.z; fi[3] = q.w;
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float fo = post ? v[e] + rr[e] : v[e];
                        if (DIST == RS_DIST_L2) { const float d = fo - fi[e]; p0 += d * d; }
                        else if (DIST == RS_DIST_L1) { p0 += fabsf(fo - fi[e]); }
                        else { p0 += fo * fi[e]; p1 += fo * fo; p2 += fi[e] * fi[e]; }
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += rr[e];
            }
            store16_wt(rs_out, m_ok ? (r * N + tx * 4) * 4 : 0x7ff00000,
                       make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])));
            if (EPI == EPI_BIAS_RES_SHIFT) {
                // the 16 lanes of a row in a fixed butterfly order; one slot per 64 features
                p0 = lanes_sum<16>(p0);
                if (DIST == RS_DIST_COS) { p1 = lanes_sum<16>(p1); p2 = lanes_sum<16>(p2); }
                if (tx == 0 && m_ok) {
                    float* dst = partials + (int64_t)tn * M + m;
                    dst[0] = p0;
                    if (DIST == RS_DIST_COS) { dst[(int64_t)slots * M] = p1; dst[(int64_t)2 * slots * M] = p2; }
                }
            }
        }
    }
};

template <int EPI, int DIST>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(
    const float* __restrict__ a, const float* __restrict__ w, const float* __restrict__ bias,
    const float* __restrict__ res, float* __restrict__ out, float* __restrict__ partials,
    const float* __restrict__ ref, int post, int M, int N, int K, int tiles_m,
    int tiles_n) {
    constexpr int BM = 32, BN = 64;
    constexpr int NST = 3;                            // ring stages
    constexpr int A_BYTES = BM * 64, W_BYTES = 16 * BN * 4, SLICE = A_BYTES + W_BYTES;  // per wave
    constexpr int L = SLICE / 1024;                   // copies per slice
    constexpr int PITCH = BN * 4 + 16;                // staged fp32 row of the final sum
    constexpr int STAGE = 4 * SLICE;
    constexpr int HALF_RED = 2 * BM * PITCH;          // two waves' partial tiles
    // one array per stage, so that the compiler knows which copies a slice's reads wait for; the
    // partial tiles of waves 0, 1 and 2, 3 go through the first two at the end
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE > HALF_RED ? STAGE : HALF_RED];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE > HALF_RED ? STAGE : HALF_RED];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    // tile of this workgroup: ids go round-robin to the 8 XCDs, XCD x takes a contiguous range of the
    // row-major tile sequence, so that the column tiles of a row panel find it in one L2
    const int nblk = tiles_m * tiles_n;
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    const int xq = nblk >> 3, xr = nblk & 7;
    if (seq >= xq + (xcd < xr ? 1 : 0)) return;  // whole workgroup, before any barrier
    const int bid = xcd * xq + (xcd < xr ? xcd : xr) + seq;
    const int tn = bid % tiles_n, slots = tiles_n;
    const int m0 = bid / tiles_n * BM, n0 = tn * BN;

    // activation slice: BM rows of 16 k (64 bytes); 16-byte chunk c of row r sits in slot c ^ ((r >> 2) & 3)
    // (the 16 rows a 16-byte read touches at a time fall into 16 different bank groups).  Copy i: rows
    // 16 i .. + 15, lane l: row l / 4, slot l % 4.  Rows past M read as zeros.
    const __amdgpu_buffer_rsrc_t rs_a = rsrc_f(a + (int64_t)m0 * K, (int64_t)min(M - m0, BM) * K * 4);
    const int a_voff = (lane >> 2) * K * 4 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
    // weight slice: 16 k rows of 64 features (256 bytes); rows with (k >> 2) odd swap their two halves, so
    // that the half-waves, which read rows k and k + 4, use different banks.  Copy i: rows 4 i .. + 3,
    // lane l: row l / 16, slot l % 16.
    const int w_voff = (lane >> 4) * N * 4 + ((lane & 15) << 4);
    const int w_flip = 128 * (lane & 8 ? -1 : 1);  // byte distance to the chunk of the other half

    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    const int S = K >> 6;
// copies of this wave's share of slice t_; past the last slice the resource is empty (zeros arrive)
#define RS_F32_DMA(st_, t_)                                                                                   \
    {                                                                                                         \
        unsigned char* p_ = (st_) + wave * SLICE;                                                             \
        const bool real_ = (t_) < S;                                                                          \
        const int k_ = (t_) * 64 + wave * 16;                                                                 \
        _Pragma("unroll") for (int i = 0; i < A_BYTES / 1024; ++i)                                            \
            dma16_f(rs_a, p_ + i * 1024, a_voff, real_ ? i * 16 * K * 4 + k_ * 4 : 0x7ff00000);               \
        const __amdgpu_buffer_rsrc_t rs_w =                                                                   \
            rsrc_f(w + (real_ ? (int64_t)k_ * N + n0 : 0), real_ ? (15 * (int64_t)N + BN) * 4 : 0);           \
        _Pragma("unroll") for (int i = 0; i < W_BYTES / 1024; ++i)                                            \
            dma16_f(rs_w, p_ + A_BYTES + i * 1024, w_voff + (i & 1 ? w_flip : 0), i * 4 * N * 4);             \
    }
#define RS_F32_COMPUTE(st_)                                                                                   \
    {                                                                                                         \
        const unsigned char* p_ = (st_) + wave * SLICE;                                                       \
        _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                                       \
            const f32x4 af =                                                                                  \
                *reinterpret_cast<const f32x4*>(p_ + l32 * 64 + (((2 * h + g) ^ ((l32 >> 2) & 3)) << 4));     \
            float wf[4][2];                                                                                   \
            _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                     \
                _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                 \
                    wf[e][i] = *reinterpret_cast<const float*>(p_ + A_BYTES + (8 * h + 4 * g + e) * 256 +     \
                                                               (((i * 32 + l32) * 4) ^ (g << 7)));            \
            _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                     \
                _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                 \
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[e][i], af[e], acc[i], 0, 0, 0);          \
        }                                                                                                     \
    }
// slice t_ from cur_ while the copies of slice t_ + NST - 1 go into free_ (read NST slices ago: those reads
// have been answered, the matrix instructions behind them are issued)
#define RS_F32_STEP(cur_, free_, t_)                                                                          \
    {                                                                                                         \
        __builtin_amdgcn_s_waitcnt(0xC07F); /* lgkmcnt(0) */                                                  \
        RS_F32_DMA(free_, (t_) + NST - 1)                                                                     \
        __builtin_amdgcn_s_waitcnt((((NST - 1) * L) & 15) | ((((NST - 1) * L) >> 4) << 14) | 0x0F70);         \
        RS_F32_COMPUTE(cur_)                                                                                  \
    }

    RS_F32_DMA(st0, 0)
    RS_F32_DMA(st1, 1)
    for (int t = 0; t < S; t += 3) {
        RS_F32_STEP(st0, st2, t)
        if (t + 1 >= S) break;
        RS_F32_STEP(st1, st0, t + 1)
        if (t + 2 >= S) break;
        RS_F32_STEP(st2, st1, t + 2)
    }
#undef RS_F32_DMA
#undef RS_F32_COMPUTE
#undef RS_F32_STEP

    // ---- sum of the four partial tiles, row-major: 16 lanes per row, 4 features per lane
    __builtin_amdgcn_s_waitcnt(0x0070);  // trailing (empty) copies and LDS reads: the stages get reused
    __syncthreads();
    unsigned char* red = (wave < 2 ? st0 : st1) + (wave & 1) * BM * PITCH;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
            *reinterpret_cast<f32x4*>(red + l32 * PITCH + (i * 32 + q * 8 + g * 4) * 4) = v;
        }
    F32Epilogue<BM, EPI, DIST> epi;
    epi.load(bias, res, m0, n0, M, N);
    __syncthreads();
    epi.run([&](int r, int c4) {
        f32x4 s4[4], v;
#pragma unroll
        for (int u = 0; u < 4; ++u) s4[u] = *reinterpret_cast<const f32x4*>((u < 2 ? st0 : st1) + ((u & 1) * BM + r) * PITCH + c4 * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (s4[0][e] + s4[1][e]) + (s4[2][e] + s4[3][e]);
        return v;
    }, out, partials, ref, post, m0, tn, slots, M, N);
}

// The same products and sums for grids that fill the chip: 64 x 64 tile, a wave owns a quarter of it (32 rows x 32
// features) over the whole of K and keeps the four partial sums of an element in four accumulators, so that the
// final sum is three additions in registers and not 64 KB written to LDS and read back.  The waves share the
// slices (one barrier each).  Slices of 32 k, so that two stages are 32 KB and four workgroups share a CU: tiles are a
// few slices long, and what three of them wait for (first slice, stores) the fourth fills.  Slices of 64 and two workgroups
// before: 12608 x 768 x 192 40.6 us, 35.5 now, with GELU 50.5 / 41.3, 12608 x 768 x 768 128.6 / 117.
// Where the choice asks for three workgroups per CU, a launch claims kWidePad bytes of LDS more, which nobody uses.
constexpr unsigned kWidePad = 8192;
template <int EPI, int DIST>
__global__ __launch_bounds__(256, 4) void gemm_f32_wide_kernel(
    const float* __restrict__ a, const float* __restrict__ w, const float* __restrict__ bias,
    const float* __restrict__ res, float* __restrict__ out, float* __restrict__ partials,
    const float* __restrict__ ref, int post, int M, int N, int K, int tiles_m, int tiles_n) {
    constexpr int BM = 64, BN = 64, A_BYTES = BM * 64, W_BYTES = 16 * BN * 4, SLICE = A_BYTES + W_BYTES, PITCH = BN * 4 + 16;
    __shared__ __attribute__((aligned(1024))) unsigned char st0[BM * PITCH];  // the sums go through it at the end
    __shared__ __attribute__((aligned(1024))) unsigned char st1[2 * SLICE];
    static_assert(BM * PITCH >= 2 * SLICE, "a stage: two partial sums' k");
    constexpr int LDS = BM * PITCH + 2 * SLICE, CU_LDS = 160 * 1024;
    static_assert(4 * LDS <= CU_LDS && 3 * (LDS + (int)kWidePad) <= CU_LDS && 4 * (LDS + (int)kWidePad) > CU_LDS, "four, or with the padding three workgroups");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int rq = (wave & 1) * 32, fq = (wave >> 1) * 32;  // this wave's quarter
    const int nblk = tiles_m * tiles_n;
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    const int xq = nblk >> 3, xr = nblk & 7;
    if (seq >= xq + (xcd < xr ? 1 : 0)) return;  // whole workgroup, before any barrier
    const int bid = xcd * xq + (xcd < xr ? xcd : xr) + seq;
    const int tn = bid % tiles_n, slots = tiles_n;
    const int m0 = bid / tiles_n * BM, n0 = tn * BN;

    // LDS layout and copies as above: region u of the even slices holds the 16 k of partial sums 0 and 1, of the odd ones of
    // 2 and 3; waves 0, 1 copy the activation rows of a region each, waves 2, 3 the weights
    const __amdgpu_buffer_rsrc_t rs_a = rsrc_f(a + (int64_t)m0 * K, (int64_t)min(M - m0, BM) * K * 4);
    const int a_voff = (lane >> 2) * K * 4 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
    const int w_voff = (lane >> 4) * N * 4 + ((lane & 15) << 4);
    const int w_flip = 128 * (lane & 8 ? -1 : 1);
    f32x16 acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][r] = 0.f;

    const int S = K >> 5;  // even: K % 64 == 0
#define RS_F32W_DMA(st_, t_)                                                                                  \
    if ((t_) < S) {                                                                                           \
        unsigned char* p_ = (st_) + (wave & 1) * SLICE;                                                       \
        const int k_ = (t_) * 32 + (wave & 1) * 16;                                                           \
        if (wave < 2) {                                                                                       \
            _Pragma("unroll") for (int i = 0; i < A_BYTES / 1024; ++i)                                        \
                dma16_f(rs_a, p_ + i * 1024, a_voff, i * 16 * K * 4 + k_ * 4);                                \
        } else {                                                                                              \
            const __amdgpu_buffer_rsrc_t rs_w = rsrc_f(w + (int64_t)k_ * N + n0, (15 * (int64_t)N + BN) * 4); \
            _Pragma("unroll") for (int i = 0; i < W_BYTES / 1024; ++i)                                        \
                dma16_f(rs_w, p_ + A_BYTES + i * 1024, w_voff + (i & 1 ? w_flip : 0), i * 4 * N * 4);         \
        }                                                                                                     \
    }
// slice t_ from cur_ into partial sums u0_ and u0_ + 1; its barrier also says that every wave is done with the slice
// before, whose stage the next copies fill
#define RS_F32W_STEP(cur_, other_, t_, u0_)                                                                   \
    {                                                                                                         \
        __builtin_amdgcn_s_waitcnt(0x0070); /* own copies of this slice, own reads of the one before */       \
        __builtin_amdgcn_s_barrier();                                                                         \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");                                                \
        RS_F32W_DMA(other_, (t_) + 1)                                                                         \
        _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                                       \
            f32x4 af[2];                                                                                      \
            float wf[2][4];                                                                                   \
            _Pragma("unroll") for (int u = 0; u < 2; ++u) {                                                   \
                const unsigned char* p_ = (cur_) + u * SLICE;                                                 \
                af[u] = *reinterpret_cast<const f32x4*>(p_ + (rq + l32) * 64 + (((2 * h + g) ^ ((l32 >> 2) & 3)) << 4)); \
                _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                 \
                    wf[u][e] = *reinterpret_cast<const float*>(p_ + A_BYTES + (8 * h + 4 * g + e) * 256 +     \
                                                               (((fq + l32) * 4) ^ (g << 7)));                \
            }                                                                                                 \
            _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                     \
                _Pragma("unroll") for (int u = 0; u < 2; ++u)                                                 \
                    acc[(u0_) + u] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[u][e], af[u][e], acc[(u0_) + u], 0, 0, 0); \
        }                                                                                                     \
    }
    RS_F32W_DMA(st0, 0)
    for (int t = 0; t < S; t += 2) {
        RS_F32W_STEP(st0, st1, t, 0)
        RS_F32W_STEP(st1, st0, t + 1, 2)
    }
#undef RS_F32W_DMA
#undef RS_F32W_STEP

    F32Epilogue<BM, EPI, DIST> epi;
    epi.load(bias, res, m0, n0, M, N);
    // through the stage that the last slice does not lie in: no wave reads it any more and no copy is in flight
    unsigned char* red = st0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (acc[0][4 * q + e] + acc[1][4 * q + e]) + (acc[2][4 * q + e] + acc[3][4 * q + e]);
        *reinterpret_cast<f32x4*>(red + (rq + l32) * PITCH + (fq + q * 8 + g * 4) * 4) = v;
    }
    __syncthreads();
    epi.run([&](int r, int c4) { return *reinterpret_cast<const f32x4*>(red + r * PITCH + c4 * 16); }, out, partials, ref, post,
            m0, tn, slots, M, N);
}

template <int EPI, int DIST>
static hipError_t launch_t(const void* a, const void* w, const void* bias, const void* res, void* out, float* partials,
                           const void* ref, bool post, int64_t M, int N, int K, hipStream_t s) {
    const int tiles_n = N / 64;
    const GemmF32Choice c = gemm_f32_choose(M, N, K, device_cus());
    const bool wide = c.per_cu > 0;
    const int bm = wide ? 64 : 32;
    const unsigned lds = c.per_cu == 3 ? kWidePad : 0;
    const int64_t rows = gemm_f32_launch_rows(N, bm);
    if (partials && M > rows) return hipErrorInvalidValue;  // the sums' slots lie M apart: one launch (rows of 4096 values at most)
    for (int64_t r = 0; r < M; r += rows) {
        const int64_t m = M - r < rows ? M - r : rows, tiles_m = (m + bm - 1) / bm, nblk = tiles_m * tiles_n;
        auto go = [&](auto* kernel, unsigned pad) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * ((nblk + 7) / 8))), dim3(256), pad, s, (const float*)a + r * K,
                               (const float*)w, (const float*)bias, res ? (const float*)res + r * N : nullptr, (float*)out + r * N,
                               partials, ref ? (const float*)ref + r * N : nullptr, post ? 1 : 0, (int)m, N, K, (int)tiles_m, tiles_n);
        };
        if (wide) go(&gemm_f32_wide_kernel<EPI, DIST>, lds);
        else go(&gemm_f32_kernel<EPI, DIST>, 0u);
    }
    return hipGetLastError();
}

hipError_t launch_gemm_f32(GemmEpilogue epi, rs_dist dist, const void* a, const void* w, const void* bias,
                           const void* res, void* out, float* partials, const void* ref, bool post, int64_t M, int N,
                           int K, hipStream_t s) {
    switch (epi) {
        case EPI_BIAS: return launch_t<EPI_BIAS, 0>(a, w, bias, res, out, partials, ref, post, M, N, K, s);
        case EPI_BIAS_GELU: return launch_t<EPI_BIAS_GELU, 0>(a, w, bias, res, out, partials, ref, post, M, N, K, s);
        case EPI_BIAS_RES: return launch_t<EPI_BIAS_RES, 0>(a, w, bias, res, out, partials, ref, post, M, N, K, s);
        case EPI_BIAS_RES_SHIFT:
            if (dist == RS_DIST_L2) return launch_t<EPI_BIAS_RES_SHIFT, RS_DIST_L2>(a, w, bias, res, out, partials, ref, post, M, N, K, s);
            if (dist == RS_DIST_L1) return launch_t<EPI_BIAS_RES_SHIFT, RS_DIST_L1>(a, w, bias, res, out, partials, ref, post, M, N, K, s);
            return launch_t<EPI_BIAS_RES_SHIFT, RS_DIST_COS>(a, w, bias, res, out, partials, ref, post, M, N, K, s);
        default: break;  // the LayerNorm-folded epilogues are bf16 only
    }
    return hipErrorInvalidValue;
}

}  // namespace rs
