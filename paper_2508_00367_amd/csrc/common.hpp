// Shared device/host helpers of the representation-shift HIP library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rs.h"

namespace rs {

constexpr int kWave = 64;  // CDNA wavefront width

typedef uint16_t bf16raw;  // bf16 storage: upper half of an fp32
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// plain vectors: arrays of the HIP vector classes (uint4) that are not written on every path end up in LDS
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ---- bf16 <-> fp32 -------------------------------------------------------
__device__ __forceinline__ float bf2f(bf16raw b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even, NaN stays NaN: the hardware conversion (v_cvt_pk_bf16_f32)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16raw f2bf(float f) { return __builtin_bit_cast(bf16raw, (__bf16)f); }

__device__ __forceinline__ uint32_t pack2bf(float lo, float hi) {
    bf16x2 v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// Stores of a kernel's output that go through the L2 to memory at once (sc1, the scope of the whole GPU) instead of staying
// there dirty: every kernel ends with a write-back of its XCDs' L2s, and the next one, whose tiles lie elsewhere on the
// chip, finds the lines in the memory-side cache either way.  For stores of whole lines only.  us per forward, GEMM epilogues alone:
// vit_s16 961 -> 923, video_vit_b16 1750 -> 1712, video_vit_l14 8540 -> 8466, deit_t 1766 -> 1745; bf16 attention, its rows gathered
// into lines in LDS first: deit_t 1690 -> 1652, video_vit_l14 8300 -> 8210; fp32 GEMMs: deit_t_fp32 1423 -> 1366; the prune step's
// rows: vit_s16 882 -> 877.  (Slower: half lines per instruction, as fp32 attention and LayerNorm store,
// deit_t_fp32 +2 %; 8 bytes per lane and row, bf16 attention's accumulators, +5 %; non-temporal stores, which also pass by the
// memory-side cache, deit_t and one image +3.5 %.)
constexpr int kWriteThrough = 16;  // cache policy of a buffer store: sc1
__device__ __forceinline__ void store16_wt(__amdgpu_buffer_rsrc_t rsrc, int voff, u32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, voff, 0, kWriteThrough);
}
__device__ __forceinline__ void store16_wt(__amdgpu_buffer_rsrc_t rsrc, int voff, uint4 v) {
    store16_wt(rsrc, voff, u32x4{v.x, v.y, v.z, v.w});
}

// Storage-type traits: load/store 8 consecutive elements as fp32.
template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr rs_dtype dtype = RS_F32;
    __device__ static __forceinline__ void load8(const float* p, float (&v)[8]) {
        float4 a = *reinterpret_cast<const float4*>(p);
        float4 b = *reinterpret_cast<const float4*>(p + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
    __device__ static __forceinline__ void store8(float* p, const float (&v)[8]) {
        *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
    __device__ static __forceinline__ float ld(const float* p) { return *p; }
    __device__ static __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16raw> {
    static constexpr rs_dtype dtype = RS_BF16;
    __device__ static __forceinline__ void load8(const bf16raw* p, float (&v)[8]) {
        uint4 a = *reinterpret_cast<const uint4*>(p);
        uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ static __forceinline__ void store8(bf16raw* p, const float (&v)[8]) {
        uint4 a;
        a.x = pack2bf(v[0], v[1]); a.y = pack2bf(v[2], v[3]);
        a.z = pack2bf(v[4], v[5]); a.w = pack2bf(v[6], v[7]);
        *reinterpret_cast<uint4*>(p) = a;
    }
    __device__ static __forceinline__ float ld(const bf16raw* p) { return bf2f(*p); }
    __device__ static __forceinline__ void st(bf16raw* p, float v) { *p = f2bf(v); }
};

// ---- wave reductions (fixed butterfly order: deterministic) ---------------
// op over the G lanes of a group (aligned, all of them active): every lane combines with the one G / 2 away, then G / 4, ... 1,
// for an op that does not care which of two comes first.  The partner comes by lane swaps and DPP moves that the
// compiler folds into the op, one or two instructions a step; through __shfl_xor a step is a trip through the LDS pipe
// plus address arithmetic and a wait (row statistics of 50432 x 768 23.4 -> 21.0 us, scores, selection and copy of 8 x 1569 x 768
// out of the caches 25.7 -> 24.5, one image through 12 blocks 442 -> 434).
//   32, 16 apart: v_permlane32_swap / v_permlane16_swap of a value with itself leave both halves' values in every lane.
//   8 apart: a rotation of the 16-lane row by 8; 4 apart: by 4, where the lanes 8 apart already agree.
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_mov(T v) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int G, typename T, typename Op>
__device__ __forceinline__ T lanes_reduce(T v, Op op) {
    static_assert(G == 8 || G == 16 || G == 32 || G == 64, "a group is 8 lanes or whole 16-lane rows");
    if constexpr (G >= 64) {
        const uint32_t u = __builtin_bit_cast(uint32_t, v);
        const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(u, u, false, false));
        const uint32_t lo = r[0], hi = r[1];
        v = op(__builtin_bit_cast(T, lo), __builtin_bit_cast(T, hi));
    }
    if constexpr (G >= 32) {
        const uint32_t u = __builtin_bit_cast(uint32_t, v);
        const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(u, u, false, false));
        const uint32_t lo = r[0], hi = r[1];
        v = op(__builtin_bit_cast(T, lo), __builtin_bit_cast(T, hi));
    }
    if constexpr (G >= 16) {
        v = op(v, dpp_mov<0x128>(v));  // row_ror:8
        v = op(v, dpp_mov<0x124>(v));  // row_ror:4
    } else {  // row_shl:4 into lanes 0-3 and 8-11, row_shr:4 into the others
        const int i = __builtin_bit_cast(int, v), up = __builtin_amdgcn_update_dpp(i, i, 0x104, 0xf, 0x5, false);
        const int both = __builtin_amdgcn_update_dpp(up, i, 0x114, 0xf, 0xa, false);
        v = op(v, __builtin_bit_cast(T, both));
    }
    v = op(v, dpp_mov<0x4e>(v));   // quad_perm [2,3,0,1]
    return op(v, dpp_mov<0xb1>(v));  // quad_perm [1,0,3,2]
}
template <int G>
__device__ __forceinline__ float lanes_sum(float v) {
    return lanes_reduce<G>(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_sum(float v) { return lanes_sum<64>(v); }

// Inclusive sum over the lanes of a wave (all of them active), by DPP moves: row_shr 1, 2, 4, 8 inside the 16-lane rows (lanes
// with nobody that far below add 0), then the rows' last lanes by row_bcast 15 into rows 1 and 3 and row_bcast 31 into 2 and 3.
__device__ __forceinline__ int wave_scan_incl(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// A lane's value and that of its partner 32 lanes away, the lower lane's first, by v_permlane32_swap: no trip through the LDS
// pipe, whose latency would stand in the middle of a softmax's chain, and no lane arithmetic for its address.
__device__ __forceinline__ float2 half_pair(float v) {
    const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
    return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_max(float v) {
    const float2 p = half_pair(v);
    return fmaxf(p.x, p.y);
}
__device__ __forceinline__ float half_sum(float v) {
    const float2 p = half_pair(v);
    return p.x + p.y;
}

// Buffer resource over `bytes` of one row: what lies past them reads as zero, so that a row's loads need no branches.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// Squared deviations of a row's first 8 values (its first two terms as one fused product, the others behind them), or of the
// next 8 added to `sq`: written out, since the compiler is free to fuse a sum of products either way.
__device__ __forceinline__ float chunk_sq(const float (&v)[8], float mean) {
    const float d0 = v[0] - mean, d1 = v[1] - mean;
    float t = fmaf(d0, d0, d1 * d1);
#pragma unroll
    for (int i = 2; i < 8; ++i) { const float d = v[i] - mean; t = fmaf(d, d, t); }
    return t;
}
__device__ __forceinline__ float chunk_sq(const float (&v)[8], float mean, float sq) {
#pragma unroll
    for (int i = 0; i < 8; ++i) { const float d = v[i] - mean; sq = fmaf(d, d, sq); }
    return sq;
}

// Statistics of a row a wave holds as MAXC chunks of 8 values per lane (lane l: chunks l, l + 64,
// ...; chunks at or past nchunk hold zeros): (mean, 1 / sqrt(population variance + eps)), the
// variance taken over the deviations from the mean.  One fixed order of additions, shared by
// every kernel that produces LayerNorm statistics, so that they all give the same bits.
template <int MAXC>
__device__ __forceinline__ float2 wave_row_stats(const float (&v)[MAXC][8], int nchunk, int lane, int D, float eps) {
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += v[c][i];
    }
    const float mean = wave_sum(sum) / (float)D;
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const float t = c == 0 ? chunk_sq(v[0], mean) : chunk_sq(v[c], mean, sq);
        sq = lane + c * 64 < nchunk ? t : sq;
    }
    return make_float2(mean, rsqrtf(wave_sum(sq) / (float)D + eps));
}

// exact GELU: x * Phi(x)
__device__ __forceinline__ float gelu_erf(float x) {
    return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f));
}

// ---- host-side error plumbing ---------------------------------------------
void set_error(const char* fmt, ...);
rs_status device_error(const char* what, hipError_t e);

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
// compute units of the device in use at the first call (256 where there is none to ask)
int device_cus();
inline size_t elem_size(rs_dtype t) { return t == RS_F32 ? 4 : 2; }

// ---- kernel launchers (one per .hip file) -----------------------------------
// LayerNorm over the last axis of x[M, D]; gamma/beta may be null; iota_out as in launch_rowstats.
hipError_t launch_layernorm(rs_dtype dt, const void* x, const void* gamma, const void* beta, void* out, int64_t M, int D,
                            float eps, hipStream_t s, int32_t* iota_out = nullptr, int iota_n = 1);

// stats[M] = (mean, 1 / sqrt(population variance + eps)) of each row of x[M, D], as float pairs.
// iota_out (optional): int32 [M], receives row % iota_n (the kept_idx of a block that keeps every token).
hipError_t launch_rowstats(rs_dtype dt, const void* x, float* stats, int64_t M, int D, float eps,
                           hipStream_t s, int32_t* iota_out = nullptr, int iota_n = 1);

enum GemmEpilogue {
    EPI_BIAS = 0,            // out = acc + bias
    EPI_BIAS_GELU = 1,       // out = gelu(acc + bias)
    EPI_BIAS_RES = 2,        // out = acc + bias + res
    EPI_BIAS_RES_SHIFT = 3,  // out = acc + bias + res; partial sums of D(f_out, f_in) per row, with
                             // f_out = acc + bias (or out, if `post`) and f_in = res (or `ref`, if given)
    // bf16 only: the A operand is the raw input x of a LayerNorm whose scale is folded into the
    // packed weights, acc = x (gamma * W);  LN(x) W + b = rstd * (acc - mean * colsum) + bias'
    // with per-row (mean, rstd) and per-column colsum = sum_k gamma_k W_kn, bias' = beta W + b.
    EPI_LN_BIAS = 4,         // out = rstd * (acc - mean * colsum) + bias'
    EPI_LN_BIAS_GELU = 5     // out = gelu(rstd * (acc - mean * colsum) + bias')
};

// Per-row and per-column vectors of the EPI_LN_* epilogues (all fp32, device memory).
struct GemmLnFold {
    const float* stats;   // [M][2]  (mean, rstd)
    const float* colsum;  // [N]
    const float* bias;    // [N]
};

// Largest K and N of a GEMM: a workgroup addresses the (at most 256) rows of its tile with 32-bit
// byte offsets from the tile's first row, 256 * K * 2 bytes, and the copies of a K slice that does
// not exist are aimed at byte 0x7ff00000 of a resource that ends with the tile's last row.
constexpr int kGemmMaxK = 1 << 20;
constexpr int kGemmMaxN = 1 << 20;

// Tile configurations the bf16 GEMM was built with (measurements carried from one run to another
// are only valid for the same string).
const char* gemm_build_info();
// bf16 tile variant switch (0 = by shape, 1 = 256 x 256 persistent, 2 = 256 x 128, 3 = 128 x 128 ring, 4 = 128 x 256 ring)
int gemm_variant();
void set_gemm_variant(int v);

// Number of per-row partial slots the SHIFT epilogue writes for an output width N.
int gemm_shift_slots(rs_dtype dt, int N);
constexpr int kShiftLanes = 3;  // sums per slot (L2/L1 use the first, cosine all three)

// Row pitch (elements) of the MLP's hidden activations in a block whose caller has packed the weights (one that packs on
// every call keeps the plain pitch, its scratch has no room for another): the rows of an operand
// tile are requested together, and when the pitch is a multiple of 512 bytes they meet in a few of the
// L2's channels.  One extra line per row spreads them: 768 x 3072 at 50432 rows 252 -> 243 us, at 3152 rows
// 26.5 -> 23.7, 384 x 1536 at 12608 rows 24.8 -> 23.0 (128, 192 or 256 extra elements: the same; 32 or less
// split lines and cost 5-30 %), measured with W_fc2 in rows of the same pitch.  (The attention output, padded the
// same way: no change.)  Rows under 1 KB stay as they are: such a GEMM has at most four slices of K.
inline int padded_ld(int K) { return K >= 512 && K % 256 == 0 ? K + 64 : K; }

// out[M, N] = epilogue(a[M, K] @ W).  bf16: `w` is the packed [N, K] matrix, or (frag: EPI_BIAS_RES and
// EPI_BIAS_RES_SHIFT) a matrix in fragment order; fp32: `w` is the caller's [K, N] matrix.  partials: float [kShiftLanes][slots][M] for EPI_BIAS_RES_SHIFT
// (rows innermost: the epilogues store and the selection reads whole lines).  ld: elements between the rows
// of a (bf16; 0 = K), ldo: of out (0 = N).
hipError_t launch_gemm(rs_dtype dt, GemmEpilogue epi, rs_dist dist, const void* a, const void* w,
                       const void* bias, const void* res, void* out, float* partials,
                       const void* ref, bool post, int64_t M, int N, int K, hipStream_t s, bool frag = false,
                       int ld = 0, int ldo = 0);
hipError_t launch_gemm_f32(GemmEpilogue epi, rs_dist dist, const void* a, const void* w, const void* bias,
                           const void* res, void* out, float* partials, const void* ref, bool post, int64_t M, int N,
                           int K, hipStream_t s);
// bf16 GEMM behind a LayerNorm (EPI_LN_BIAS / EPI_LN_BIAS_GELU), weights in fragment order.
hipError_t launch_gemm_ln(GemmEpilogue epi, const void* x, const void* w_folded, GemmLnFold ln, void* out,
                          int64_t M, int N, int K, hipStream_t s, int ld = 0, int ldo = 0);

// The MLP half of a bf16 block in one launch (mlp_fused_fits): out = x + fc2(gelu(fc1(LN(x)))), the LayerNorm folded
// into w1 as for EPI_LN_BIAS_GELU with the statistics of x formed inside; partials as for
// EPI_BIAS_RES_SHIFT (`shift`); out_stats (optional): the statistics of the rows of `out`; iota_out as in
// launch_rowstats.
struct MlpArgs {
    const void *x, *w1, *w2, *b2, *ref;
    GemmLnFold ln;  // colsum and bias of fc1
    void* out;
    float *partials, *out_stats;
    int32_t* iota_out;
    int iota_n;
    bool post;
    float eps;
    int64_t M;
    int Dm;
};
bool mlp_fused_fits(rs_dtype dt, int64_t M, int D, int Dm);
hipError_t launch_mlp_fused(const MlpArgs& g, rs_dist dist, bool shift, hipStream_t s);

// out[M, N] = LN(x) W + b for rows of 192 (qkv_rows_fits), folded as for EPI_LN_BIAS; ln.stats null: formed inside.
bool qkv_rows_fits(rs_dtype dt, int64_t M, int D, int N);
hipError_t launch_qkv_rows(const void* x, const void* w, GemmLnFold ln, void* out, int64_t M, int N, float eps, hipStream_t s);

// `count` independent bf16 products out_p[M, N] = a_p[M, K] @ wt_p[N, K]^T, problem p at element offset
// p * stride from each base pointer (K % 32 == 0, N % 64 == 0; rows of wt_p past N must exist as zeros)
hipError_t launch_gemm_batched(const void* a, const void* wt, void* out, int count, int64_t stride_a,
                               int64_t stride_w, int64_t stride_out, int M, int N, int K, hipStream_t s);

// Standard (unfused) attention with the map written to memory, the comparison system of Sec. 3.1:
// pack q, k (zero-padded to Np rows) and v^T per head; softmax rows of the [N, Np] score matrices in
// place; column sums of the map; output rows back to the caller's layout.
hipError_t launch_attn_pack(const void* q, const void* k, const void* v, void* qh, void* kh, void* vt, int B, int H,
                            int N, int Np, int64_t sb, int64_t sn, int64_t sh, hipStream_t s);
hipError_t launch_attn_softmax_rows(void* map, int64_t rows, int N, int Np, float scale_log2e, hipStream_t s);
hipError_t launch_attn_map_scores(const void* map, float* partial, float* s_cls, float* s_mean, int B, int H, int N,
                                  int Np, int cls_index, hipStream_t s);
hipError_t launch_attn_unpack(const void* oh, void* o, int B, int H, int N, int64_t osb, int64_t osn, int64_t osh,
                              hipStream_t s);

// bf16 [K, N] row-major -> [N, K] row-major
hipError_t launch_pack_transpose(const void* w, void* wt, int K, int N, hipStream_t s);
// bf16 [K, N] row-major (multiples of 64) -> fragment order (frag_off); with `gamma` ([K] bf16) row k is scaled by gamma[k]
// (product rounded to bf16); `tail` elements behind the fragments are written as zeros.
hipError_t launch_pack_frag(const void* w, const void* gamma, void* wf, int K, int N, int64_t tail, hipStream_t s);
// colsum[n] = sum_k bf16(gamma[k] * w[k][n]),  bias_out[n] = sum_k beta[k] * w[k][n] + bias[n]
// (w [K, N] bf16; gamma, beta, bias bf16 or null = 1, 0, 0; outputs fp32).
hipError_t launch_pack_ln_fold(const void* w, const void* gamma, const void* beta, const void* bias,
                               float* colsum, float* bias_out, int K, int N, hipStream_t s);

hipError_t launch_attention(rs_dtype dt, const void* q, const void* k, const void* v, void* o,
                            int B, int H, int N, int64_t sb, int64_t sn, int64_t sh,
                            int64_t osb, int64_t osn, int64_t osh, float scale, hipStream_t s);

// scores[M] = D(f_out[M, D], f_in[M, D])
hipError_t launch_shift_scores(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in,
                               float* scores, int64_t M, int D, hipStream_t s);
// scores[M] from the GEMM epilogue's partial slots
hipError_t launch_finalize_scores(rs_dist dist, const float* partials, int slots, float* scores,
                                  int64_t M, hipStream_t s);
// Scores, selection and gather of short images (select_gather_fits) in one launch; stats as in
// launch_gather_stats, or null; partials null: from the scores.
bool select_gather_fits(rs_dtype dt, int N, int D);
hipError_t launch_select_gather(rs_dtype dt, rs_dist dist, const float* partials, int slots, float* scores,
                                int32_t* kept_idx, const void* src, void* out, float* stats, int B, int N, int n_prefix,
                                int n_keep, int D, float eps, hipStream_t s);
// The same for a few longer sequences, from their scores (select_gather_long_fits; 0 < n_keep < N - n_prefix).
bool select_gather_long_fits(rs_dtype dt, int B, int N, int D);
hipError_t launch_select_gather_long(rs_dtype dt, const float* scores, int32_t* kept_idx, const void* src, void* out,
                                     float* stats, int B, int N, int n_prefix, int n_keep, int D, float eps, hipStream_t s);
// per image: the n_keep highest scores among tokens >= n_prefix, ascending kept_idx[B, K]
// the two steps above in one launch (a real selection only: n_keep < N - n_prefix, n_keep > 0;
// N must pass select_from_partials_fits)
bool select_from_partials_fits(int N);
hipError_t launch_select_from_partials(rs_dist dist, const float* partials, int slots, float* scores,
                                       int32_t* kept_idx, int B, int N, int n_prefix, int n_keep,
                                       hipStream_t s);
hipError_t launch_select(const float* scores, int32_t* kept_idx, int B, int N, int n_prefix,
                         int n_keep, hipStream_t s);
// out[b, j, :] = src[b, kept_idx[b, j], :]
hipError_t launch_gather(rs_dtype dt, const void* src, const int32_t* kept_idx, void* out, int B,
                         int N, int K, int D, hipStream_t s);
// The gather for bf16 rows of at most 4096 elements that also writes stats[B * K] = (mean,
// 1 / sqrt(variance + eps)) of every gathered row, bit-identical to launch_rowstats on `out`.
bool gather_stats_fits(rs_dtype dt, int D);
hipError_t launch_gather_stats(const void* src, const int32_t* kept_idx, void* out, float* stats, int B, int N,
                               int K, int D, float eps, hipStream_t s);

// scores, kept_idx and gathered = f_in[kept_idx] of every image in one launch that reads f_out and
// f_in once (images whose f_in rows fit a compute unit's registers, shift_topk_resident_form, and enough of
// them, shift_topk_resident_fits); its scores for any number of images: launch_shift_scores_paired
bool shift_topk_resident_form(rs_dtype dt, int N, int D);
hipError_t launch_shift_scores_paired(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in, float* scores, int64_t M,
                                      int D, hipStream_t s);
bool shift_topk_resident_fits(rs_dtype dt, int B, int N, int D);
hipError_t launch_shift_topk_resident(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in,
                                      float* scores, int32_t* kept_idx, void* gathered, int B, int N, int D,
                                      int n_prefix, int n_keep, hipStream_t s);

// 2-D grid: row_scores[b, h] = mean_w scores[b, h, w], col_scores[b, w] = mean_h scores[b, h, w]
hipError_t launch_grid_line_scores(const float* scores, float* row_scores, float* col_scores, int B, int H,
                                   int W, hipStream_t s);
// out[b, i, j, :] = src[b, kept_rows[b, i], kept_cols[b, j], :]   (src [B, H, W, C], out [B, R, Q, C])
hipError_t launch_grid_gather(rs_dtype dt, const void* src, const int32_t* kept_rows, const int32_t* kept_cols,
                              void* out, int B, int H, int W, int R, int Q, int C, hipStream_t s);

// line scores and both selections in one launch (grid_line_select_fits)
bool grid_line_select_fits(int B, int H, int W);
hipError_t launch_grid_line_select(const float* scores, float* row_scores, float* col_scores, int32_t* kept_rows,
                                   int32_t* kept_cols, int B, int H, int W, int R, int Q, hipStream_t s);
// token-wise grid pruning in two launches (grid_token_fused_fits): scores, kept_cols and (unless null) the
// compacted col_scores; then kept_rows and (unless null) the gathered map
bool grid_token_fused_fits(int64_t B, int H, int W, int Q);
hipError_t launch_grid_row_select(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in, float* scores,
                                  int32_t* kept_cols, float* col_scores, int B, int H, int W, int C, int Q, hipStream_t s);
hipError_t launch_grid_col_gather(rs_dtype dt, const void* src, const int32_t* kept_cols, const float* col_scores,
                                  int32_t* kept_rows, void* out, int B, int H, int W, int R, int Q, int C, hipStream_t s);
// token-wise grid pruning, lines of any length: col_scores[b, j, h] = scores[b, h, kept_cols[b, h, j]]
hipError_t launch_grid_compact_scores(const float* scores, const int32_t* kept_cols, float* col_scores, int B, int H,
                                      int W, int Q, hipStream_t s);
// out[b, i, j, :] = src[b, r, kept_cols[b, r, j], :], r = kept_rows[b, j, i]
hipError_t launch_grid_token_gather(rs_dtype dt, const void* src, const int32_t* kept_cols, const int32_t* kept_rows,
                                    void* out, int B, int H, int W, int R, int Q, int C, hipStream_t s);

}  // namespace rs
