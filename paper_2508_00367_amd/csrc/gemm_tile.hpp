// Device code shared by the bf16 kernels of the linear layers (gemm.hip) and of the fused MLP (mlp.hip): copies
// from memory into LDS, GELU, the shift's terms and the epilogue in the accumulator layout.
#pragma once

#include "common.hpp"

namespace rs {

// Exact-erf GELU x * Phi(x) for the bf16 epilogue: Phi(x) = sigmoid(x (a + b x^2 + c x^4)) with
// (a, b, c) fitted (minimax over [-9, 9]) to the erf form; max |error| of x * Phi(x) is 2.5e-5,
// below half a bf16 ulp of every output larger than 6e-3.  7 plain + 2 transcendental ops per
// element (libm erff: ~40) -- it matters: the fc1 epilogue runs M * Dm of them and plain ALU
// work does not overlap with the matrix cores on this chip.  The polynomial argument is
// clamped to [-10, 10] (it changes sign near |x| = 11); beyond that the sigmoid is 0 or 1 in
// fp32 anyway.  Constants carry the factor -log2(e) for v_exp_f32.
__device__ __forceinline__ float gelu_sp(float x) {
    const float xc = __builtin_amdgcn_fmed3f(x, -10.0f, 10.0f);
    const float x2 = xc * xc;
    float p = fmaf(1.0142687e-3f, x2, -0.10677576f);
    p = fmaf(p, x2, -2.3011212f);
    const float e = __builtin_amdgcn_exp2f(p * xc);  // exp(-x (a + b x^2 + c x^4))
    return x * __builtin_amdgcn_rcpf(1.0f + e);
}

// One element's contribution to the per-row sums of the shift: the same operations, in the same
// order per 8-feature chunk and over the chunks of a 64-feature slot, in every GEMM variant, so that
// the scores do not depend on which tile shape ran.
template <int DIST>
__device__ __forceinline__ void shift_term(float fo, float fi, float& p0, float& p1, float& p2) {
    if (DIST == RS_DIST_L2) { const float d = fo - fi; p0 = fmaf(d, d, p0); }
    else if (DIST == RS_DIST_L1) { p0 += fabsf(fo - fi); }
    else { p0 = fmaf(fo, fi, p0); p1 = fmaf(fo, fo, p1); p2 = fmaf(fi, fi, p2); }
}

template <int TN, int TM>
struct Frags {
    bf16x8 w[TN], a[TM];
};

typedef __attribute__((address_space(3))) void* lds_ptr;

// One wave-wide 16-byte-per-lane copy from a buffer resource straight into LDS
// (buffer_load_dwordx4 ... lds): lane l lands at lds_base + 16 * l; reads past the
// resource's size return zeros.  `voff` is the lane's byte offset, `soff` a uniform one.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rsrc, unsigned char* lds_base, int voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr)lds_base, 16, voff, soff, 0, 0);
}

// Buffer resource over the rows of ONE tile (at most 256 rows of K <= kGemmMaxK elements: under
// 2^29 bytes), so that every offset from kPastEnd upwards lies outside it and reads as zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
constexpr int kPastEnd = 0x7ff00000;

// Fragment order of the weights a block has packed: [N / 32][K / 16] fragments of 32 features x 16 k, 1 KB each, lane l's 16
// bytes of a matrix instruction's A operand in a row: feature l & 31, k 8 (l >> 5) .. + 7.  One wave-wide load of
// a fragment, into registers or LDS, is 1 KB of whole lines, and an LDS read of it meets no bank twice.
// Fragments of 32 features lie K * 64 bytes apart; features past N are past the end of a tile's resource.
__device__ __forceinline__ int frag_off(int f, int kk, int K) { return f * (K * 64) + kk * 1024; }

// s_waitcnt immediate for "at most n vector-memory operations outstanding" (gfx9 encoding,
// other counters left at their maximum).
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// ---------------------------------------------------------------------------
// Epilogue in the accumulator layout (the direct, slim and ring kernels and those of 192-wide blocks).
//
// A wave owns WM = 32 TM token rows x 64 features; lane (l32, g) holds, for row 32 j + l32 of
// every 32-row group j, features 32 i + 8 q + 4 g + e in register 4 q + e of acc[i][j].  All the
// arithmetic of the epilogue -- LayerNorm fold, bias, GELU, residual add, the per-row partial sums
// of the shift -- runs on that layout: per-row quantities (mean, rstd, the shift sums) are lane
// private, per-column vectors are the same for the 32 lanes of a half-wave.  Only the traffic with
// global memory goes through LDS, in bf16, one 4 KB region (32 rows x 128 bytes) per 32-row group:
// the residual rows arrive there by direct copies (8 lanes per 128-byte row segment), a lane picks
// up its 4 features at a time (8 bytes), puts the result back IN PLACE, and the group then leaves
// as 16 bytes per lane, 8 lanes per row segment.  An element is rounded to bf16 once, after all
// arithmetic in fp32, whatever the epilogue.
// All residual copies of the tile are requested before anything else and awaited once: vector
// memory loads and stores complete out of order with respect to each other, so "all but the
// newest n operations have completed" says nothing about a copy once output stores are in flight.
// 16-byte chunk c of row r sits in slot c ^ ((r ^ (r >> 3)) & 7).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int epi_swz(int r) { return (r ^ (r >> 3)) & 7; }

template <int TM>
struct EpiRegions {
    unsigned char* r[TM];  // one 4 KB LDS region per 32-row group of this wave
};

constexpr bool epi_ln(int epi) { return epi == EPI_LN_BIAS || epi == EPI_LN_BIAS_GELU; }
constexpr bool epi_res(int epi) { return epi == EPI_BIAS_RES || epi == EPI_BIAS_RES_SHIFT; }

// What the epilogue of one wave reads besides the accumulators: the per-column vectors of the lane's 32
// features and the LayerNorm statistics of its TM rows.  The bias stays as it is in memory until it is
// used, and nothing here depends on a loaded value: all the loads are in flight together.
template <int TM, int EPI>
struct EpiVecs {
    static constexpr bool LN = epi_ln(EPI);
    f32x4 bv[LN ? 2 : 1][4], cs[LN ? 2 : 1][4];
    u32x2 raw[LN ? 1 : 2][4];
    float2 stats[LN ? TM : 1];
    __device__ __forceinline__ void load(const bf16raw* __restrict__ bias, const GemmLnFold& ln, int M, int N, int m_base,
                                         int n_base, int lane) {
        const int l32 = lane & 31, g = lane >> 5;
        n_base = n_base < N ? n_base : 0;  // a wave's 64 features are all inside N or all outside (N % 64 == 0)
        if constexpr (LN) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = n_base + i * 32 + q * 8 + g * 4;
                    bv[i][q] = *reinterpret_cast<const f32x4*>(ln.bias + n);
                    cs[i][q] = *reinterpret_cast<const f32x4*>(ln.colsum + n);
                }
#pragma unroll
            for (int j = 0; j < TM; ++j)  // rows past M are computed on a copy and never stored
                stats[j] = reinterpret_cast<const float2*>(ln.stats)[min(m_base + j * 32 + l32, M - 1)];
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) raw[i][q] = u32x2{0u, 0u};
            if (bias) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        raw[i][q] = *reinterpret_cast<const u32x2*>(bias + n_base + i * 32 + q * 8 + g * 4);
            }
        }
    }
    // The LayerNorm vectors from LDS: 1 KB each of colsum and bias' of the tile's 256 features and of the statistics of its 128
    // rows, this wave's 64 features from `f0` on (request() below has fetched them).
    __device__ __forceinline__ void from_lds(const unsigned char* s, int f0, int lane) {
        const int l32 = lane & 31, g = lane >> 5;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = (f0 + i * 32 + q * 8 + g * 4) * 4;
                cs[LN ? i : 0][q] = *reinterpret_cast<const f32x4*>(s + at);
                bv[LN ? i : 0][q] = *reinterpret_cast<const f32x4*>(s + 1024 + at);
            }
#pragma unroll
        for (int j = 0; j < TM; ++j) stats[LN ? j : 0] = *reinterpret_cast<const float2*>(s + 2048 + (j * 32 + l32) * 8);
    }
    // One copy per wave (waves 0, 1, 2) into the 3 KB at `s`; past N and M zeros, of which nothing is stored.
    static __device__ __forceinline__ void request(unsigned char* s, const GemmLnFold& ln, int M, int N, int m0, int n0, int wave, int lane) {
        const int f = min(N - n0, 256) * 4;
        const __amdgpu_buffer_rsrc_t rs = wave == 0 ? make_rsrc(ln.colsum + n0, f) : wave == 1 ? make_rsrc(ln.bias + n0, f)
                                                    : make_rsrc(ln.stats + 2 * (int64_t)m0, min(M - m0, 128) * 8);
        if (wave < 3) dma16(rs, s + wave * 1024, lane * 16, 0);
    }
    __device__ __forceinline__ float bias_at(int i, int q, int e) const {
        if constexpr (LN) return bv[i][q][e];
        else return __uint_as_float((e & 1) ? (raw[i][q][e >> 1] & 0xffff0000u) : (raw[i][q][e >> 1] << 16));
    }
};

// Requests the residual rows of a wave tile: per 32-row group 4 copies of 8 rows x 128 bytes (lane l:
// row l / 8, slot l % 8 holds chunk (l % 8) ^ swz(row)); rows past M, and every row when the wave's features
// lie past N, read as zeros through the resource.
template <int TM>
__device__ __forceinline__ void epi_request_residual(const EpiRegions<TM>& reg, const bf16raw* __restrict__ res, int M, int N,
                                                     int m_base, int n_base, int lane) {
    const int rows_valid = n_base < N ? min(max(M - m_base, 0), 32 * TM) : 0;
    const __amdgpu_buffer_rsrc_t rs_res =
        make_rsrc(rows_valid > 0 ? res + (int64_t)m_base * N + n_base : res, rows_valid > 0 ? ((int64_t)(rows_valid - 1) * N + 64) * 2 : 0);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int r = p * 8 + (lane >> 3);
        const int voff = (r * N + (((lane & 7) ^ epi_swz(r)) << 3)) * 2;
#pragma unroll
        for (int j = 0; j < TM; ++j) dma16(rs_res, reg.r[j] + p * 1024, voff, j * 32 * N * 2);
    }
}

// The arithmetic and the stores.  The residual rows have landed in the regions.
template <int TM, int EPI, int DIST>
__device__ __forceinline__ void gemm_epilogue_acc_layout(
    f32x16 (&acc)[2][TM], const EpiRegions<TM>& reg, const EpiVecs<TM, EPI>& vec, bf16raw* __restrict__ out,
    float* __restrict__ partials, const bf16raw* __restrict__ ref, int post,
    int M, int N, int ldo, int slots, int64_t ldp, int m_base /* first row of the wave tile */, int n_base /* first feature */,
    int lane) {
    constexpr bool LN = epi_ln(EPI);
    constexpr bool GELU = EPI == EPI_BIAS_GELU || EPI == EPI_LN_BIAS_GELU;
    constexpr bool RES = epi_res(EPI);
    constexpr bool SHIFT = EPI == EPI_BIAS_RES_SHIFT;
    if (n_base >= N || m_base >= M) return;
    const int l32 = lane & 31, g = lane >> 5;

    const int sw = epi_swz(l32);
    const __amdgpu_buffer_rsrc_t rs_out =  // the wave tile's rows inside M
        make_rsrc(out + (int64_t)m_base * ldo + n_base, ((int64_t)(min(M - m_base, 32 * TM) - 1) * ldo + 64) * 2);
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int m = m_base + j * 32 + l32;
        const bool m_ok = m < M;
        const float2 st = vec.stats[LN ? j : 0];
        unsigned char* buf = reg.r[j];
        // Shift sums of the row's 64 features: per chunk of 8 features a running sum in feature order
        // (half-wave g = 0 holds the first four terms and hands its sum to g = 1, which goes on with
        // the other four), then the 8 chunk sums pairwise (c, c ^ 4), (.., c ^ 2), (.., c ^ 1).
        float pc0[8], pc1[DIST == RS_DIST_COS ? 8 : 1], pc2[DIST == RS_DIST_COS ? 8 : 1];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned char* at = buf + l32 * 128 + (((i * 4 + q) ^ sw) << 4) + g * 8;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a_ = acc[i][j][4 * q + e];
                    v[e] = LN ? fmaf(st.y, fmaf(-st.x, vec.cs[LN ? i : 0][q][e], a_), vec.bias_at(i, q, e)) : a_ + vec.bias_at(i, q, e);
                    if (GELU) v[e] = gelu_sp(v[e]);
                }
                if (RES) {
                    const uint2 r2 = *reinterpret_cast<const uint2*>(at);
                    float rr[4] = {__uint_as_float(r2.x << 16), __uint_as_float(r2.x & 0xffff0000u),
                                   __uint_as_float(r2.y << 16), __uint_as_float(r2.y & 0xffff0000u)};
                    if (SHIFT) {
                        // D(f_out, f_in): f_out is the branch output, or (post) the residual stream after
                        // the add; f_in is the residual operand, or `ref` when one is given
                        float fi[4] = {rr[0], rr[1], rr[2], rr[3]};
                        if (ref && m_ok) {
                            const uint2 f2 = *reinterpret_cast<const uint2*>(ref + (int64_t)m * N + n_base + i * 32 + q * 8 + g * 4);
                            fi[0] = __uint_as_float(f2.x << 16); fi[1] = __uint_as_float(f2.x & 0xffff0000u);
                            fi[2] = __uint_as_float(f2.y << 16); fi[3] = __uint_as_float(f2.y & 0xffff0000u);
                        }
                        float s0 = 0.f, s1 = 0.f, s2 = 0.f;
                        if (m_ok) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) shift_term<DIST>(post ? v[e] + rr[e] : v[e], fi[e], s0, s1, s2);
                        }
                        // g = 1 restarts from the sum of g = 0 (its own first pass is discarded)
                        const float h0 = half_pair(s0).x;
                        float t0 = h0, t1 = 0.f, t2 = 0.f;
                        if (DIST == RS_DIST_COS) { t1 = half_pair(s1).x; t2 = half_pair(s2).x; }
                        if (m_ok) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) shift_term<DIST>(post ? v[e] + rr[e] : v[e], fi[e], t0, t1, t2);
                        }
                        pc0[i * 4 + q] = t0;
                        if (DIST == RS_DIST_COS) { pc1[DIST == RS_DIST_COS ? i * 4 + q : 0] = t1; pc2[DIST == RS_DIST_COS ? i * 4 + q : 0] = t2; }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += rr[e];
                }
                uint2 w2;
                w2.x = pack2bf(v[0], v[1]);
                w2.y = pack2bf(v[2], v[3]);
                *reinterpret_cast<uint2*>(at) = w2;  // in place: this lane alone reads and writes these 8 bytes
            }
        if (SHIFT) {
            if (g == 1 && m_ok) {  // the half-wave that holds the complete chunk sums
                float* dst = partials + (n_base >> 6) * ldp + m;
                dst[0] = ((pc0[0] + pc0[4]) + (pc0[2] + pc0[6])) + ((pc0[1] + pc0[5]) + (pc0[3] + pc0[7]));
                if (DIST == RS_DIST_COS) {
                    constexpr int C = DIST == RS_DIST_COS ? 1 : 0;
                    dst[slots * ldp] = ((pc1[0] + pc1[4 * C]) + (pc1[2 * C] + pc1[6 * C])) + ((pc1[1 * C] + pc1[5 * C]) + (pc1[3 * C] + pc1[7 * C]));
                    dst[2 * slots * ldp] = ((pc2[0] + pc2[4 * C]) + (pc2[2 * C] + pc2[6 * C])) + ((pc2[1 * C] + pc2[5 * C]) + (pc2[3 * C] + pc2[7 * C]));
                }
            }
        }
        // the group leaves as 16 bytes per lane (LDS accesses of one wave are served in order)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = p * 8 + (lane >> 3), cc = lane & 7;
            const uint4 o4 = *reinterpret_cast<const uint4*>(buf + r * 128 + ((cc ^ epi_swz(r)) << 4));
            const int mo = m_base + j * 32 + r;
            store16_wt(rs_out, mo < M ? ((j * 32 + r) * ldo + cc * 8) * 2 : kPastEnd, o4);
        }
    }
}

}  // namespace rs
