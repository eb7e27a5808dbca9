// Fused multi-head self-attention, Eq. (1) of Sec. 3.1:  O = Softmax(Q K^T * scale) V
// per (image, head), head width 64.  The N x N attention map is never stored: K/V
// stream through LDS in tiles of 64 keys while each wavefront keeps a running row
// maximum, row sum and output accumulator in registers (online softmax).
//
// bf16 path (v_mfma_f32_32x32x16_bf16).  Everything is computed transposed so that the
// softmax state of a query row lives in ONE lane:
//     S^T = K Q^T     A operand = K rows from LDS, B operand = Q rows held in registers;
//                     accumulator: lane (q = lane%32, g = lane/32) holds, for its query q,
//                     keys 8j + 4g + i  (register 4j + i)  of each 32-key block.
//     O^T = V^T P^T   B operand = P taken straight from the S^T accumulator registers
//                     (8 registers = the lane's 8 keys of a 16-key group), A operand = V^T.
//                     V sits in LDS as it sits in memory, one row per key; the transposing
//                     LDS read of gfx950 (ds_read_b64_tr_b16) hands a lane one channel at 4
//                     keys, and two of them fetch the 8 keys in the order the accumulator
//                     layout yields them (slot 4u + i  <->  key 8u + 4g + i of the group).
// Row max / row sum need one exchange between the two half-waves per tile.
//
// fp32 path (v_mfma_f32_32x32x2_f32, parity configuration): the same transposed form.
#include <float.h>

#include "common.hpp"
#include "attention_choice.hpp"

namespace rs {

constexpr int ATT_BN = 64;   // keys per tile
constexpr int DH = 64;

// 16-byte chunk `c` (0..7) of 128-byte LDS row `r` of a K tile; the XOR spreads the 16-lane
// operand reads over the 64 banks.
__device__ __forceinline__ int att_swz(int r, int c) { return r * 128 + (((c ^ r ^ (r >> 3)) & 7) << 4); }

typedef __attribute__((address_space(3))) void* att_lds_ptr;
// 16 bytes per lane from a buffer resource straight into LDS (lane l at dst + 16 l)
__device__ __forceinline__ void att_copy(__amdgpu_buffer_rsrc_t rsrc, unsigned char* dst, int voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (att_lds_ptr)dst, 16, voff, soff, 0, 0);
}
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16* lds_v4i16;

// Row-major V tile [64 keys][128 B]: 16-byte chunk c of key row r sits in slot c ^ att_vswz(r).  A
// transposing read touches 4 consecutive key rows x 64 bytes per 32 lanes; flipping the 64-byte
// half on every second pair of rows keeps those four rows on different banks.
__device__ __forceinline__ int att_vswz(int r) { return ((r >> 1) & 1) << 2; }

// One block of 32 query rows against one resident tile of 64 keys: S^T = K Q^T, online softmax
// in registers (one lane = one query row, half of the tile's keys), O^T += V^T P^T.
// `sk`: K tile [64 keys][128 B] (att_swz); `sv`: V tile [64 keys][128 B] (att_vswz).
template <bool MASK>
__device__ __forceinline__ void att_tile(const unsigned char* sk, const unsigned char* sv,
                                         const bf16x8 (&qf)[4], f32x16 (&oacc)[2], float& m_run,
                                         float& l_run, int key0, int N, float scale_log2e, int l32, int g) {
    // In the padded last tile only the 32-key blocks and 16-key groups that hold real keys are
    // worked on (wave-uniform conditions): N = 197 leaves 5 keys in its fourth tile.
    const int valid = MASK ? N - key0 : ATT_BN;  // real keys in this tile, 1 .. 64
    f32x16 sacc[2];
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[kb2][r] = 0.f;
    if (!MASK || valid > 32) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int kb2 = 0; kb2 < 2; ++kb2) {  // independent accumulator chains alternate
                const bf16x8 kf = *reinterpret_cast<const bf16x8*>(sk + att_swz(kb2 * 32 + l32, kk * 2 + g));
                sacc[kb2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk], sacc[kb2], 0, 0, 0);
            }
    } else {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const bf16x8 kf = *reinterpret_cast<const bf16x8*>(sk + att_swz(l32, kk * 2 + g));
            sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk], sacc[0], 0, 0, 0);
        }
    }
    if (MASK) {  // keys past the end
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = key0 + kb2 * 32 + (r >> 2) * 8 + g * 4 + (r & 3);
                if (key >= N) sacc[kb2][r] = -INFINITY;
            }
    }
    float mx = fmaxf(sacc[0][0], sacc[1][0]);
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(fmaxf(mx, sacc[0][r]), sacc[1][r]);
    mx = half_max(mx);
    const float m_new = fmaxf(m_run, mx);  // finite: every tile holds at least one real key
    const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2e);
    const float mb = m_new * scale_log2e;
    m_run = m_new;
    if (!MASK || valid > 32) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sacc[0][r] = __builtin_amdgcn_exp2f(fmaf(sacc[0][r], scale_log2e, -mb));
            sacc[1][r] = __builtin_amdgcn_exp2f(fmaf(sacc[1][r], scale_log2e, -mb));
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[0][r] = __builtin_amdgcn_exp2f(fmaf(sacc[0][r], scale_log2e, -mb));
    }
    if (__ballot(alpha != 1.0f)) {  // the running maximum moved for some row of this block
        // in-place multiplies: with plain C++ the compiler renames the 32 accumulators on this
        // rarely taken path and pays 32 register copies on EVERY tile to merge the two paths
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float t = oacc[i][r];
                asm volatile("v_mul_f32 %0, %0, %1" : "+v"(t) : "v"(alpha));
                oacc[i][r] = t;
            }
    }
    // P goes to bf16 once; the row sum is taken over the same rounded values (v_dot2 with ones)
    float psum = 0.f;
    const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (MASK && 16 * t >= valid) break;  // groups of padding keys only: P = 0
        const int kb2 = t >> 1, r0 = (t & 1) * 8;
        union { uint32_t u[4]; bf16x8 v; } pf;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pf.u[e] = pack2bf(sacc[kb2][r0 + 2 * e], sacc[kb2][r0 + 2 * e + 1]);
            psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pf.u[e]), ones, psum, false);
        }
#pragma unroll
        for (int db = 0; db < 2; ++db) {
            // V tile as it sits in memory, [64 keys][64 channels]: two transposing LDS reads
            // (ds_read_b64_tr_b16) hand this lane its channel's values at 4 keys each.  Within a
            // group of 16 lanes, lane s = 4 j + a points at key j, channels 4 a .. 4 a + 3, and
            // lane L receives channel L of keys j = 0 .. 3.  The keys are taken in the order of
            // the P operand: slot 4 u + j of this lane is key 16 t + 8 u + 4 g + j.
            const int s16 = l32 & 15;
            const int chunk = db * 4 + 2 * (l32 >> 4) + ((s16 & 3) >> 1);
            union { v4i16 h[2]; bf16x8 v; } tr;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int key = 16 * t + 8 * u + 4 * g + (s16 >> 2);
                tr.h[u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_v4i16)(sv + key * 128 + ((chunk ^ att_vswz(key)) << 4) + (s16 & 1) * 8));
            }
            oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr.v, pf.v, oacc[db], 0, 0, 0);
        }
    }
    l_run = l_run * alpha + psum;
}

// Normalises and stores a wave's 32 output rows (lane: O[row l32][db*32 + 8j + 4g + i] in oacc[db][4j + i]) through 4 KB of
// LDS that nobody else reads any more, so that rows leave as whole 128-byte lines: straight from the accumulators a store
// covers 16 bytes of each of 32 lines.  `o`: row 0 of the wave, `rows` of them inside N.
constexpr int64_t ATT_O_FAR = (int64_t)1 << 24;  // output row stride (elements) at which 32 rows leave 32-bit byte offsets
__device__ __forceinline__ void att_store(const f32x16 (&oacc)[2], float inv, unsigned char* buf, bf16raw* __restrict__ o,
                                          int64_t osn, int rows, int lane) {
    const int l32 = lane & 31, g = lane >> 5;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint2 w;
            w.x = pack2bf(oacc[db][4 * j] * inv, oacc[db][4 * j + 1] * inv);
            w.y = pack2bf(oacc[db][4 * j + 2] * inv, oacc[db][4 * j + 3] * inv);
            *reinterpret_cast<uint2*>(buf + att_swz(l32, db * 4 + j) + g * 8) = w;
        }
    const __amdgpu_buffer_rsrc_t rs_o =
        __builtin_amdgcn_make_buffer_rsrc(o, 0, osn < ATT_O_FAR ? (int)(((rows - 1) * osn + DH) * 2) : 0, 0x00020000);
#pragma unroll
    for (int p = 0; p < 4; ++p) {  // LDS accesses of one wave are served in order
        const int r = p * 8 + (lane >> 3), c = lane & 7;
        const uint4 v = *reinterpret_cast<const uint4*>(buf + att_swz(r, c));
        if (osn < ATT_O_FAR) store16_wt(rs_o, r < rows ? (int)(r * osn + c * 8) * 2 : 0x7ff00000, v);
        else if (r < rows) *reinterpret_cast<uint4*>(o + r * osn + c * 8) = v;
    }
}

// The same straight from the accumulators, 8 bytes per lane and row: no barrier and no trip through LDS before the stores.
__device__ __forceinline__ void att_store_direct(const f32x16 (&oacc)[2], float inv, bf16raw* __restrict__ o, int64_t osn, int rows, int lane) {
    const int l32 = lane & 31, g = lane >> 5;
    if (l32 >= rows) return;
    bf16raw* row = o + l32 * osn + g * 4;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint2 w;
            w.x = pack2bf(oacc[db][4 * j] * inv, oacc[db][4 * j + 1] * inv);
            w.y = pack2bf(oacc[db][4 * j + 2] * inv, oacc[db][4 * j + 3] * inv);
            *reinterpret_cast<uint2*>(row + db * 32 + j * 8) = w;
        }
}

// Long sequences: workgroup = 256 or 128 query rows (NW = 8 or 4 waves x 32 rows) of one (image, head); two or
// four workgroups share a CU (at most 128 registers), four waves per SIMD.  K and V tiles stream
// global -> LDS directly (buffer_load ... lds, rows past N read as zero through the buffer
// resource).  Two stages each; the copies of tile t+1 are issued before the MFMAs of tile t, one barrier per tile.
template <int NW>
__global__ __launch_bounds__(NW * 64, 4) void attention_bf16_kernel(
    const bf16raw* __restrict__ q, const bf16raw* __restrict__ k, const bf16raw* __restrict__ v,
    bf16raw* __restrict__ o, int N, int64_t sb, int64_t sn, int64_t sh, int64_t osb, int64_t osn,
    int64_t osh, float scale_log2e, int H, int BH, int q_tiles) {
    __shared__ __attribute__((aligned(1024))) unsigned char sk0[ATT_BN * 128];
    __shared__ __attribute__((aligned(1024))) unsigned char sk1[ATT_BN * 128];
    __shared__ __attribute__((aligned(16))) unsigned char sv0[DH * 128];
    __shared__ __attribute__((aligned(16))) unsigned char sv1[DH * 128];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    // Workgroup ids go round-robin to the 8 XCDs; all query tiles of one (image, head) are given
    // to the same XCD so that its K/V tiles are fetched into that XCD's L2 once and hit afterwards.
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int head = xcd + 8 * (local / q_tiles);
    if (head >= BH) return;  // whole workgroup, before any barrier
    const int b = head / H, h = head - b * H;
    const int q0 = (local % q_tiles) * (NW * 32) + wave * 32;
    const int64_t base = (int64_t)b * sb + (int64_t)h * sh;

    // Q fragments: B operand, column = query row q0 + l32, k-slots = 8 channels 16*kk + 8*g ..
    bf16x8 qf[4];
    {
        int qr = q0 + l32;
        qr = qr < N ? qr : N - 1;  // rows past the end are computed on a copy and never stored
        const bf16raw* qp = q + base + (int64_t)qr * sn;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16 + g * 8);
    }

    // K copies: copy i of wave w fills LDS rows 8 (w + NW i) .. + 7 of the tile (lane l: row l/8, slot l%8 holds
    // chunk (l%8) ^ f(row)); the resource ends with key N-1, so later rows arrive as zeros.
    constexpr int CP = 8 / NW;
    const int64_t k_bytes = ((int64_t)(N - 1) * sn + DH) * 2;
    const __amdgpu_buffer_rsrc_t rs_k = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16raw*>(k + base), 0, (int)(k_bytes < 0xffffffffll ? k_bytes : 0xffffffffll), 0x00020000);
    const int k_lr = lane >> 3;
    int k_voff[CP];
#pragma unroll
    for (int i = 0; i < CP; ++i)
        k_voff[i] = (int)(((int64_t)((wave + NW * i) * 8 + k_lr) * sn + (((lane & 7) ^ k_lr ^ (wave + NW * i)) << 3)) * 2);
    const int k_tile_bytes = (int)(ATT_BN * sn * 2);

    // V copies: the same rows and lanes as K, chunk (l%8) ^ att_vswz(row) in slot l%8.
    const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16raw*>(v + base), 0, (int)(k_bytes < 0xffffffffll ? k_bytes : 0xffffffffll), 0x00020000);
    const int v_voff = (int)(((int64_t)(wave * 8 + k_lr) * sn + (((lane & 7) ^ att_vswz(k_lr)) << 3)) * 2);
    const int v_pass = (int)(NW * 8 * sn * 2);

#define ATT_LOAD_NEXT(SKn, SVn, kt_)                                                                     \
    _Pragma("unroll") for (int i = 0; i < CP; ++i) {                                                     \
        att_copy(rs_k, (SKn) + (wave + NW * i) * 1024, k_voff[i], (kt_) * k_tile_bytes);                 \
        att_copy(rs_v, (SVn) + (wave + NW * i) * 1024, v_voff, (kt_) * k_tile_bytes + i * v_pass);       \
    }
// tile kt_ is resident in (SKc, SVc); tile kt_+1 is fetched into (SKn, SVn) meanwhile
#define ATT_STEP(SKc, SVc, SKn, SVn, kt_, MASK_)                                                              \
    {                                                                                                    \
        ATT_LOAD_NEXT(SKn, SVn, (kt_) + 1)                                                               \
        if (active)                                                                                      \
            att_tile<MASK_>(SKc, SVc, qf, oacc, m_run, l_run, (kt_) * ATT_BN, N, scale_log2e, l32, g);   \
        __builtin_amdgcn_s_waitcnt(0x0F70); /* this wave's K and V copies have landed */                 \
        __syncthreads();                                                                                 \
    }

    f32x16 oacc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
    float m_run = -INFINITY;  // running max of the raw logits of this lane's query row
    float l_run = 0.f;        // this lane's share of the running row sum

    // A wave whose query rows all lie past N (last query tile of a head) copies its share of the
    // K/V tiles and meets the barriers but computes nothing: the wave it shares a SIMD with then
    // has that SIMD to itself.
    const bool active = q0 < N;
    const int KT = (N + ATT_BN - 1) / ATT_BN;
    ATT_LOAD_NEXT(sk0, sv0, 0)
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    const int KF = N / ATT_BN;  // tiles without padding keys
    int kt = 0;
    for (; kt + 2 <= KF; kt += 2) {
        ATT_STEP(sk0, sv0, sk1, sv1, kt, false)
        ATT_STEP(sk1, sv1, sk0, sv0, kt + 1, false)
    }
    if (kt < KT) {  // one or two tiles left, the last one possibly padded
        ATT_STEP(sk0, sv0, sk1, sv1, kt, true)
        if (kt + 1 < KT) ATT_STEP(sk1, sv1, sk0, sv0, kt + 1, true)
    }
#undef ATT_LOAD_NEXT
#undef ATT_STEP

    // every wave is past its last tile: the stages are free
    if (!active) return;
    const float l_tot = half_sum(l_run);
    unsigned char* const buf = (NW == 4 ? (wave < 2 ? sk0 : sk1) : wave < 2 ? sk0 : wave < 4 ? sk1 : wave < 6 ? sv0 : sv1) + (wave & 1) * 4096;
    att_store(oacc, 1.0f / l_tot, buf, o + (int64_t)b * osb + (int64_t)q0 * osn + (int64_t)h * osh, osn, min(N - q0, 32), lane);
}

// ---------------------------------------------------------------------------
// Last rows of a long sequence.  When N leaves a few rows (at most 64) beyond the last full
// query tile, a whole workgroup of the kernel above would stream every K/V tile for them with
// one or two of its eight waves working.  Here one workgroup per (image, head) takes those rows
// and its eight waves split the KEY tiles instead (wave w: tiles w, w + 8, ...), each with its
// own K / V tile in LDS and no workgroup barrier inside the loop; the eight partial results
// (running maximum, row sum, unnormalised output) are merged through LDS in wave order, so the
// result does not depend on timing.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(512, 2) void attention_bf16_tail_kernel(
    const bf16raw* __restrict__ q, const bf16raw* __restrict__ k, const bf16raw* __restrict__ v,
    bf16raw* __restrict__ o, int N, int64_t sb, int64_t sn, int64_t sh, int64_t osb, int64_t osn,
    int64_t osh, float scale_log2e, int H, int q_begin) {
    // per wave: K tile (8 KB) + V tile (8 KB); after the loop the same 16 KB hold the wave's
    // output partial [2 blocks][32 rows][64 channels] fp32
    __shared__ __attribute__((aligned(1024))) unsigned char s_tiles[8][16384];
    __shared__ float s_m[8][2][32];
    __shared__ float s_l[8][2][32];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int b = blockIdx.x / H, h = blockIdx.x - b * H;
    const int64_t base = (int64_t)b * sb + (int64_t)h * sh;
    unsigned char* sk = s_tiles[wave];
    unsigned char* svt = sk + ATT_BN * 128;

    bf16x8 qf[2][4];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        int qr = q_begin + qb * 32 + l32;
        qr = qr < N ? qr : N - 1;  // rows past the end are computed on a copy and never stored
        const bf16raw* qp = q + base + (int64_t)qr * sn;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) qf[qb][kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16 + g * 8);
    }
    const int64_t k_bytes = ((int64_t)(N - 1) * sn + DH) * 2;
    const __amdgpu_buffer_rsrc_t rs_k = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16raw*>(k + base), 0, (int)(k_bytes < 0xffffffffll ? k_bytes : 0xffffffffll), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16raw*>(v + base), 0, (int)(k_bytes < 0xffffffffll ? k_bytes : 0xffffffffll), 0x00020000);
    const int k_lr = lane >> 3;
    const int k_tile_bytes = (int)(ATT_BN * sn * 2);

    f32x16 oacc[2][2];
    float m_run[2], l_run[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[qb][i][r] = 0.f;
        m_run[qb] = -INFINITY;
        l_run[qb] = 0.f;
    }

    const bool second = N - q_begin > 32;  // rows in the second block of 32
    const int KT = (N + ATT_BN - 1) / ATT_BN;
    for (int kt = wave; kt < KT; kt += 8) {
        // K tile: copy i fills rows 8i .. 8i+7 (lane l: row l/8, slot l%8 holds chunk (l%8) ^ f(row))
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int voff = (int)(((int64_t)(i * 8 + k_lr) * sn + (((lane & 7) ^ k_lr ^ i) << 3)) * 2);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_k, (att_lds_ptr)(sk + i * 1024), 16, voff, kt * k_tile_bytes, 0, 0);
        }
        // V tile: the same rows and lanes, chunk (l%8) ^ att_vswz(row) in slot l%8
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int voff = (int)(((int64_t)(i * 8 + k_lr) * sn + (((lane & 7) ^ att_vswz(k_lr)) << 3)) * 2);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_v, (att_lds_ptr)(svt + i * 1024), 16, voff, kt * k_tile_bytes, 0, 0);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's K and V copies have landed
        // one block of 32 rows at a time: fewer live registers than both at once, and LDS
        // bandwidth is not what limits this kernel
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            if (qb == 1 && !second) break;  // at most 32 rows left: the second block has none
            if (kt == KT - 1 && (N & (ATT_BN - 1)))
                att_tile<true>(sk, svt, qf[qb], oacc[qb], m_run[qb], l_run[qb], kt * ATT_BN, N, scale_log2e, l32, g);
            else
                att_tile<false>(sk, svt, qf[qb], oacc[qb], m_run[qb], l_run[qb], kt * ATT_BN, N, scale_log2e, l32, g);
        }
    }

    // ---- merge the eight partials
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const float l_tot = half_sum(l_run[qb]);
        if (g == 0) {
            s_m[wave][qb][l32] = m_run[qb];
            s_l[wave][qb][l32] = l_tot;
        }
    }
    __syncthreads();  // every wave has left its tiles: the partials may overwrite them
    float* part = reinterpret_cast<float*>(s_tiles[wave]);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        if (qb == 1 && !second) break;  // its rows are never stored
        float m_tot = s_m[0][qb][l32];
#pragma unroll
        for (int w = 1; w < 8; ++w) m_tot = fmaxf(m_tot, s_m[w][qb][l32]);
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w)
            L += s_l[w][qb][l32] * __builtin_amdgcn_exp2f((s_m[w][qb][l32] - m_tot) * scale_log2e);
        const float f = __builtin_amdgcn_exp2f((m_run[qb] - m_tot) * scale_log2e) / L;  // 0 for a wave without tiles
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int slot = db * 8 + 2 * j + g;  // 4 channels db*32 + 8j + 4g ..
                const f32x4 val = {oacc[qb][db][4 * j] * f, oacc[qb][db][4 * j + 1] * f,
                                   oacc[qb][db][4 * j + 2] * f, oacc[qb][db][4 * j + 3] * f};
                *reinterpret_cast<f32x4*>(part + (qb * 32 + l32) * 64 + ((slot ^ (l32 & 15)) << 2)) = val;
            }
    }
    __syncthreads();
    {
        const int r = tid >> 3, c8 = tid & 7;  // row of the 64, channels 8 c8 .. 8 c8 + 7
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const float* pw = reinterpret_cast<const float*>(s_tiles[w]) + r * 64;
            const f32x4 lo = *reinterpret_cast<const f32x4*>(pw + (((2 * c8) ^ (r & 15)) << 2));
            const f32x4 hi = *reinterpret_cast<const f32x4*>(pw + (((2 * c8 + 1) ^ (r & 15)) << 2));
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[e] += lo[e]; acc[4 + e] += hi[e]; }
        }
        const int qr = q_begin + r;
        if (qr < N) Elem<bf16raw>::store8(o + (int64_t)b * osb + (int64_t)qr * osn + (int64_t)h * osh + c8 * 8, acc);
    }
}

// ---------------------------------------------------------------------------
// Short sequences (N <= 256, every image-classification block): one workgroup of 8 waves per
// (image, head).  K and V (N x 64 each) of the head are copied into LDS once; wave w runs query
// rows 32w .. 32w+31 against all key tiles.  The copies are requested in tile order and the
// first two tiles are used as soon as they have landed, while the other two still stream in:
// two barriers in all.  Against the tiled kernel this reads K and V once instead of once per
// query tile and has no per-tile barrier; two workgroups share a CU, so one's load phase runs
// under the other's tile loop.  The tile loop itself is bound by instruction issue (plain ALU
// and matrix instructions of a SIMD's waves do not overlap), so it carries no masking work
// outside the last key tile.
// LDS: K and V rows of 128 bytes in the tiled kernel's two slot orders (att_swz, att_vswz).
// ---------------------------------------------------------------------------
constexpr int SM_MAXN = 256, SM_DIRECT = 48;

__global__ __launch_bounds__(512, 4) void attention_bf16_small_kernel(
    const bf16raw* __restrict__ q, const bf16raw* __restrict__ k, const bf16raw* __restrict__ v,
    bf16raw* __restrict__ o, int N, int64_t sb, int64_t sn, int64_t sh, int64_t osb, int64_t osn,
    int64_t osh, float scale_log2e, int q_waves) {
    // one array per half and operand: the compiler then knows which copies a half's LDS reads wait for
    __shared__ __attribute__((aligned(1024))) unsigned char s_ka[2 * ATT_BN * 128], s_kb[2 * ATT_BN * 128];
    __shared__ __attribute__((aligned(1024))) unsigned char s_va[2 * ATT_BN * 128], s_vb[2 * ATT_BN * 128];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int b = blockIdx.y, h = blockIdx.x;
    const int64_t base = (int64_t)b * sb + (int64_t)h * sh;
    const int KT = (N + ATT_BN - 1) / ATT_BN;   // key tiles of 64
    const int KF = N / ATT_BN;                  // tiles without padding keys: no masking work in them

    const int q0 = wave < q_waves ? (blockIdx.z * q_waves + wave) * 32 : N;  // N: copies only
    // Q fragments (B operand): column = query row q0 + l32, k-slots = channels 16 kk + 8 g ..
    bf16x8 qf[4];
    {
        int qr = q0 + l32;
        qr = qr < N ? qr : N - 1;
        const bf16raw* qp = q + base + (int64_t)qr * sn;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16 + g * 8);
    }
    // K and V of the head go from memory straight into LDS: per tile of 64 keys, wave w copies
    // rows 8w .. 8w+7 (lane l: row l/8, 16-byte slot l%8).  Both resources end with key N-1, so
    // rows past the end arrive as zeros without touching memory: zero V rows add nothing, and
    // the padded keys' logits are masked in the last tile.  All four tiles are always requested,
    // in tile order, so that "all but the newest 2 (3 - i) copies" means "tile i has landed".
    const int64_t k_bytes = ((int64_t)(N - 1) * sn + DH) * 2;
    const __amdgpu_buffer_rsrc_t rs_k = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16raw*>(k + base), 0, (int)(k_bytes < 0xffffffffll ? k_bytes : 0xffffffffll), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16raw*>(v + base), 0, (int)(k_bytes < 0xffffffffll ? k_bytes : 0xffffffffll), 0x00020000);
    const int k_lr = lane >> 3;
    const int k_voff = (int)(((int64_t)(wave * 8 + k_lr) * sn + (((lane & 7) ^ k_lr ^ wave) << 3)) * 2);
    const int v_voff = (int)(((int64_t)(wave * 8 + k_lr) * sn + (((lane & 7) ^ att_vswz(k_lr)) << 3)) * 2);
    const int k_tile_bytes = (int)(ATT_BN * sn * 2);
#define SM_COPY(SK, SV, i_)                                                                                       \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_k, (att_lds_ptr)((SK) + wave * 1024), 16, k_voff, (i_) * k_tile_bytes, 0, 0); \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_v, (att_lds_ptr)((SV) + wave * 1024), 16, v_voff, (i_) * k_tile_bytes, 0, 0);
    SM_COPY(s_ka, s_va, 0)
    SM_COPY(s_ka + ATT_BN * 128, s_va + ATT_BN * 128, 1)
    SM_COPY(s_kb, s_vb, 2)
    SM_COPY(s_kb + ATT_BN * 128, s_vb + ATT_BN * 128, 3)
#undef SM_COPY

    f32x16 oacc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // The first two tiles are used as soon as every wave's share of them has landed; the other
    // two keep streaming in meanwhile.  Waves without query rows (q0 >= N) still wait and meet
    // the barriers: the others read the rows they copied.
#define SM_HALF(SK, SV, t0_, WAIT)                                                                                \
    if ((t0_) < KT) {                                                                                             \
        __builtin_amdgcn_s_waitcnt(WAIT);                                                                         \
        __builtin_amdgcn_s_barrier();                                                                             \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); /* the LDS reads stay below the barrier */         \
        if (q0 < N) {                                                                                             \
            const int t1 = KF < (t0_) + 2 ? KF : (t0_) + 2;                                                       \
            int t = (t0_);                                                                                        \
            for (; t < t1; ++t)                                                                                   \
                att_tile<false>((SK) + (t - (t0_)) * (ATT_BN * 128), (SV) + (t - (t0_)) * (ATT_BN * 128), qf, oacc, \
                                   m_run, l_run, t * ATT_BN, N, scale_log2e, l32, g);                             \
            if (t < KT && t < (t0_) + 2)                                                                          \
                att_tile<true>((SK) + (t - (t0_)) * (ATT_BN * 128), (SV) + (t - (t0_)) * (ATT_BN * 128), qf, oacc, \
                                  m_run, l_run, t * ATT_BN, N, scale_log2e, l32, g);                              \
        }                                                                                                         \
    }
    SM_HALF(s_ka, s_va, 0, 0x0F74)  // vmcnt(4): all but the newest four copies
    SM_HALF(s_kb, s_vb, 2, 0x0F70)
#undef SM_HALF
    __builtin_amdgcn_s_waitcnt(0x0070);  // no copy is in flight, and every read has been answered
    bf16raw* const o_wave = o + (int64_t)b * osb + (int64_t)q0 * osn + (int64_t)h * osh;
    // One or two waves' rows: their stores alone do not pay for the barrier.  us, direct / through LDS, 1 x 1 and 256 x 12 heads: N = 1
    // 3.2 / 3.4, 16.1 / 18.6; 21 3.4 / 3.55, 19.1 / 20.2; 37 3.7 / 4.0, 23.3 / 23.7; 53 4.0 / 4.1, 25.5 / 24.7; 64 3.6 / 3.8, 24.7 / 23.1.
    if (N <= SM_DIRECT) {
        if (q0 < N) att_store_direct(oacc, 1.0f / half_sum(l_run), o_wave, osn, min(N - q0, 32), lane);
        return;
    }
    __builtin_amdgcn_s_barrier();  // K and V are free
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (q0 >= N) return;
    const float l_tot = half_sum(l_run);
    unsigned char* const buf = (wave < 4 ? s_ka : s_va) + (wave & 3) * 4096;
    att_store(oacc, 1.0f / l_tot, buf, o_wave, osn, min(N - q0, 32), lane);
}

// ---------------------------------------------------------------------------
// fp32 path (v_mfma_f32_32x32x2_f32, true fp32 products): workgroup = 32 query rows of one
// (image, head), its four waves split the KEYS (wave w: tiles of 32 keys w, w + 4, ...), K in registers, V in an LDS
// tile of the wave's own, no barrier in the loop; the four partial results are merged through
// LDS in wave order.  Transposed like the bf16 kernels: S^T = K Q^T, and a lane's scores (query l32,
// keys 8 j + 4 g + i in register 4 j + i) feed O^T = V^T P^T as they are: one k step of the instruction
// takes one key from each half-wave.  The first half of the next K tile is requested before the softmax, the copies of the
// next V tile behind the products that read the present one, and the second half of K at the top of its turn: answers come in
// order, so what covers V is the first half of the scores, and the second half waits for V as well.
// The key split is there for small batches: four images of 197 tokens and three heads are 84 blocks
// of 32 rows, which leave two thirds of the CUs empty and would walk seven key tiles one after the other.
// A wave has one or two tiles at N = 197, so most of its time is waiting and merging: what counts is how many
// workgroups share a CU.  V alone takes 32 KB of LDS and half a K tile of registers leaves 128: four (K in LDS as well:
// two).  us, two / four: 64 x 197 x 3 heads 44.1 / 37.3, 64 x 158 x 3 29.8 / 23.4, 20 x 260 x 12 73.8 / 60, 8 x 689 x 12 138 / 122 (97 TFLOP/s of
// the 137 the chip gives fp32 products); with a whole K tile in registers and three workgroups 39.0, 25.0, 62.5, 124.
// ---------------------------------------------------------------------------
constexpr int F32_BN = 32;
constexpr int64_t F32_FAR = (int64_t)1 << 27;  // row stride (elements) at which four rows leave 32-bit byte offsets

// FAR: rows F32_FAR elements apart and more; a tile's rows then pass through registers, each read at its own
// 64-bit address.  Everything behind the copies is the same.
template <bool FAR>
__global__ __launch_bounds__(256, FAR ? 2 : 4) void attention_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, int N, int64_t sb, int64_t sn, int64_t sh, int64_t osb, int64_t osn,
    int64_t osh, float scale_log2e) {
    // V: [32 keys][64 channels] per wave, the two 128-byte halves of a row swapped where (r >> 2) is odd (the half-waves
    // read rows 4 apart)
    __shared__ __attribute__((aligned(1024))) unsigned char s_v[4][F32_BN * 256];
    __shared__ float s_m[4][32], s_l[4][32];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int h = blockIdx.y, b = blockIdx.z;
    const int64_t base = (int64_t)b * sb + (int64_t)h * sh;
    const int q0 = blockIdx.x * 32;
    const int KT = (N + F32_BN - 1) / F32_BN;

    // copy i brings rows 4 i .. 4 i + 3 of a tile through a resource of its own (64-bit base, so that only
    // four rows have to lie within 32-bit offsets); rows past N read as zeros
    const int sn4 = FAR ? 0 : (int)(sn * 4);
    const int v_voff = (lane >> 4) * sn4;
#define F32_COPY_V(kt_)                                                                                           \
    _Pragma("unroll") for (int i = 0; i < 8; ++i) {                                                               \
        const int row_ = (kt_) * F32_BN + 4 * i, rows_ = min(N - row_, 4);                                        \
        const int chunk_ = (lane & 15) ^ ((i & 1) << 3);                                                          \
        if constexpr (FAR) {                                                                                      \
            f32x4 t_ = {0.f, 0.f, 0.f, 0.f};                                                                      \
            if ((lane >> 4) < rows_)                                                                              \
                t_ = *reinterpret_cast<const f32x4*>(v + base + (row_ + (lane >> 4)) * sn + (chunk_ << 2));       \
            *reinterpret_cast<f32x4*>(s_v[wave] + i * 1024 + lane * 16) = t_;                                     \
            continue;                                                                                             \
        }                                                                                                         \
        const __amdgpu_buffer_rsrc_t rs_ = __builtin_amdgcn_make_buffer_rsrc(                                     \
            const_cast<float*>(v + base + (rows_ > 0 ? (int64_t)row_ * sn : 0)), 0,                               \
            rows_ > 0 ? (rows_ - 1) * sn4 + DH * 4 : 0, 0x00020000);                                              \
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_, (att_lds_ptr)(s_v[wave] + i * 1024), 16,                    \
                                                 v_voff + (chunk_ << 4), 0, 0, 0);                                \
    }
// Four of the eight chunks of a K tile, straight into the registers of the matrix instruction's A operand: lane l32 holds channels
// 8 s + 4 g .. of key l32 of the tile (keys past the end: a copy of the last one, masked below)
#define F32_LOAD_K(kf_, kt_, s0_)                                                                                 \
    {                                                                                                             \
        const float* kp_ = k + base + (int64_t)min((kt_) * F32_BN + l32, N - 1) * sn + 4 * g + 8 * (s0_);         \
        _Pragma("unroll") for (int s = 0; s < 4; ++s) kf_[s] = *reinterpret_cast<const f32x4*>(kp_ + 8 * s);      \
    }

    f32x4 qf[8];  // channels 8 s + 4 g .. + 3 of query row q0 + l32
    {
        int qr = q0 + l32;
        qr = qr < N ? qr : N - 1;  // rows past the end are computed on a copy and never stored
        const float* qp = q + base + (int64_t)qr * sn;
#pragma unroll
        for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const f32x4*>(qp + 8 * s + 4 * g);
    }
    f32x4 kf[4];
    F32_LOAD_K(kf, wave, 0)
    F32_COPY_V(wave)
    f32x16 oacc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
    // Keys masked by -inf or a very low value may be all that a wave's first tile holds.  The maximum starts at the
    // lowest value whose multiple by the scale, rounded, is still within 128 of the exact one: such keys weigh 0 (from
    // -inf - -inf or from a lower maximum, whose rounding error alone would overflow the exponential, they would be NaN)
    float m_run = fmaxf(-0x1p32f * __builtin_amdgcn_rcpf(scale_log2e), -FLT_MAX), l_run = 0.f;

    for (int kt = wave; kt < KT; kt += 4) {
        f32x16 sacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[r] = 0.f;
        f32x4 kg[4];
        F32_LOAD_K(kg, kt, 4)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s][e], qf[s][e], sacc, 0, 0, 0);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(kg[s][e], qf[4 + s][e], sacc, 0, 0, 0);
        F32_LOAD_K(kf, kt + 4, 0)
        const int key0 = kt * F32_BN;
        if (key0 + F32_BN > N) {  // keys past the end
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + (r >> 2) * 8 + g * 4 + (r & 3) >= N) sacc[r] = -INFINITY;
        }
        float mx = sacc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sacc[r]);
        mx = half_max(mx);
        const float m_new = fmaxf(m_run, mx);
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2e);
        const float mb = m_new * scale_log2e;
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sacc[r] = __builtin_amdgcn_exp2f(fmaf(sacc[r], scale_log2e, -mb));
            l_run += sacc[r];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");  // V has landed (as it had before the second half of K; the next K may be in flight)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int db = 0; db < 2; ++db) {
                    const float vf = *reinterpret_cast<const float*>(s_v[wave] + (8 * j + 4 * g + i) * 256 + (((db * 32 + l32) * 4) ^ (g << 7)));
                    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf, sacc[4 * j + i], oacc[db], 0, 0, 0);
                }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        F32_COPY_V(kt + 4)
    }
#undef F32_LOAD_K
#undef F32_COPY_V
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // trailing (empty) copies: the tiles get reused

    // ---- merge the four partials
    const float l_tot = half_sum(l_run);
    if (g == 0) {
        s_m[wave][l32] = m_run;
        s_l[wave][l32] = l_tot;
    }
    __syncthreads();
    float m_all = s_m[0][l32];
#pragma unroll
    for (int w = 1; w < 4; ++w) m_all = fmaxf(m_all, s_m[w][l32]);
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) L += s_l[w][l32] * __builtin_amdgcn_exp2f((s_m[w][l32] - m_all) * scale_log2e);
    // 0 for a wave without tiles or with no score above -inf; a row without any such score is NaN, as its softmax is
    const float f = __builtin_amdgcn_exp2f((m_run - m_all) * scale_log2e) / L;
    float* part = reinterpret_cast<float*>(s_v[wave]);  // [32 rows][64 channels], this wave's own tile
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int slot = db * 8 + 2 * j + g;  // 4 channels db*32 + 8j + 4g ..
            const f32x4 val = {oacc[db][4 * j] * f, oacc[db][4 * j + 1] * f, oacc[db][4 * j + 2] * f, oacc[db][4 * j + 3] * f};
            *reinterpret_cast<f32x4*>(part + l32 * 64 + ((slot ^ (l32 & 15)) << 2)) = val;
        }
    __syncthreads();
    const int r = tid >> 3, c8 = tid & 7;  // row of the 32, channels 8 c8 .. 8 c8 + 7
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float* pw = reinterpret_cast<const float*>(s_v[w]) + r * 64;
        const f32x4 lo = *reinterpret_cast<const f32x4*>(pw + (((2 * c8) ^ (r & 15)) << 2));
        const f32x4 hi = *reinterpret_cast<const f32x4*>(pw + (((2 * c8 + 1) ^ (r & 15)) << 2));
#pragma unroll
        for (int e = 0; e < 4; ++e) { acc[e] += lo[e]; acc[4 + e] += hi[e]; }
    }
    if (q0 + r < N) Elem<float>::store8(o + (int64_t)b * osb + (int64_t)(q0 + r) * osn + (int64_t)h * osh + c8 * 8, acc);
}

hipError_t launch_attention(rs_dtype dt, const void* q, const void* k, const void* v, void* o, int B,
                            int H, int N, int64_t sb, int64_t sn, int64_t sh, int64_t osb,
                            int64_t osn, int64_t osh, float scale, hipStream_t s) {
    if (B == 0 || H == 0 || N == 0) return hipSuccess;
    const float scale_log2e = scale * 1.44269504088896340736f;
    if (dt == RS_BF16 && N <= SM_MAXN) {
        // While every workgroup has a CU to itself a head's query rows go to two workgroups of four busy waves, one
        // per SIMD (each copies the whole K and V): 1 image x 6 heads x 197 tokens 8.3 -> 7.0 us, 10 x 12 x 197 8.7
        // -> 7.6; with two on some CUs it costs more than it gives (16 x 12 x 197 9.2 / 9.5, 21 x 12 x 256 11.2 /
        // 13.3).  A row's arithmetic is the same either way.
        const int q_waves = N > 128 && (int64_t)B * H * 2 <= device_cus() ? 4 : 8;
        hipLaunchKernelGGL(attention_bf16_small_kernel, dim3(H, B, q_waves == 4 ? 2 : 1), dim3(512), 0, s, (const bf16raw*)q,
                           (const bf16raw*)k, (const bf16raw*)v, (bf16raw*)o, N, sb, sn, sh, osb, osn, osh,
                           scale_log2e, q_waves);
    } else if (dt == RS_BF16) {
        const int BH = B * H;
        const AttentionPlan plan = attention_plan(BH, N, device_cus());
        const int q_tiles = plan.q_tiles;
        dim3 grid(8 * ((BH + 7) / 8) * q_tiles);
#define ATT_GO(NW_)                                                                                                  \
    hipLaunchKernelGGL((attention_bf16_kernel<NW_>), grid, dim3(NW_ * 64), 0, s, (const bf16raw*)q, (const bf16raw*)k, \
                       (const bf16raw*)v, (bf16raw*)o, N, sb, sn, sh, osb, osn, osh, scale_log2e, H, BH, q_tiles)
        if (plan.rows == ATT_BM) ATT_GO(8);
        else ATT_GO(4);
#undef ATT_GO
        if (plan.tail)
            hipLaunchKernelGGL(attention_bf16_tail_kernel, dim3(BH), dim3(512), 0, s, (const bf16raw*)q,
                               (const bf16raw*)k, (const bf16raw*)v, (bf16raw*)o, N, sb, sn, sh, osb, osn,
                               osh, scale_log2e, H, q_tiles * ATT_BM);
    } else {
        dim3 grid((N + 31) / 32, H, B);
        hipLaunchKernelGGL(sn < F32_FAR ? attention_f32_kernel<false> : attention_f32_kernel<true>, grid, dim3(256), 0, s,
                           (const float*)q, (const float*)k, (const float*)v, (float*)o, N, sb, sn, sh, osb, osn, osh,
                           scale_log2e);
    }
    return hipGetLastError();
}

}  // namespace rs

// ---------------------------------------------------------------------------
// Standard (unfused) attention, the comparison system of Sec. 3.1 / Table 1: the attention map
// A = Softmax(Q K^T * scale) is written to memory, which is what the attention-based importance
// scores of Eqs. (2), (3) need and what the fused kernels above avoid.  Steps: pack the heads
// (q, k as [B H, Np, 64] with zero rows up to Np = N rounded up to 64, v transposed to
// [B H, 64, Np]); S = Q K^T as a batched matrix-core GEMM; softmax over every row in place;
// O = A V as a second batched GEMM; rows back to the caller's layout; column sums of the map.
// ---------------------------------------------------------------------------
namespace rs {

// one workgroup per (image * head, 64-token tile)
__global__ __launch_bounds__(256) void attn_pack_kernel(const bf16raw* __restrict__ q, const bf16raw* __restrict__ k,
                                                        const bf16raw* __restrict__ v, bf16raw* __restrict__ qh,
                                                        bf16raw* __restrict__ kh, bf16raw* __restrict__ vt, int H, int N,
                                                        int Np, int64_t sb, int64_t sn, int64_t sh) {
    __shared__ bf16raw tile[64][72];  // v rows of this tile, padded against bank conflicts
    const int bh = blockIdx.y, b = bh / H, h = bh - b * H;
    const int n0 = blockIdx.x * 64;
    const int64_t base = (int64_t)b * sb + (int64_t)h * sh;
    // 64 rows x 8 chunks of 16 bytes: two chunks per thread
    for (int t = threadIdx.x; t < 512; t += 256) {
        const int r = t >> 3, c = (t & 7) * 8;
        const int n = n0 + r;
        uint4 zq = make_uint4(0u, 0u, 0u, 0u), zk = zq, zv = zq;
        if (n < N) {
            zq = *reinterpret_cast<const uint4*>(q + base + (int64_t)n * sn + c);
            zk = *reinterpret_cast<const uint4*>(k + base + (int64_t)n * sn + c);
            zv = *reinterpret_cast<const uint4*>(v + base + (int64_t)n * sn + c);
        }
        *reinterpret_cast<uint4*>(qh + ((int64_t)bh * Np + n) * 64 + c) = zq;
        *reinterpret_cast<uint4*>(kh + ((int64_t)bh * Np + n) * 64 + c) = zk;
        *reinterpret_cast<uint4*>(&tile[r][c]) = zv;
    }
    __syncthreads();
    // vt[bh][d][n0 + r]: thread (d, r-chunk of 8)
    for (int t = threadIdx.x; t < 512; t += 256) {
        const int d = t >> 3, r0 = (t & 7) * 8;
        union { bf16raw e[8]; uint4 u; } w;
#pragma unroll
        for (int i = 0; i < 8; ++i) w.e[i] = tile[r0 + i][d];
        *reinterpret_cast<uint4*>(vt + ((int64_t)bh * 64 + d) * Np + n0 + r0) = w.u;
    }
}

hipError_t launch_attn_pack(const void* q, const void* k, const void* v, void* qh, void* kh, void* vt, int B, int H,
                            int N, int Np, int64_t sb, int64_t sn, int64_t sh, hipStream_t s) {
    hipLaunchKernelGGL(attn_pack_kernel, dim3(Np / 64, B * H), dim3(256), 0, s, (const bf16raw*)q, (const bf16raw*)k,
                       (const bf16raw*)v, (bf16raw*)qh, (bf16raw*)kh, (bf16raw*)vt, H, N, Np, sb, sn, sh);
    return hipGetLastError();
}

// one wavefront per row of the [rows, Np] score matrices: three passes over the row (maximum, sum,
// normalised write), the columns past N become zero
__global__ __launch_bounds__(256) void attn_softmax_rows_kernel(bf16raw* __restrict__ map, int64_t rows, int N, int Np,
                                                                float scale_log2e) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    bf16raw* p = map + row * Np;
    float mx = -INFINITY;
    for (int c = lane * 8; c < Np; c += 512) {
        float x[8];
        Elem<bf16raw>::load8(p + c, x);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (c + i < N) mx = fmaxf(mx, x[i]);
    }
    mx = lanes_reduce<64>(mx, [](float a, float b) { return fmaxf(a, b); });
    const float mb = mx * scale_log2e;
    float sum = 0.f;
    for (int c = lane * 8; c < Np; c += 512) {
        float x[8];
        Elem<bf16raw>::load8(p + c, x);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (c + i < N) sum += __builtin_amdgcn_exp2f(fmaf(x[i], scale_log2e, -mb));
    }
    sum = wave_sum(sum);
    const float inv = 1.0f / sum;
    for (int c = lane * 8; c < Np; c += 512) {
        float x[8];
        Elem<bf16raw>::load8(p + c, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = c + i < N ? __builtin_amdgcn_exp2f(fmaf(x[i], scale_log2e, -mb)) * inv : 0.f;
        Elem<bf16raw>::store8(p + c, x);
    }
}

hipError_t launch_attn_softmax_rows(void* map, int64_t rows, int N, int Np, float scale_log2e, hipStream_t s) {
    if (rows == 0) return hipSuccess;
    hipLaunchKernelGGL(attn_softmax_rows_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, (bf16raw*)map, rows,
                       N, Np, scale_log2e);
    return hipGetLastError();
}

// partial[bh][j] = sum_i A[bh][i][j]  (thread j walks the rows in order: fixed order, coalesced)
__global__ __launch_bounds__(256) void attn_colsum_kernel(const bf16raw* __restrict__ map, float* __restrict__ partial,
                                                          int N, int Np) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    const int bh = blockIdx.y;
    if (j >= N) return;
    const bf16raw* p = map + (int64_t)bh * N * Np + j;
    float acc = 0.f;
    for (int i = 0; i < N; ++i) acc += bf2f(p[(int64_t)i * Np]);
    partial[(int64_t)bh * N + j] = acc;
}

// Eq. (2): s_cls[b][j] = mean_h A[b,h,cls,j];  Eq. (3): s_mean[b][j] = mean_h (1/N) sum_i A[b,h,i,j]
__global__ __launch_bounds__(256) void attn_scores_kernel(const bf16raw* __restrict__ map, const float* __restrict__ partial,
                                                          float* __restrict__ s_cls, float* __restrict__ s_mean, int H,
                                                          int N, int Np, int cls_index) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    const int b = blockIdx.y;
    if (j >= N) return;
    float c = 0.f, m = 0.f;
    for (int h = 0; h < H; ++h) {
        const int64_t bh = (int64_t)b * H + h;
        c += bf2f(map[(bh * N + cls_index) * Np + j]);
        m += partial[bh * N + j];
    }
    if (s_cls) s_cls[(int64_t)b * N + j] = c / (float)H;
    if (s_mean) s_mean[(int64_t)b * N + j] = m / ((float)H * (float)N);
}

hipError_t launch_attn_map_scores(const void* map, float* partial, float* s_cls, float* s_mean, int B, int H, int N,
                                  int Np, int cls_index, hipStream_t s) {
    if (!s_cls && !s_mean) return hipSuccess;
    if (s_mean)
        hipLaunchKernelGGL(attn_colsum_kernel, dim3((N + 255) / 256, B * H), dim3(256), 0, s, (const bf16raw*)map, partial, N, Np);
    hipLaunchKernelGGL(attn_scores_kernel, dim3((N + 255) / 256, B), dim3(256), 0, s, (const bf16raw*)map, partial,
                       s_cls, s_mean, H, N, Np, cls_index);
    return hipGetLastError();
}

// o[b, n, h, :] = oh[b h][n][:]; 8 lanes per 128-byte row
__global__ __launch_bounds__(256) void attn_unpack_kernel(const bf16raw* __restrict__ oh, bf16raw* __restrict__ o, int H,
                                                          int N, int64_t rows, int64_t osb, int64_t osn, int64_t osh) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t r = t >> 3;  // row index into [B H, N]
    if (r >= rows) return;
    const int c = (int)(t & 7) * 8;
    const int64_t bh = r / N;
    const int n = (int)(r - bh * N);
    const int64_t b = bh / H;
    const int h = (int)(bh - b * H);
    *reinterpret_cast<uint4*>(o + b * osb + (int64_t)n * osn + (int64_t)h * osh + c) =
        *reinterpret_cast<const uint4*>(oh + r * 64 + c);
}

hipError_t launch_attn_unpack(const void* oh, void* o, int B, int H, int N, int64_t osb, int64_t osn, int64_t osh,
                              hipStream_t s) {
    const int64_t rows = (int64_t)B * H * N;
    if (rows == 0) return hipSuccess;
    hipLaunchKernelGGL(attn_unpack_kernel, dim3((unsigned)((rows * 8 + 255) / 256)), dim3(256), 0, s, (const bf16raw*)oh,
                       (bf16raw*)o, H, N, rows, osb, osn, osh);
    return hipGetLastError();
}

}  // namespace rs
