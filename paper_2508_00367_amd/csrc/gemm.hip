// Linear layers of the encoder block (QKV, output projection, fc1, fc2; the O(N C^2)
// term of Sec. 3.1) with the block's elementwise work fused into the epilogue:
// bias, exact GELU, residual add (Eqs. (5),(6)) and the per-row partial sums of the
// representation shift D(MLP(LN(x')), x') (Eq. (4); case (ii) of "Operation choice").
//
// bf16 path: v_mfma_f32_32x32x16_bf16, fp32 accumulation.  The weight matrix is the
// A operand (rows = output features n) and the activations are the B operand
// (columns = token rows m), so that in the accumulator layout a lane owns ONE token
// row and 4 consecutive output features per register quad: row-wise epilogue work
// (residual, shift partial sums) stays inside a lane, and stores are 8-byte vectors.
//
// fp32 path: gemm_f32.hip.
#include <stdlib.h>

#include <atomic>

#include "gemm_choice.hpp"
#include "gemm_tile.hpp"

namespace rs {

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM:  out[m, n] = epi( sum_k a[m, k] * wt[n, k] )
//   a  : [M, K] bf16 (token rows),  K % 64 == 0;  wt : [N, K] bf16, in rows (WF false: rs_linear_fwd) or in
//   fragment order (WF true: the weights a block has packed; LDS then holds whole fragments, no swizzle).
// The compiler knows which copies a fragment read need not wait for only through few steps of address
// arithmetic from the stage's array: a lane's offset is one number (wlane), added to the array at once.
// Workgroup tile BM x BN, K slices of BK, WGM x WGN waves, a ring of LDS stages.
// LDS rows are 64 bf16 = 8 slots of 16 B; chunk c of row r sits in slot c ^ ((r ^ (r >> 3)) & 7).
// The LDS has 64 banks of 4 bytes and serves a 16-byte-per-lane read 16 lanes at a time, so the
// 16 consecutive rows those lanes read for one MFMA operand must fall into 16 different
// 16-byte bank groups: the row parity picks the 128-byte half, the XOR makes the slots of rows
// r and r + 8 differ (measured: zero SQ_LDS_BANK_CONFLICT, against every second cycle with
// the plain c ^ (r & 7)).
// ---------------------------------------------------------------------------

// element strides between the problems of a batched launch (0 = one problem)
struct GemmBatch {
    int64_t a, w, out;
};

// WGM x WGN waves; workgroup tile BM x BN, wave tile BM/WGM x BN/WGN, K slice BK (32 or 64).
// A ring of LDS stages of (BM + BN) rows x 2*BK bytes (NSTAGE = 2), or three stages for the
// activation rows and two for the weight rows (NSTAGE = 3, long K): K slices stream from global
// memory directly into LDS (buffer_load ... lds, no register staging), one slice ahead of the
// one the matrix cores work on (activation rows with NSTAGE = 3: two).  Loads return in order,
// so "slice t has landed" is s_waitcnt vmcnt(<loads issued after it>); one workgroup barrier per
// slice.  The slice count is padded to a multiple of the unrolled trip (2 or 6 slices) with copies
// aimed past the end of the buffer resource (they deliver zeros), which keeps the loop free of
// tail branches.  Operand fragments are double buffered in registers and each LDS read is
// interleaved with its share of the previous K step's MFMAs (sched_group_barrier).  One
// workgroup per CU; the register budget is that of NW / 4 waves per SIMD.
template <int BM, int BN, int BK, int NSTAGE, int WGM, int WGN, int EPI, int DIST, bool WF>
__global__ __launch_bounds__(WGM* WGN * 64, WGM* WGN / 4) void gemm_bf16_kernel(
    const bf16raw* __restrict__ a, const bf16raw* __restrict__ wt, const bf16raw* __restrict__ bias,
    const bf16raw* __restrict__ res, bf16raw* __restrict__ out, float* __restrict__ partials,
    const bf16raw* __restrict__ ref, int post, GemmLnFold ln, int M, int N, int K, int ld, int ldo, int tiles_m,
    int tiles_n, int slots, int64_t ldp, int gm) {
    constexpr int NW = WGM * WGN;               // waves: WGM along tokens x WGN along features
    constexpr int WM = BM / WGM, WN = BN / WGN; // wave tile
    constexpr int TM = WM / 32, TN = WN / 32;   // MFMA tiles per wave
    constexpr int RB = BK * 2;                  // bytes per LDS row
    constexpr int SPR = BK / 8;                 // 16-byte slots per row (4 or 8)
    constexpr int RPI = 64 / SPR;               // rows one wave copy (1 KiB) covers
    constexpr int A_LOADS = BM / RPI / NW, W_LOADS = BN / RPI / NW;  // wave copies per slice and wave
    constexpr int LPW = A_LOADS + W_LOADS;
    constexpr int KK = BK / 16;                 // MFMA K steps per slice
    constexpr int STAGE = (BM + BN) * RB;
    static_assert(WM % 64 == 0 && WN % 64 == 0, "wave tiles must be multiples of 64 rows");
    static_assert(NW == 4 || NW == 8, "4 or 8 waves");
    static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile rows must split evenly over the wave copies");
    static_assert(BK == 32 || BK == 64, "K slice of 32 or 64");
    static_assert(NSTAGE == 2 || NSTAGE == 3, "two stages, or three for the activation rows (deeper rings of narrower slices measured no better)");

    // LDS, NSTAGE = 2: two stages of (BM + BN) rows.  Epilogue staging (32 fp32 rows of the wave tile
    // + the wave's row statistics per wave) lives in the array of stage 1, which is made large
    // enough for all waves: stage 0 receives the next tile's first K slice meanwhile, and being a
    // different array the compiler knows that the epilogue's LDS traffic need not wait for those
    // copies.
    // NSTAGE = 3 (long K): the activation rows of a slice and its weight rows live in arrays of
    // their own, THREE for the activations (requested two slices ahead: they are the rows that
    // come from HBM, and under load a CU's 64 KB request takes longer than one slice of matrix
    // work) and two for the weights (shared by every row panel, they come from the L2): all 160
    // KB.  Epilogue staging in activation stages 1, 2 and weight stage 1.
    constexpr int EPW = (32 * (WN * 4 + 16) + WM * 8 + 255) / 256 * 256;  // bytes per wave
    constexpr int SA = BM * RB, SW = BN * RB;
    constexpr bool DEEP = NSTAGE == 3;
    static_assert(!DEEP || (NW == 8 && 3 * EPW <= SA && 2 * EPW <= SW), "staging of waves 0-2, 3-5, 6-7 in three stage arrays");
    __shared__ __attribute__((aligned(1024))) unsigned char stage0[DEEP ? 16 : STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char stage1[DEEP ? 16 : (STAGE > NW * EPW ? STAGE : NW * EPW)];
    __shared__ __attribute__((aligned(1024))) unsigned char sa0[DEEP ? SA : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char sa1[DEEP ? SA : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char sa2[DEEP ? SA : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char sw0[DEEP ? SW : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char sw1[DEEP ? SW : 16];

    // Tile order.  Consecutive workgroup ids go round-robin to the 8 XCDs, each with its own
    // 4 MB L2, so XCD x takes a contiguous range of the tile sequence.  The sequence walks the tile
    // grid in groups of `gm` row panels, n-major inside a group (m fastest): the ~32 tiles an XCD
    // runs at a time then share gm activation panels, which stay in its L2 while the weight
    // panels stream past, instead of re-reading the whole weight matrix for every row panel.
    //
    // Persistent workgroups: the grid is one workgroup per CU; workgroup (x, j) of XCD x walks
    // positions j, j + per_xcd, ... of that XCD's range, so the tiles an XCD runs at a time are the
    // same as with one workgroup per tile, but the first K slice of the next tile is fetched while
    // the epilogue of the current one runs.
    const int nblk = tiles_m * tiles_n;
    const int xcd = blockIdx.x & 7, per_xcd = gridDim.x >> 3;
    const int xq = nblk >> 3, xr = nblk & 7;  // XCD x owns xq (+1 if x < xr) tiles
    const int x_cnt = xq + (xcd < xr ? 1 : 0), x_start = xcd * xq + (xcd < xr ? xcd : xr);
    int seq = blockIdx.x >> 3;
    if (seq >= x_cnt) return;  // whole workgroup, before any barrier
#define RS_GEMM_DECODE(seq_, m0_, n0_)                                                                    \
    {                                                                                                     \
        const int bid_ = x_start + (seq_);                                                                \
        const int per_group_ = gm * tiles_n;                                                              \
        const int grp_ = bid_ / per_group_, rem_ = bid_ - grp_ * per_group_;                              \
        const int first_m_ = grp_ * gm;                                                                   \
        const int gsz_ = min(tiles_m - first_m_, gm);                                                     \
        const int tn_ = rem_ / gsz_;                                                                      \
        (n0_) = tn_ * BN;                                                                                 \
        (m0_) = (first_m_ + rem_ - tn_ * gsz_) * BM;                                                      \
    }
    int m0, n0;
    RS_GEMM_DECODE(seq, m0, n0)

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: LDS copy targets go to M0
    const int wm = wave % WGM, wn = wave / WGM;
    const int l32 = lane & 31, g = lane >> 5;

    // LDS layout.  Chunk c (16 bytes = 8 k values) of row r sits in slot c ^ f(r).  gfx950's LDS has
    // 64 banks of 4 bytes and serves a 16-byte-per-lane read 16 lanes at a time, so the 16
    // consecutive rows those lanes read for one MFMA operand must fall into 16 different 16-byte
    // bank groups of a 256-byte line:
    //   128-byte rows (BK 64): f(r) = (r & 7) ^ ((r >> 3) & 1)   (row parity picks the half line, the
    //                          XOR makes rows r and r + 8 differ; the plain r & 7 conflicts every
    //                          second cycle.  f has period 16 in r, so one set of lane offsets
    //                          serves every 32-row MFMA tile of the wave)
    //    64-byte rows (BK 32): f(r) = (r >> 2) & 3         (r & 3 picks the quarter line)
    // global -> LDS: wave copy i of wave w fills rows (NW*i + w)*RPI .. +RPI-1 (lane l: row l / SPR,
    // slot l % SPR), so the lane fetches chunk (l % SPR) ^ f(row).
    __amdgpu_buffer_rsrc_t rs_a = make_rsrc(a + (int64_t)m0 * ld, (int64_t)min(M - m0, BM) * ld * 2);
    const int ldw = WF ? K : ld, wlane = wn * TN * KK * 1024 + lane * 16, wvoff = frag_off(wave / KK, wave % KK, K) + lane * 16;
    __amdgpu_buffer_rsrc_t rs_w = make_rsrc(wt + (int64_t)n0 * ldw, (int64_t)min(N - n0, BN) * ldw * 2);
    const int ld_r = lane / SPR, ld_p = lane % SPR;
    // lane byte offset inside a wave copy (NW is even, so row >> 3 = NW*i + w has the parity of w)
    const int voff = SPR == 8 ? ((wave * RPI + ld_r) * ld + ((ld_p ^ ld_r ^ (wave & 1)) << 3)) * 2
                              : ((wave * RPI + ld_r) * ld + ((ld_p ^ ((ld_r >> 2) & 3)) << 3)) * 2;
    const int pass_bytes = NW * RPI * ld * 2;

    const int S = K / BK;                                   // real slices
    constexpr int PERIOD = DEEP ? 6 : 2;                    // slices per trip of the unrolled ring
    const int S_pad = (S + PERIOD - 1) / PERIOD * PERIOD;   // loop trip count (zero slices at the end)
    const int a_row0 = wm * WM + l32, w_row0 = wn * WN + l32;
    // slot XOR of operand row 32*t + l32 (the same for every MFMA tile t of the wave tile)
    const int sw = SPR == 8 ? ((l32 & 7) ^ ((l32 >> 3) & 1)) : ((l32 >> 2) & 3);

// copies of K slice t_ into stage_; slices past the end are aimed beyond the resource (which covers
// this tile's rows only, so the aim is past its end whatever the size of the whole matrix)
#define RS_GEMM_DMA_A(sa_, t_)                                                                            \
    {                                                                                                     \
        const bool real_ = (t_) < S;                                                                      \
        const int kb_ = (t_) * RB;                                                                        \
        _Pragma("unroll") for (int i = 0; i < A_LOADS; ++i)                                               \
            dma16(rs_a, (sa_) + (i * NW + wave) * 1024, voff, real_ ? i * pass_bytes + kb_ : kPastEnd);   \
    }
#define RS_GEMM_DMA_W(sw_, t_)                                                                            \
    {                                                                                                     \
        const bool real_ = (t_) < S;                                                                      \
        const int kb_ = (t_) * RB;                                                                        \
        _Pragma("unroll") for (int i = 0; i < W_LOADS; ++i) {                                             \
            const int f_ = i * NW + wave;                                                                 \
            if constexpr (WF) dma16(rs_w, (sw_) + f_ * 1024, wvoff, real_ ? frag_off(i * NW / KK, i * NW % KK, K) + (t_) * (KK * 1024) : kPastEnd); \
            else dma16(rs_w, (sw_) + f_ * 1024, voff, real_ ? i * pass_bytes + kb_ : kPastEnd);           \
        }                                                                                                 \
    }
#define RS_GEMM_DMA(stage_, t_)                                                                           \
    {                                                                                                     \
        RS_GEMM_DMA_A(stage_, t_)                                                                         \
        RS_GEMM_DMA_W((stage_) + BM * RB, t_)                                                             \
    }
#define RS_GEMM_LOAD_FRAGS2(f_, sa_, sw_, kk_)                                                            \
    {                                                                                                     \
        const int c_ = ((((kk_) * 2 + g) ^ sw) << 4);                                                     \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                    \
            (f_).w[i] = *reinterpret_cast<const bf16x8*>(                                                 \
                (sw_) + (WF ? wlane + (i * KK + (kk_)) * 1024 : (w_row0 + i * 32) * RB + c_));            \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                    \
            (f_).a[j] = *reinterpret_cast<const bf16x8*>((sa_) + (a_row0 + j * 32) * RB + c_);            \
    }
#define RS_GEMM_LOAD_FRAGS(f_, stage_, kk_) RS_GEMM_LOAD_FRAGS2(f_, stage_, (stage_) + BM * RB, kk_)
#define RS_GEMM_MFMA(f_)                                                                                  \
    {                                                                                                     \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                    \
            _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                \
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16((f_).w[i], (f_).a[j], acc[i][j], 0, 0, 0); \
    }
// Scheduling recipe for one K step (one scheduling region): every LDS fragment read of the
// next step is followed by its share of global->LDS copies (vm_) and of this step's MFMAs.
#define RS_GEMM_INTERLEAVE(vm_)                                                                           \
    {                                                                                                     \
        _Pragma("unroll") for (int s_ = 0; s_ < TN + TM; ++s_) {                                          \
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                            \
            if (vm_) __builtin_amdgcn_sched_group_barrier(0x020, (LPW + TN + TM - 1) / (TN + TM), 0);     \
            __builtin_amdgcn_sched_group_barrier(0x008, (TN * TM) / (TN + TM), 0);                        \
        }                                                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                                \
    }
// One K slice from cur_ (its first fragments are already in f0).  Three of the four K steps run
// with the LDS reads of the following step between their MFMAs; then the wave waits for slice
// t+1 (in nxt_) to land, meets the others at the slice's one barrier -- after it every wave has
// finished reading cur_, so the copies of slice t+2 may overwrite it -- and the last K step's
// MFMAs cover those copies and the first fragment reads of slice t+1: the matrix cores have
// work on both sides of the barrier.
#define RS_GEMM_SLICE(cur_, nxt_, t_)                                                                     \
    {                                                                                                     \
        RS_GEMM_LOAD_FRAGS(f1, cur_, 1)                                                                   \
        RS_GEMM_MFMA(f0)                                                                                  \
        RS_GEMM_INTERLEAVE(0)                                                                             \
        RS_GEMM_LOAD_FRAGS(f0, cur_, 2)                                                                   \
        RS_GEMM_MFMA(f1)                                                                                  \
        RS_GEMM_INTERLEAVE(0)                                                                             \
        RS_GEMM_LOAD_FRAGS(f1, cur_, 3)                                                                   \
        RS_GEMM_MFMA(f0)                                                                                  \
        RS_GEMM_INTERLEAVE(0)                                                                             \
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                                                         \
        __syncthreads();                                                                                  \
        RS_GEMM_DMA(cur_, (t_) + 2)                                                                       \
        RS_GEMM_LOAD_FRAGS(f0, nxt_, 0)                                                                   \
        RS_GEMM_MFMA(f1)                                                                                  \
        RS_GEMM_INTERLEAVE(1)                                                                             \
    }

// The same slice with three activation stages (sa_ / sw_: this slice, san_ / swn_: the next): the
// wave waits for slice t+1 only -- the activation rows of slice t+2, requested last, may still be
// on their way: loads complete in order, and no global store is in flight inside the K loop --
// and after the barrier requests the weights of slice t+2, then the activation rows of slice t+3.
#define RS_GEMM_SLICE3(sa_, sw_, san_, swn_, t_)                                                          \
    {                                                                                                     \
        RS_GEMM_LOAD_FRAGS2(f1, sa_, sw_, 1)                                                              \
        RS_GEMM_MFMA(f0)                                                                                  \
        RS_GEMM_INTERLEAVE(0)                                                                             \
        RS_GEMM_LOAD_FRAGS2(f0, sa_, sw_, 2)                                                              \
        RS_GEMM_MFMA(f1)                                                                                  \
        RS_GEMM_INTERLEAVE(0)                                                                             \
        RS_GEMM_LOAD_FRAGS2(f1, sa_, sw_, 3)                                                              \
        RS_GEMM_MFMA(f0)                                                                                  \
        RS_GEMM_INTERLEAVE(0)                                                                             \
        __builtin_amdgcn_s_waitcnt(((A_LOADS) & 15) | (((A_LOADS) >> 4) << 14) | 0x0070);                 \
        __builtin_amdgcn_s_barrier();                                                                     \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); /* LDS reads stay below the barrier */     \
        __builtin_amdgcn_sched_barrier(0);                                                                \
        RS_GEMM_DMA_W(sw_, (t_) + 2)                                                                      \
        RS_GEMM_DMA_A(sa_, (t_) + 3)                                                                      \
        RS_GEMM_LOAD_FRAGS2(f0, san_, swn_, 0)                                                            \
        RS_GEMM_MFMA(f1)                                                                                  \
        RS_GEMM_INTERLEAVE(1)                                                                             \
    }

    static_assert(KK == 4, "the slice schedules are written for 64-wide slices");
    static_assert(A_LOADS <= 15, "copies in flight across a barrier must fit the counter");
    // first K slice of the first tile
    if constexpr (DEEP) {
        RS_GEMM_DMA_A(sa0, 0)
        RS_GEMM_DMA_W(sw0, 0)
    } else {
        RS_GEMM_DMA(stage0, 0)
    }

    for (;;) {  // one tile per iteration
    // LayerNorm-folded epilogues: fetch the (mean, rstd) of this wave's WM rows now (lane l: rows
    // l, l + 64, ...), so that the loads are long done when the epilogue wants them
    constexpr bool LN_EPI = EPI == EPI_LN_BIAS || EPI == EPI_LN_BIAS_GELU;
    float2 row_st[LN_EPI ? WM / 64 : 1];
    if (LN_EPI) {
#pragma unroll
        for (int h = 0; h < WM / 64; ++h) {
            const int m = m0 + wm * WM + h * 64 + lane;
            row_st[h] = m < M ? reinterpret_cast<const float2*>(ln.stats)[m] : make_float2(0.f, 0.f);
        }
    }

    // Likewise the per-column epilogue vectors of the lane's 8 output features (on the way out a
    // row of the wave tile is covered by WN / 8 lanes, 8 consecutive features each).
    const int ep_oc = (lane % (WN / 8)) * 8;
    const int ep_n = n0 + wn * WN + ep_oc;
    const bool ep_n_ok = ep_n < N;  // N % 8 == 0
    uint4 bias_raw = make_uint4(0u, 0u, 0u, 0u);
    float ln_bv[LN_EPI ? 8 : 1], ln_cs[LN_EPI ? 8 : 1];
    if (LN_EPI) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { ln_bv[e] = 0.f; ln_cs[e] = 0.f; }
        if (ep_n_ok) {
            Elem<float>::load8(ln.bias + ep_n, reinterpret_cast<float(&)[8]>(ln_bv));
            Elem<float>::load8(ln.colsum + ep_n, reinterpret_cast<float(&)[8]>(ln_cs));
        }
    } else if (bias && ep_n_ok) {
        bias_raw = *reinterpret_cast<const uint4*>(bias + ep_n);
    }

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // slice 0 has been requested (before the loop, or under the previous tile's epilogue); when it
    // has landed and every wave is past that epilogue, slice 1 goes on its way and the first
    // fragments into registers
    Frags<TN, TM> f0, f1;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    if constexpr (DEEP) {
        // slices 1 and 2 go on their way, the activation rows of slice 2 last (they may stay in
        // flight across the first barrier).  Three activation stages and two weight stages: six
        // slices per trip, no way out in between (an exit inside the trip would make the
        // compiler keep copies of the accumulators for each way out)
        RS_GEMM_DMA_W(sw1, 1)
        RS_GEMM_DMA_A(sa1, 1)
        RS_GEMM_DMA_A(sa2, 2)
        RS_GEMM_LOAD_FRAGS2(f0, sa0, sw0, 0)
        __builtin_amdgcn_sched_barrier(0);
        for (int t = 0; t < S_pad; t += 6) {
            RS_GEMM_SLICE3(sa0, sw0, sa1, sw1, t)
            RS_GEMM_SLICE3(sa1, sw1, sa2, sw0, t + 1)
            RS_GEMM_SLICE3(sa2, sw0, sa0, sw1, t + 2)
            RS_GEMM_SLICE3(sa0, sw1, sa1, sw0, t + 3)
            RS_GEMM_SLICE3(sa1, sw0, sa2, sw1, t + 4)
            RS_GEMM_SLICE3(sa2, sw1, sa0, sw0, t + 5)
        }
    } else {
        RS_GEMM_DMA(stage1, 1)
        RS_GEMM_LOAD_FRAGS(f0, stage0, 0)
        __builtin_amdgcn_sched_barrier(0);
        for (int t = 0; t < S_pad; t += 2) {
            RS_GEMM_SLICE(stage0, stage1, t)
            RS_GEMM_SLICE(stage1, stage0, t + 1)
        }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // the trailing (empty) copies too: the stages get reused
    __syncthreads();  // every wave is done with the K-loop stages


    // next tile: its first K slice streams into stage0 while the epilogue runs (past the last tile
    // the copies are aimed outside the resource and deliver zeros nobody reads).  The copies are
    // issued inside the epilogue, right after its first residual loads: loads return in order,
    // and those must not queue up behind 64 KB of copies.
    const int m0_cur = m0, n0_cur = n0;
    seq += per_xcd;
    const bool more = seq < x_cnt;
    if (more) {
        RS_GEMM_DECODE(seq, m0, n0)
        rs_a = make_rsrc(a + (int64_t)m0 * ld, (int64_t)min(M - m0, BM) * ld * 2);
        rs_w = make_rsrc(wt + (int64_t)n0 * ldw, (int64_t)min(N - n0, BN) * ldw * 2);
    }

    // ---- epilogue, staged through LDS so that global traffic is row-contiguous.
    // Accumulator layout: lane (l32, g) owns token row l32 of each 32-row group; register
    // 4*q + e of tile (i, j) is feature 32*i + 8*q + 4*g + e.  Per 32-row group j the wave writes
    // its 32 x WN fp32 block into a private LDS region (row pitch WN*4 + 16 bytes: conflict
    // free), then re-reads it with 16 lanes per row, 8 consecutive features per lane; bias,
    // GELU, residual, the shift partial sums and the bf16 rounding happen on that layout, and
    // every global load/store instruction covers whole 16 * WN / 8-byte row segments.
    {
        constexpr int PITCH = WN * 4 + 16;         // bytes per staged row
        constexpr int LPR = WN / 8;                // lanes per row on the way out (16 for WN = 128)
        constexpr int RPS = 64 / LPR;              // rows per step
        static_assert(32 * PITCH + WM * 8 <= EPW, "epilogue staging does not fit");
        unsigned char* ep = !DEEP ? stage1 + wave * EPW
                            : wave < 3 ? sa1 + wave * EPW : wave < 6 ? sa2 + (wave - 3) * EPW : sw1 + (wave - 6) * EPW;
        float2* ep_st = reinterpret_cast<float2*>(ep + 32 * PITCH);  // the wave's row statistics
        if (LN_EPI) {
#pragma unroll
            for (int h = 0; h < WM / 64; ++h) ep_st[h * 64 + lane] = row_st[h];
        }
        const int oc = ep_oc;                      // this lane's first feature inside the wave tile
        const int orow = lane / LPR;
        const int n = ep_n;
        const bool n_ok = ep_n_ok;
        constexpr bool LN = LN_EPI;
        float bv[8], cs[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            bv[e] = LN ? ln_bv[LN ? e : 0] : 0.f;
            cs[e] = LN ? ln_cs[LN ? e : 0] : 0.f;
        }
        if (!LN) {
            const uint32_t w4[4] = {bias_raw.x, bias_raw.y, bias_raw.z, bias_raw.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bv[2 * e] = __uint_as_float(w4[e] << 16);
                bv[2 * e + 1] = __uint_as_float(w4[e] & 0xffff0000u);
            }
        }
        // The residual rows of a 32-row group are requested one group ahead (those of group 0 before
        // the loop): a group's staging round trip through LDS is far shorter than a trip to memory.
        constexpr bool RES = EPI == EPI_BIAS_RES || EPI == EPI_BIAS_RES_SHIFT;
        uint4 res_all[RES ? TM : 1][RES ? 32 / RPS : 1];
#define RS_GEMM_LOAD_RES(j_)                                                                              \
    if (RES) {                                                                                            \
        _Pragma("unroll") for (int st = 0; st < 32 / RPS; ++st) {                                         \
            const int m = m0_cur + wm * WM + (j_) * 32 + st * RPS + orow;                                 \
            res_all[RES ? (j_) : 0][st] = (m < M && n_ok) ? *reinterpret_cast<const uint4*>(res + (int64_t)m * N + n) \
                                                           : make_uint4(0u, 0u, 0u, 0u);                  \
        }                                                                                                 \
    }
        // the wave tile's rows inside M (a wave whose features lie past N stores nothing)
        const int m_w = m0_cur + wm * WM, n_w = n0_cur + wn * WN;
        const __amdgpu_buffer_rsrc_t rs_out = make_rsrc(m_w < M && n_w < N ? out + (int64_t)m_w * ldo + n_w : out,
                                                        m_w < M && n_w < N ? ((int64_t)(min(M - m_w, WM) - 1) * ldo + WN) * 2 : 0);
        RS_GEMM_LOAD_RES(0)
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            if (j + 1 < TM) RS_GEMM_LOAD_RES(j + 1)
            const uint4 (&res_raw)[RES ? 32 / RPS : 1] = res_all[RES ? j : 0];
            if (j == 0) {
                if constexpr (DEEP) {
                    RS_GEMM_DMA_A(sa0, more ? 0 : S)
                    RS_GEMM_DMA_W(sw0, more ? 0 : S)
                } else {
                    RS_GEMM_DMA(stage0, more ? 0 : S)
                }
            }
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                    *reinterpret_cast<f32x4*>(ep + l32 * PITCH + (i * 32 + q * 8 + g * 4) * 4) = v;
                }
#pragma unroll
            for (int st = 0; st < 32 / RPS; ++st) {
                const int r = st * RPS + orow;
                const int m = m0_cur + wm * WM + j * 32 + r;
                const bool ok = m < M && n_ok;
                float v[8];
                {
                    const f32x4 lo = *reinterpret_cast<const f32x4*>(ep + r * PITCH + oc * 4);
                    const f32x4 hi = *reinterpret_cast<const f32x4*>(ep + r * PITCH + oc * 4 + 16);
                    if (LN) {
                        const float2 st = ep_st[j * 32 + r];
                        const float nm = -st.x;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            v[e] = fmaf(st.y, fmaf(nm, cs[e], lo[e]), bv[e]);
                            v[4 + e] = fmaf(st.y, fmaf(nm, cs[4 + e], hi[e]), bv[4 + e]);
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) { v[e] = lo[e] + bv[e]; v[4 + e] = hi[e] + bv[4 + e]; }
                    }
                }
                if (EPI == EPI_BIAS_GELU || EPI == EPI_LN_BIAS_GELU) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = gelu_sp(v[e]);
                }
                float p0 = 0.f, p1 = 0.f, p2 = 0.f;
                if (EPI == EPI_BIAS_RES || EPI == EPI_BIAS_RES_SHIFT) {
                    float rr[8];
                    {
                        const uint4 q4 = res_raw[RES ? st : 0];
                        const uint32_t w4[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            rr[2 * e] = __uint_as_float(w4[e] << 16);
                            rr[2 * e + 1] = __uint_as_float(w4[e] & 0xffff0000u);
                        }
                    }
                    if (EPI == EPI_BIAS_RES_SHIFT && ok) {
                        // D(f_out, f_in): f_out is the branch output, or (post) the residual stream
                        // after the add; f_in is the residual operand, or `ref` when one is given
                        float fi[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) fi[e] = rr[e];
                        if (ref) Elem<bf16raw>::load8(ref + (int64_t)m * N + n, fi);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float fo = post ? v[e] + rr[e] : v[e];
                            shift_term<DIST>(fo, fi[e], p0, p1, p2);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] += rr[e];
                }
                store16_wt(rs_out, ok ? ((j * 32 + r) * ldo + oc) * 2 : kPastEnd,
                           make_uint4(pack2bf(v[0], v[1]), pack2bf(v[2], v[3]), pack2bf(v[4], v[5]), pack2bf(v[6], v[7])));
                if (EPI == EPI_BIAS_RES_SHIFT) {
                    // sum over the LPR lanes that share the row (fixed butterfly order)
                    p0 = lanes_sum<LPR>(p0);
                    if (DIST == RS_DIST_COS) { p1 = lanes_sum<LPR>(p1); p2 = lanes_sum<LPR>(p2); }
                    const int slot = (n0_cur + wn * WN) / WN;
                    if ((lane % LPR) == 0 && m < M && slot < slots) {
                        float* dst = partials + slot * ldp + m;
                        dst[0] = p0;
                        if (DIST == RS_DIST_COS) { dst[slots * ldp] = p1; dst[2 * slots * ldp] = p2; }
                    }
                }
            }
        }
    }
        if (!more) break;
    }  // tiles
#undef RS_GEMM_DMA
#undef RS_GEMM_DMA_A
#undef RS_GEMM_DMA_W
#undef RS_GEMM_LOAD_RES
#undef RS_GEMM_LOAD_FRAGS2
#undef RS_GEMM_SLICE3
#undef RS_GEMM_DECODE
#undef RS_GEMM_LOAD_FRAGS
#undef RS_GEMM_MFMA
#undef RS_GEMM_INTERLEAVE
#undef RS_GEMM_SLICE
}

// ---------------------------------------------------------------------------
// Ring kernel: workgroup tile BM x BN (BM token rows, BN features), four waves (WGM x WGN, wave
// tile BM / WGM x 64), K slices of 32 in a ring of three LDS stages, one tile per workgroup and TWO
// workgroups per compute unit (at most 72 KB of LDS and 256 registers each).  The two run out of
// step: while one is in its epilogue, or waits at its per-slice barrier for a late copy, the
// other's K loop keeps the matrix cores busy, and the hardware hands a finished workgroup's slot
// to the next tile, so the tail of a launch is balanced at half-tile granularity.  Copies run two
// slices ahead of the matrix work.
// Slice schedule (one barrier per slice, matrix work on both sides of it): the second K step's
// fragments are read under the first step's MFMAs; then the wave waits for the next slice's
// copies, meets the barrier (now every wave has read this slice: its stage is free), requests the
// slice three ahead into the freed stage and reads the next slice's first fragments under the
// second step's MFMAs.
// ---------------------------------------------------------------------------
template <int BM, int BN, int WGM, int WGN, int EPI, int DIST, bool WF>
__global__ __launch_bounds__(256, 2) void gemm_bf16_ring_kernel(
    const bf16raw* __restrict__ a, const bf16raw* __restrict__ wt, const bf16raw* __restrict__ bias,
    const bf16raw* __restrict__ res, bf16raw* __restrict__ out, float* __restrict__ partials,
    const bf16raw* __restrict__ ref, int post, GemmLnFold ln, int M, int N, int K, int ld, int ldo, int tiles_m,
    int tiles_n, int slots, int64_t ldp, int gm, GemmBatch batch) {
    constexpr int NW = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int BK = 32, RB = BK * 2, RPI = 16;   // 64-byte LDS rows, 16 rows per wave copy
    // batched use (blockIdx.y = problem): the same shape at other addresses, plain epilogues only
    a += (int64_t)blockIdx.y * batch.a;
    wt += (int64_t)blockIdx.y * batch.w;
    out += (int64_t)blockIdx.y * batch.out;
    constexpr int A_LOADS = BM / RPI / NW, W_LOADS = BN / RPI / NW, LPW = A_LOADS + W_LOADS;
    constexpr int STAGE = (BM + BN) * RB;
    static_assert(NW == 4 && WN == 64 && TN == 2, "four waves, wave tiles 64 features wide");
    static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile rows must split evenly over the wave copies");
    static_assert(3 * (STAGE / 4096) >= NW * TM, "the three stages must hold TM 4 KB epilogue regions per wave");
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGE];

    // tile of this workgroup: ids go round-robin to the 8 XCDs, XCD x takes a contiguous range of a
    // sequence that walks the grid in groups of gm row panels, m fastest (see gemm_bf16_kernel)
    const int nblk = tiles_m * tiles_n;
    const int xcd = blockIdx.x & 7;
    const int xq = nblk >> 3, xr = nblk & 7;
    const int x_cnt = xq + (xcd < xr ? 1 : 0), x_start = xcd * xq + (xcd < xr ? xcd : xr);
    const int seq = blockIdx.x >> 3;
    if (seq >= x_cnt) return;  // whole workgroup, before any barrier
    int m0, n0;
    {
        const int bid = x_start + seq;
        const int per_group = gm * tiles_n;
        const int grp = bid / per_group, rem = bid - grp * per_group;
        const int first_m = grp * gm;
        const int gsz = min(tiles_m - first_m, gm);
        const int tn = rem / gsz;
        n0 = tn * BN;
        m0 = (first_m + rem - tn * gsz) * BM;
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;
    const int l32 = lane & 31, g = lane >> 5;

    // global -> LDS: wave copy i of wave w fills rows (NW i + w) 16 .. + 15 (lane l: row l / 4, slot
    // l % 4 holds chunk (l % 4) ^ f(row), f(r) = (r >> 2) & 3: the 16 rows an operand read touches
    // fall into 16 different 16-byte bank groups)
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(a + (int64_t)m0 * ld, (int64_t)min(M - m0, BM) * ld * 2);
    const int ldw = WF ? K : ld, wlane = BM * RB + wn * TN * 2048 + lane * 16, wvoff = frag_off(wave / 2, wave % 2, K) + lane * 16;
    const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(wt + (int64_t)n0 * ldw, (int64_t)min(N - n0, BN) * ldw * 2);
    const int ld_r = lane >> 2, ld_p = lane & 3;
    const int voff = ((wave * RPI + ld_r) * ld + ((ld_p ^ ((ld_r >> 2) & 3)) << 3)) * 2;
    const int pass_bytes = NW * RPI * ld * 2;
    const int S = K / BK;
    const int S_pad = (S + 2) / 3 * 3;
    const int a_row0 = wm * WM + l32, w_row0 = wn * WN + l32;
    const int sw = (l32 >> 2) & 3;

#define RS_RING_DMA(stage_, t_)                                                                           \
    {                                                                                                     \
        const bool real_ = (t_) < S;                                                                      \
        const int kb_ = (t_) * RB;                                                                        \
        _Pragma("unroll") for (int i = 0; i < A_LOADS; ++i)                                               \
            dma16(rs_a, (stage_) + (i * NW + wave) * 1024, voff, real_ ? i * pass_bytes + kb_ : kPastEnd); \
        _Pragma("unroll") for (int i = 0; i < W_LOADS; ++i) {                                             \
            const int f_ = i * NW + wave;                                                                 \
            if constexpr (WF) dma16(rs_w, (stage_) + BM * RB + f_ * 1024, wvoff, real_ ? frag_off(i * NW / 2, i * NW % 2, K) + (t_) * 2048 : kPastEnd); \
            else dma16(rs_w, (stage_) + BM * RB + f_ * 1024, voff, real_ ? i * pass_bytes + kb_ : kPastEnd); \
        }                                                                                                 \
    }
#define RS_RING_FRAGS(f_, stage_, kk_)                                                                    \
    {                                                                                                     \
        const int co_ = ((((kk_) * 2 + g) ^ sw) << 4);                                                    \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                    \
            (f_).w[i] = *reinterpret_cast<const bf16x8*>(                                                 \
                (stage_) + (WF ? wlane + (i * 2 + (kk_)) * 1024 : (BM + w_row0 + i * 32) * RB + co_)); \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                    \
            (f_).a[j] = *reinterpret_cast<const bf16x8*>((stage_) + (a_row0 + j * 32) * RB + co_);        \
    }
#define RS_RING_MFMA(f_)                                                                                  \
    {                                                                                                     \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                    \
            _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                \
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16((f_).w[i], (f_).a[j], acc[i][j], 0, 0, 0); \
    }
// every LDS fragment read is followed by its share of copies and of the running step's MFMAs
#define RS_RING_INTERLEAVE(vm_)                                                                           \
    {                                                                                                     \
        _Pragma("unroll") for (int s_ = 0; s_ < TN + TM; ++s_) {                                          \
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                            \
            if (vm_) __builtin_amdgcn_sched_group_barrier(0x020, (LPW + TN + TM - 1) / (TN + TM), 0);     \
            __builtin_amdgcn_sched_group_barrier(0x008, (TN * TM + TN + TM - 1) / (TN + TM), 0);          \
        }                                                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                                \
    }
// vmcnt <= LPW: the copies of the slice after next may be in flight; LDS reads all answered
#define RS_RING_SLICE(cur_, nxt_, t_)                                                                     \
    {                                                                                                     \
        RS_RING_FRAGS(f1, cur_, 1)                                                                        \
        RS_RING_MFMA(f0)                                                                                  \
        RS_RING_INTERLEAVE(0)                                                                             \
        __builtin_amdgcn_s_waitcnt(((LPW) & 15) | (((LPW) >> 4) << 14) | 0x0070);                         \
        __builtin_amdgcn_s_barrier();                                                                     \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); /* LDS reads stay below the barrier */     \
        __builtin_amdgcn_sched_barrier(0);                                                                \
        RS_RING_DMA(cur_, (t_) + 3)                                                                       \
        RS_RING_FRAGS(f0, nxt_, 0)                                                                        \
        RS_RING_MFMA(f1)                                                                                  \
        RS_RING_INTERLEAVE(1)                                                                             \
    }

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    RS_RING_DMA(st0, 0)
    RS_RING_DMA(st1, 1)
    RS_RING_DMA(st2, 2)
    Frags<TN, TM> f0, f1;
    __builtin_amdgcn_s_waitcnt(((2 * LPW) & 15) | (((2 * LPW) >> 4) << 14) | 0x0070);  // slice 0 has landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    __builtin_amdgcn_sched_barrier(0);
    RS_RING_FRAGS(f0, st0, 0)
    for (int t = 0; t < S_pad; t += 3) {
        RS_RING_SLICE(st0, st1, t)
        RS_RING_SLICE(st1, st2, t + 1)
        RS_RING_SLICE(st2, st0, t + 2)
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & 0xC07F);  // trailing (empty) copies and LDS reads: the stages get reused
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    __builtin_amdgcn_sched_barrier(0);
#undef RS_RING_DMA
#undef RS_RING_FRAGS
#undef RS_RING_MFMA
#undef RS_RING_INTERLEAVE
#undef RS_RING_SLICE

    // epilogue regions: TM x 4 KB per wave, numbered through the three stage arrays
    EpiRegions<TM> reg;
    {
        constexpr int PER = STAGE / 4096;  // regions per stage array
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int gi = wave * TM + j;
            reg.r[j] = (gi / PER == 0 ? st0 : gi / PER == 1 ? st1 : st2) + (gi % PER) * 4096;
        }
    }
    const int m_base = m0 + wm * WM, n_base = n0 + wn * WN;
    EpiVecs<TM, EPI> vec;
    if (epi_res(EPI)) epi_request_residual<TM>(reg, res, M, N, m_base, n_base, lane);
    vec.load(bias, ln, M, N, m_base, n_base, lane);
    if (epi_res(EPI)) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // every residual row of the tile has landed
    gemm_epilogue_acc_layout<TM, EPI, DIST>(acc, reg, vec, out, partials, ref, post, M, N, ldo, slots, ldp, m_base, n_base, lane);
}

// ---------------------------------------------------------------------------
// Slim kernel, for grids that leave the chip empty with larger tiles: workgroup tile (32 TM WGM) x (64 WGN),
// wave tile (32 TM) x 64, K slices of 64 in a ring of NST stages (copies run NST - 1 slices ahead), one tile
// per workgroup.  What bounds such a problem is how fast one CU can stream its operands (a latency per
// slice times the slices, 45 GB/s with a shallow ring), so the tile is small (more CUs stream, each
// fewer bytes), the ring deep, and everything the epilogue needs -- residual rows, bias, LayerNorm
// statistics -- is requested before the first slice instead of after the last.
// Same MFMA, same order of the sums as the other kernels: the same bits.
// ---------------------------------------------------------------------------
template <int WGM, int WGN, int TM, int NST, int EPI, int DIST, bool WF>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_bf16_slim_kernel(
    const bf16raw* __restrict__ a, const bf16raw* __restrict__ wt, const bf16raw* __restrict__ bias,
    const bf16raw* __restrict__ res, bf16raw* __restrict__ out, float* __restrict__ partials,
    const bf16raw* __restrict__ ref, int post, GemmLnFold ln, int M, int N, int K, int ld, int ldo, int tiles_m,
    int tiles_n, int slots, int64_t ldp, int gm) {
    constexpr int NW = WGM * WGN, TN = 2, WM = 32 * TM, WN = 64, BM = WM * WGM, BN = WN * WGN;
    constexpr int RB = 128, RPI = 8;                       // LDS row bytes, rows per wave copy
    constexpr int A_LOADS = BM / RPI / NW, W_LOADS = BN / RPI / NW, LPW = A_LOADS + W_LOADS;
    constexpr int STAGE = (BM + BN) * RB;
    constexpr bool RES = epi_res(EPI);
    static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile rows must split evenly over the wave copies");
    static_assert(NST == 3 || NST == 4, "ring of three or four stages");
    static_assert(NW % 2 == 0, "the parity of a copy's rows >> 3 is that of its wave");
    static_assert(LPW * (NST - 1) <= 63, "copies in flight must fit the counter");
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st3[NST == 4 ? STAGE : 16];
    // residual rows requested up front when there is room for them next to the ring
    constexpr bool PRE_RES = RES && NST * STAGE + NW * TM * 4096 <= 160 * 1024;
    constexpr bool PRE_VEC = NW <= 4;  // two waves per SIMD: no registers for the epilogue's vectors during the loop
    __shared__ __attribute__((aligned(1024))) unsigned char s_epi[PRE_RES ? NW * TM * 4096 : 16];

    const int nblk = tiles_m * tiles_n;
    const int xcd = blockIdx.x & 7;
    const int xq = nblk >> 3, xr = nblk & 7;
    const int x_cnt = xq + (xcd < xr ? 1 : 0), x_start = xcd * xq + (xcd < xr ? xcd : xr);
    const int seq = blockIdx.x >> 3;
    if (seq >= x_cnt) return;  // whole workgroup, before any barrier
    int m0, n0;
    {
        const int bid = x_start + seq;
        const int per_group = gm * tiles_n;
        const int grp = bid / per_group, rem = bid - grp * per_group;
        const int first_m = grp * gm;
        const int gsz = min(tiles_m - first_m, gm);
        const int tn = rem / gsz;
        n0 = tn * BN;
        m0 = (first_m + rem - tn * gsz) * BM;
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;
    const int l32 = lane & 31, g = lane >> 5;
    const int m_base = m0 + wm * WM, n_base = n0 + wn * WN;

    // LDS layout as in gemm_bf16_kernel: chunk c of row r in slot c ^ (r & 7) ^ ((r >> 3) & 1).  Wave copy i of
    // wave w fills rows (NW i + w) 8 .. + 7 (NW is even, so row >> 3 has the parity of w).
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(a + (int64_t)m0 * ld, (int64_t)min(M - m0, BM) * ld * 2);
    const int ldw = WF ? K : ld, wlane = BM * RB + wn * TN * 4096 + lane * 16, wvoff = frag_off(wave / 4, wave % 4, K) + lane * 16;
    const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(wt + (int64_t)n0 * ldw, (int64_t)min(N - n0, BN) * ldw * 2);
    const int ld_r = lane >> 3, ld_p = lane & 7;
    const int voff = ((wave * RPI + ld_r) * ld + ((ld_p ^ ld_r ^ (wave & 1)) << 3)) * 2;
    const int pass_bytes = NW * RPI * ld * 2;
    const int S = K / 64;
    const int a_row0 = wm * WM + l32, w_row0 = wn * WN + l32;
    const int sw = (l32 & 7) ^ ((l32 >> 3) & 1);

#define RS_SLIM_DMA(stage_, t_)                                                                           \
    {                                                                                                     \
        const bool real_ = (t_) < S;                                                                      \
        const int kb_ = (t_) * RB;                                                                        \
        _Pragma("unroll") for (int i = 0; i < A_LOADS; ++i)                                               \
            dma16(rs_a, (stage_) + (i * NW + wave) * 1024, voff, real_ ? i * pass_bytes + kb_ : kPastEnd); \
        _Pragma("unroll") for (int i = 0; i < W_LOADS; ++i) {                                             \
            const int f_ = i * NW + wave;                                                                 \
            if constexpr (WF) dma16(rs_w, (stage_) + BM * RB + f_ * 1024, wvoff, real_ ? frag_off(i * NW / 4, i * NW % 4, K) + (t_) * 4096 : kPastEnd); \
            else dma16(rs_w, (stage_) + BM * RB + f_ * 1024, voff, real_ ? i * pass_bytes + kb_ : kPastEnd); \
        }                                                                                                 \
    }
#define RS_SLIM_FRAGS(f_, stage_, kk_)                                                                    \
    {                                                                                                     \
        const int co_ = ((((kk_) * 2 + g) ^ sw) << 4);                                                    \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                    \
            (f_).w[i] = *reinterpret_cast<const bf16x8*>(                                                 \
                (stage_) + (WF ? wlane + (i * 4 + (kk_)) * 1024 : (BM + w_row0 + i * 32) * RB + co_)); \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                    \
            (f_).a[j] = *reinterpret_cast<const bf16x8*>((stage_) + (a_row0 + j * 32) * RB + co_);        \
    }
#define RS_SLIM_MFMA(f_)                                                                                  \
    {                                                                                                     \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                    \
            _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                \
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16((f_).w[i], (f_).a[j], acc[i][j], 0, 0, 0); \
    }
#define RS_SLIM_WAIT(n_)                                                                                  \
    {                                                                                                     \
        __builtin_amdgcn_s_waitcnt(((n_) & 15) | (((n_) >> 4) << 14) | 0x0070);                           \
        __builtin_amdgcn_s_barrier();                                                                     \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); /* LDS reads stay below the barrier */     \
        __builtin_amdgcn_sched_barrier(0);                                                                \
    }
// Slice t from registers (fc_) while the fragments of slice t + 1 are read from nxt_ into fn_: the wave waits
// for slice t + 1 and for its own reads of slice t, meets the barrier (every wave has slice t in registers:
// cur_ is free), requests slice t + NST into cur_ and starts the reads of slice t + 1, which pass under the
// matrix work.
#define RS_SLIM_SLICE(cur_, nxt_, fc_, fn_, t_)                                                           \
    {                                                                                                     \
        RS_SLIM_WAIT((NST - 2) * LPW)                                                                     \
        RS_SLIM_DMA(cur_, (t_) + NST)                                                                     \
        _Pragma("unroll") for (int kk = 0; kk < 4; ++kk) RS_SLIM_FRAGS(fn_[kk], nxt_, kk)                 \
        _Pragma("unroll") for (int kk = 0; kk < 4; ++kk) RS_SLIM_MFMA(fc_[kk])                            \
        _Pragma("unroll") for (int s_ = 0; s_ < 4 * TN * TM; ++s_) {                                      \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                            \
            __builtin_amdgcn_sched_group_barrier(0x020, (LPW + 4 * TN * TM - 2) / (4 * TN * TM - 1), 0);  \
            __builtin_amdgcn_sched_group_barrier(0x100, (4 * (TN + TM) + 4 * TN * TM - 2) / (4 * TN * TM - 1), 0); \
        }                                                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                                \
    }

#define RS_SLIM_ALL_FRAGS(f_, stage_) { _Pragma("unroll") for (int kk = 0; kk < 4; ++kk) RS_SLIM_FRAGS(f_[kk], stage_, kk) }
#define RS_SLIM_ALL_MFMA(f_) { _Pragma("unroll") for (int kk = 0; kk < 4; ++kk) RS_SLIM_MFMA(f_[kk]) }

    EpiRegions<TM> reg;
    if constexpr (PRE_RES) {
#pragma unroll
        for (int j = 0; j < TM; ++j) reg.r[j] = s_epi + (wave * TM + j) * 4096;
        epi_request_residual<TM>(reg, res, M, N, m_base, n_base, lane);
    } else {
        static_assert(NW * TM * 4096 <= 2 * STAGE, "epilogue regions in the first two stages");
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int at = (wave * TM + j) * 4096;  // STAGE is a multiple of 4096
            reg.r[j] = at < STAGE ? st0 + at : st1 + (at - STAGE);
        }
    }
    EpiVecs<TM, EPI> vec;
    if constexpr (PRE_VEC) vec.load(bias, ln, M, N, m_base, n_base, lane);
    __builtin_amdgcn_sched_barrier(0);
    RS_SLIM_DMA(st0, 0)
    RS_SLIM_DMA(st1, 1)
    RS_SLIM_DMA(st2, 2)
    if constexpr (NST == 4) RS_SLIM_DMA(st3, 3)

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    Frags<TN, TM> f0[4], f1[4];
    RS_SLIM_WAIT((NST - 1) * LPW)  // slice 0 has landed
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) RS_SLIM_FRAGS(f0[kk], st0, kk)
    // Whole trips of the ring, then the slices that are left (fewer than a trip; all of them have been
    // requested by then).  No way out inside a trip: every exit would keep its own copy of the accumulators,
    // and the compiler would lose track of which copies a stage's reads wait for.
    constexpr int TRIP = NST == 3 ? 6 : 4;
    const int full = S / TRIP * TRIP;
    if constexpr (NST == 3) {
        for (int t = 0; t < full; t += 6) {
            RS_SLIM_SLICE(st0, st1, f0, f1, t)
            RS_SLIM_SLICE(st1, st2, f1, f0, t + 1)
            RS_SLIM_SLICE(st2, st0, f0, f1, t + 2)
            RS_SLIM_SLICE(st0, st1, f1, f0, t + 3)
            RS_SLIM_SLICE(st1, st2, f0, f1, t + 4)
            RS_SLIM_SLICE(st2, st0, f1, f0, t + 5)
        }
        const int left = S - full;
        if (left > 0) {
            RS_SLIM_SLICE(st0, st1, f0, f1, full)
            if (left > 1) RS_SLIM_SLICE(st1, st2, f1, f0, full + 1)
            if (left > 2) RS_SLIM_SLICE(st2, st0, f0, f1, full + 2)
            if (left > 3) RS_SLIM_SLICE(st0, st1, f1, f0, full + 3)
            if (left > 4) RS_SLIM_SLICE(st1, st2, f0, f1, full + 4)
        }
    } else {
        for (int t = 0; t < full; t += 4) {
            RS_SLIM_SLICE(st0, st1, f0, f1, t)
            RS_SLIM_SLICE(st1, st2, f1, f0, t + 1)
            RS_SLIM_SLICE(st2, st3, f0, f1, t + 2)
            RS_SLIM_SLICE(st3, st0, f1, f0, t + 3)
        }
        const int left = S - full;
        if (left > 0) {
            RS_SLIM_WAIT(0)
            if (left > 1) RS_SLIM_ALL_FRAGS(f1, st1)
            RS_SLIM_ALL_MFMA(f0)
            if (left > 1) {
                if (left > 2) RS_SLIM_ALL_FRAGS(f0, st2)
                RS_SLIM_ALL_MFMA(f1)
                if (left > 2) RS_SLIM_ALL_MFMA(f0)
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & 0xC07F);  // trailing (empty) copies and reads: the stages get reused
    if (!PRE_RES) __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if constexpr (RES && !PRE_RES) epi_request_residual<TM>(reg, res, M, N, m_base, n_base, lane);
    if constexpr (!PRE_VEC) vec.load(bias, ln, M, N, m_base, n_base, lane);
    if constexpr (RES && !PRE_RES) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#undef RS_SLIM_DMA
#undef RS_SLIM_FRAGS
#undef RS_SLIM_MFMA
#undef RS_SLIM_WAIT
#undef RS_SLIM_ALL_FRAGS
#undef RS_SLIM_ALL_MFMA
#undef RS_SLIM_SLICE
    gemm_epilogue_acc_layout<TM, EPI, DIST>(acc, reg, vec, out, partials, ref, post, M, N, ldo, slots, ldp, m_base, n_base, lane);
}

// ---------------------------------------------------------------------------
// Direct kernel, for weights in fragment order: the weights go from memory straight into the registers of the one
// wave that needs them, only the activations pass through LDS.  Workgroup tile 128 rows x 256 features, four waves of 128 x 64,
// two workgroups per CU.
//
// What bounds these layers at K = 768 is that a tile's epilogue (GELU, residual, 128 KB of stores) is as long as a third of
// its K loop, and in the persistent kernel, one workgroup per CU, the matrix cores wait for it.  Two
// workgroups out of step cover it, but the ring kernel, which has two, pays for that in its K loop: three
// stages of both operands leave room for slices of 32 only, 64-byte row segments, and every line is fetched into L1
// twice.  Without the weights in LDS (a wave's 64 features are no other wave's) four stages of 64-wide activation
// slices take 64 KB, LDS traffic falls from 125 to 78 bytes per cycle of full matrix rate, and every
// request is of whole lines.
//
// A slice: the weights of K step k are requested again, for the next slice, as soon as its matrix
// instructions have been issued (32 registers, 3/4 .. 1 slice ahead); the activation copies run three slices ahead but,
// answers coming in order, are waited for with the weights behind them, one slice later.  Deeper rings (48 or 64
// registers of weights) measured the same: what is left is traffic (8192^3: 810 us; without the copies 734, without
// the weight loads 690, without both 520), not latency.
// The LayerNorm vectors and statistics that the epilogue wants are copied into 3 KB of LDS before the loop (requested after
// it: 768 -> 2304 at 50432 rows +4 %, 768 -> 3072 at 25216 +3 %).
// In a block (us, persistent kernel / this): 50432 x 768 -> 2304 191 / 162, -> 768 with residual 83 / 64, -> 3072 with
// GELU 274 / 230, 50432 x 3072 -> 768 234 / 225, 16388 x 1024 -> 4096 with GELU 162 / 130.
// Same MFMA, same order of the sums as the other kernels: the same bits.
// ---------------------------------------------------------------------------
template <int EPI, int DIST>
__global__ __launch_bounds__(256, 2) void gemm_bf16_direct_kernel(
    const bf16raw* __restrict__ a, const bf16raw* __restrict__ wt, const bf16raw* __restrict__ bias,
    const bf16raw* __restrict__ res, bf16raw* __restrict__ out, float* __restrict__ partials,
    const bf16raw* __restrict__ ref, int post, GemmLnFold ln, int M, int N, int K, int ld, int ldo, int tiles_m,
    int tiles_n, int slots, int64_t ldp, int gm) {
    constexpr int TM = 4, TN = 2, BM = 128, BN = 256, RB = 128, STAGE = BM * RB;
    constexpr bool RES = epi_res(EPI);
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st3[STAGE];
    constexpr bool LN = epi_ln(EPI);
    __shared__ __attribute__((aligned(1024))) unsigned char s_vec[LN ? 3072 : 16];  // what the epilogue reads besides the sums

    const int nblk = tiles_m * tiles_n;
    const int xcd = blockIdx.x & 7;
    const int xq = nblk >> 3, xr = nblk & 7;
    const int x_cnt = xq + (xcd < xr ? 1 : 0), x_start = xcd * xq + (xcd < xr ? xcd : xr);
    const int seq = blockIdx.x >> 3;
    if (seq >= x_cnt) return;  // whole workgroup, before any barrier
    int m0, n0;
    {
        const int bid = x_start + seq;
        const int per_group = gm * tiles_n;
        const int grp = bid / per_group, rem = bid - grp * per_group;
        const int first_m = grp * gm;
        const int gsz = min(tiles_m - first_m, gm);
        const int tn = rem / gsz;
        n0 = tn * BN;
        m0 = (first_m + rem - tn * gsz) * BM;
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int n_base = n0 + wave * 64;
    const int S = K / 64;

    // activations: LDS layout and copies as in gemm_bf16_kernel.  Weights: the wave's two rows of fragments; a wave
    // whose features lie past N has an empty resource and reads zeros
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(a + (int64_t)m0 * ld, (int64_t)min(M - m0, BM) * ld * 2);
    const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(n_base < N ? wt + (int64_t)n_base * K : wt, n_base < N ? (int64_t)K * 128 : 0);
    const int ld_r = lane >> 3, ld_p = lane & 7;
    const int voff = ((wave * 8 + ld_r) * ld + ((ld_p ^ ld_r ^ (wave & 1)) << 3)) * 2;
    const int pass_bytes = 32 * ld * 2;
    const int sw = (l32 & 7) ^ ((l32 >> 3) & 1);
    const int woff0 = lane * 16, woff1 = woff0 + K * 64;

#define RS_DIRECT_DMA(stage_, t_)                                                                         \
    {                                                                                                     \
        const bool real_ = (t_) < S;                                                                      \
        const int kb_ = (t_) * RB;                                                                        \
        _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                     \
            dma16(rs_a, (stage_) + (i * 4 + wave) * 1024, voff, real_ ? i * pass_bytes + kb_ : kPastEnd); \
    }
// weights of K step kk_ of slice t_
#define RS_DIRECT_W(kk_, t_)                                                                              \
    {                                                                                                     \
        const int so_ = (t_) < S ? ((t_) * 4 + (kk_)) * 1024 : kPastEnd;                                  \
        w[kk_][0] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_w, woff0, so_, 0)); \
        w[kk_][1] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_w, woff1, so_, 0)); \
    }
#define RS_DIRECT_FRAGS(f_, stage_, kk_)                                                                  \
    {                                                                                                     \
        const int co_ = ((((kk_) * 2 + g) ^ sw) << 4);                                                    \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                    \
            f_[j] = *reinterpret_cast<const bf16x8*>((stage_) + (l32 + j * 32) * RB + co_);               \
    }
#define RS_DIRECT_MFMA(f_, kk_)                                                                           \
    {                                                                                                     \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                    \
            _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                \
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[kk_][i], f_[j], acc[i][j], 0, 0, 0); \
    }
// one K step: an LDS read of the next step's rows, two MFMAs, a request
#define RS_DIRECT_INTERLEAVE()                                                                            \
    {                                                                                                     \
        _Pragma("unroll") for (int s_ = 0; s_ < TM; ++s_) {                                               \
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                            \
            __builtin_amdgcn_sched_group_barrier(0x008, TN, 0);                                           \
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                            \
        }                                                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                                \
    }
// Everything but the newest n_ requests has been answered, and this wave's LDS reads all have.
#define RS_DIRECT_WAIT(n_)                                                                                \
    {                                                                                                     \
        __builtin_amdgcn_s_waitcnt(((n_) & 15) | (((n_) >> 4) << 14) | 0x0070);                           \
        __builtin_amdgcn_s_barrier();                                                                     \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); /* LDS reads stay below the barrier */     \
        __builtin_amdgcn_sched_barrier(0);                                                                \
    }
// Slice t from cur_ (its first fragments are in f0).  fre_ held slice t - 1, which every wave has read before the last
// barrier: the copies of slice t + 3 go there.  At this slice's barrier those of slice t + 1 must have landed: behind them
// lie at least the copies of slices t + 2 and t + 3 and this slice's 6 weight loads.
#define RS_DIRECT_SLICE(cur_, nxt_, fre_, t_)                                                             \
    {                                                                                                     \
        RS_DIRECT_DMA(fre_, (t_) + 3)                                                                     \
        RS_DIRECT_FRAGS(f1, cur_, 1)                                                                      \
        RS_DIRECT_MFMA(f0, 0)                                                                             \
        RS_DIRECT_INTERLEAVE()                                                                            \
        RS_DIRECT_W(0, (t_) + 1)                                                                          \
        RS_DIRECT_FRAGS(f0, cur_, 2)                                                                      \
        RS_DIRECT_MFMA(f1, 1)                                                                             \
        RS_DIRECT_INTERLEAVE()                                                                            \
        RS_DIRECT_W(1, (t_) + 1)                                                                          \
        RS_DIRECT_FRAGS(f1, cur_, 3)                                                                      \
        RS_DIRECT_MFMA(f0, 2)                                                                             \
        RS_DIRECT_INTERLEAVE()                                                                            \
        RS_DIRECT_W(2, (t_) + 1)                                                                          \
        RS_DIRECT_WAIT(14)                                                                                \
        RS_DIRECT_FRAGS(f0, nxt_, 0)                                                                      \
        RS_DIRECT_MFMA(f1, 3)                                                                             \
        RS_DIRECT_INTERLEAVE()                                                                            \
        RS_DIRECT_W(3, (t_) + 1)                                                                          \
    }

    bf16x8 w[4][TN], f0[TM], f1[TM];
    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    RS_DIRECT_DMA(st0, 0)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) RS_DIRECT_W(kk, 0)
    __builtin_amdgcn_sched_barrier(0);
    RS_DIRECT_DMA(st1, 1)
    RS_DIRECT_DMA(st2, 2)
    if constexpr (LN) EpiVecs<TM, EPI>::request(s_vec, ln, M, N, m0, n0, wave, lane);
    RS_DIRECT_WAIT(16)  // slice 0 has landed: behind it at least 8 weight loads and two slices' copies
    RS_DIRECT_FRAGS(f0, st0, 0)
    // whole trips of the ring, then the slices that are left; no way out inside a trip (every exit would keep its own
    // copy of the accumulators)
    const int full = S & ~3, left = S & 3;
    for (int t = 0; t < full; t += 4) {
        RS_DIRECT_SLICE(st0, st1, st3, t)
        RS_DIRECT_SLICE(st1, st2, st0, t + 1)
        RS_DIRECT_SLICE(st2, st3, st1, t + 2)
        RS_DIRECT_SLICE(st3, st0, st2, t + 3)
    }
    if (left > 0) {
        RS_DIRECT_SLICE(st0, st1, st3, full)
        if (left > 1) RS_DIRECT_SLICE(st1, st2, st0, full + 1)
        if (left > 2) RS_DIRECT_SLICE(st2, st3, st1, full + 2)
    }
    RS_DIRECT_WAIT(0)  // trailing (empty) copies: the stages get reused
#undef RS_DIRECT_DMA
#undef RS_DIRECT_W
#undef RS_DIRECT_FRAGS
#undef RS_DIRECT_MFMA
#undef RS_DIRECT_INTERLEAVE
#undef RS_DIRECT_WAIT
#undef RS_DIRECT_SLICE

    EpiRegions<TM> reg;
    unsigned char* const base = wave == 0 ? st0 : wave == 1 ? st1 : wave == 2 ? st2 : st3;
#pragma unroll
    for (int j = 0; j < TM; ++j) reg.r[j] = base + j * 4096;
    EpiVecs<TM, EPI> vec;
    if constexpr (RES) epi_request_residual<TM>(reg, res, M, N, m0, n_base, lane);
    if constexpr (LN) vec.from_lds(s_vec, wave * 64, lane);
    else vec.load(bias, ln, M, N, m0, n_base, lane);
    if constexpr (RES) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // every residual row of the tile has landed
    gemm_epilogue_acc_layout<TM, EPI, DIST>(acc, reg, vec, out, partials, ref, post, M, N, ldo, slots, ldp, m0, n_base, lane);
}

// Tile configuration of the bf16 GEMM: BM, BN, BK, NSTAGE, waves along tokens, waves along features.
#ifndef RS_GEMM_GM
#define RS_GEMM_GM 8
#endif
struct GemmCfg {
#ifndef RS_GEMM_CFG
#define RS_GEMM_CFG 256, 256, 64, 2, 2, 4
#endif
    static constexpr int P[6] = {RS_GEMM_CFG};
    static constexpr int BM = P[0], BN = P[1], BK = P[2], NSTAGE = P[3], WGM = P[4], WGN = P[5];
    static constexpr int WN = BN / WGN;
};

int device_cus() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
        return n;
    }();
    return cus;
}

// Which bf16 tile variant runs: 0 = chosen by shape (below), 1 = 256 x 256 persistent kernel,
// 2 = 256 x 128 slim kernel, 3 = 128 x 128 ring kernel, 4 = 128 x 256 direct kernel (weights in rows: ring).  Every variant gives the same bits; the
// switch exists for tuning and for the test that checks exactly that.  Initial value from the
// environment variable RS_GEMM_FORCE.
static std::atomic<int> g_gemm_variant{-1};

int gemm_variant() {
    int v = g_gemm_variant.load(std::memory_order_relaxed);
    if (v < 0) {
        const char* e = getenv("RS_GEMM_FORCE");
        v = e ? atoi(e) : 0;
        if (v < 0 || v > 4) v = 0;
        g_gemm_variant.store(v);
    }
    return v;
}

void set_gemm_variant(int v) { g_gemm_variant.store(v >= 0 && v <= 4 ? v : 0); }

struct GemmArgs {
    const bf16raw *a, *wt, *bias, *res, *ref;
    bf16raw* out;
    float* partials;
    int post;
    GemmLnFold ln;
    int64_t M;
    int N, K;
    int ld, ldo;  // elements between the rows of a and wt, and of out (res and ref: N)
    int64_t ldp;  // floats between the slots of the shift sums: the rows of the whole problem
    // the same problem restricted to rows [r0, r1)
    GemmArgs rows(int64_t r0, int64_t r1) const {
        GemmArgs g = *this;
        g.a = a + r0 * ld;
        g.res = res ? res + r0 * N : nullptr;
        g.ref = ref ? ref + r0 * N : nullptr;
        g.out = out + r0 * ldo;
        g.partials = partials ? partials + r0 : nullptr;
        g.ln.stats = ln.stats ? ln.stats + r0 * 2 : nullptr;
        g.M = r1 - r0;
        return g;
    }
};

template <int BM, int BN, int EPI, int DIST, bool WF>
static void launch_ring(const GemmArgs& g, hipStream_t s) {
    const int tiles_m = (int)((g.M + BM - 1) / BM), tiles_n = (g.N + BN - 1) / BN;
    const int nblk = tiles_m * tiles_n;
    constexpr int WGN = BN / 64, WGM = 4 / WGN;  // four waves, each 64 features wide
    hipLaunchKernelGGL((gemm_bf16_ring_kernel<BM, BN, WGM, WGN, EPI, DIST, WF>), dim3(8 * ((nblk + 7) / 8)), dim3(256), 0, s,
                       g.a, g.wt, g.bias, g.res, g.out, g.partials, g.ref, g.post, g.ln, (int)g.M, g.N, g.K, g.ld, g.ldo, tiles_m,
                       tiles_n, (g.N + 63) / 64, g.ldp, RS_GEMM_GM, GemmBatch{0, 0, 0});
}

template <int WGM, int WGN, int TM, int NST, int EPI, int DIST, bool WF>
static void launch_slim(const GemmArgs& g, hipStream_t s) {
    constexpr int BM = 32 * TM * WGM, BN = 64 * WGN;
    const int tiles_m = (int)((g.M + BM - 1) / BM), tiles_n = (g.N + BN - 1) / BN;
    const int nblk = tiles_m * tiles_n;
    hipLaunchKernelGGL((gemm_bf16_slim_kernel<WGM, WGN, TM, NST, EPI, DIST, WF>), dim3(8 * ((nblk + 7) / 8)), dim3(WGM * WGN * 64), 0, s,
                       g.a, g.wt, g.bias, g.res, g.out, g.partials, g.ref, g.post, g.ln, (int)g.M, g.N, g.K, g.ld, g.ldo, tiles_m,
                       tiles_n, (g.N + 63) / 64, g.ldp, RS_GEMM_GM);
}

// The ring kernel with the tile width that suits the grid.  128 x 128 tiles unless they would leave
// some CUs two workgroups and others one (more than one workgroup per CU, at most two): then the
// 128 x 256 tiles, half as many, give every CU one workgroup of the same length (fc2 at 6280 rows:
// 58 -> 48 us); and for large grids, where the wider tile moves fewer bytes per flop.
template <int EPI, int DIST>
static void launch_ring_auto(const GemmArgs& g, hipStream_t s) {
    const int cus = device_cus();
    const int64_t n128 = ((g.M + 127) / 128) * ((g.N + 127) / 128);  // workgroups of the 128 x 128 tiling
    if ((n128 > cus && n128 <= 2 * cus) || n128 >= 4 * cus) launch_ring<128, 256, EPI, DIST, false>(g, s);
    else launch_ring<128, 128, EPI, DIST, false>(g, s);
}

// With a long K (at least 2048, and a slice count that the six-slice trip of the deeper ring pads
// by under 5 %) the kernel runs with three activation stages: its copies, not its matrix work,
// set the pace there (fc2 of ViT-B: -5 %); with a short K the tile is mostly prologue and
// epilogue and the third stage's extra requests cost more than they hide (+2..5 %).
static bool gemm_deep_stages(int K) {
    static const int force = [] { const char* e = getenv("RS_GEMM_STAGES"); return e ? atoi(e) : 0; }();  // tuning aid: 2 or 3
    if (force == 2 || force == 3) return force == 3;
    const int S = K / 64, pad = (S + 5) / 6 * 6 - S;
    return K >= 2048 && 20 * pad <= S;
}

template <int EPI, int DIST, bool WF>
static void launch_persistent(const GemmArgs& g, hipStream_t s) {
    using C = GemmCfg;
    const int tiles_m = (int)((g.M + C::BM - 1) / C::BM), tiles_n = (g.N + C::BN - 1) / C::BN;
    // one workgroup per CU (8 XCDs x CUs / 8), fewer when an XCD's share of the tiles is smaller
    const int cus = device_cus();
    const int share = (tiles_m * tiles_n + 7) / 8;
    const int per_xcd = share < cus / 8 ? share : cus / 8;
    if (gemm_deep_stages(g.K))
        hipLaunchKernelGGL((gemm_bf16_kernel<C::BM, C::BN, C::BK, 3, C::WGM, C::WGN, EPI, DIST, WF>),
                           dim3(8 * per_xcd), dim3(C::WGM * C::WGN * 64), 0, s, g.a, g.wt, g.bias, g.res, g.out, g.partials,
                           g.ref, g.post, g.ln, (int)g.M, g.N, g.K, g.ld, g.ldo, tiles_m, tiles_n, (g.N + 63) / 64, g.ldp, RS_GEMM_GM);
    else
        hipLaunchKernelGGL((gemm_bf16_kernel<C::BM, C::BN, C::BK, 2, C::WGM, C::WGN, EPI, DIST, WF>),
                           dim3(8 * per_xcd), dim3(C::WGM * C::WGN * 64), 0, s, g.a, g.wt, g.bias, g.res, g.out, g.partials,
                           g.ref, g.post, g.ln, (int)g.M, g.N, g.K, g.ld, g.ldo, tiles_m, tiles_n, (g.N + 63) / 64, g.ldp, RS_GEMM_GM);
}

// Weights in fragment order only.
template <int EPI, int DIST>
static void launch_direct(const GemmArgs& g, hipStream_t s) {
    const int tiles_m = (int)((g.M + 127) / 128), tiles_n = (g.N + 255) / 256;
    const int nblk = tiles_m * tiles_n;
    hipLaunchKernelGGL((gemm_bf16_direct_kernel<EPI, DIST>), dim3(8 * ((nblk + 7) / 8)), dim3(256), 0, s, g.a, g.wt, g.bias, g.res,
                       g.out, g.partials, g.ref, g.post, g.ln, (int)g.M, g.N, g.K, g.ld, g.ldo, tiles_m, tiles_n, (g.N + 63) / 64,
                       g.ldp, 2 * RS_GEMM_GM);
}

// The kernels that the choice by shape (gemm_choice.hpp) names, from the first row to the last.
template <int EPI, int DIST, bool WF>
static void launch_by_shape(const GemmArgs& g, hipStream_t s) {
    for (int64_t r = 0; r < g.M;) {
        const GemmChoice c = WF ? gemm_choose_frag(g.M - r, g.N, g.K, device_cus(), epi_res(EPI)) : gemm_choose(g.M - r, g.N, g.K, device_cus());
        const GemmArgs part = g.rows(r, r + c.rows);
        switch (c.tile) {
            case GemmTile::Slim64x64: launch_slim<2, 1, 1, 4, EPI, DIST, WF>(part, s); break;
            case GemmTile::Slim128x64: launch_slim<4, 1, 1, 4, EPI, DIST, WF>(part, s); break;
            case GemmTile::Slim128x128: launch_slim<2, 2, 2, 3, EPI, DIST, WF>(part, s); break;
            case GemmTile::Slim256x128: launch_slim<4, 2, 2, 3, EPI, DIST, WF>(part, s); break;
            case GemmTile::Ring:
                if constexpr (WF) launch_ring<128, 128, EPI, DIST, true>(part, s);
                else launch_ring_auto<EPI, DIST>(part, s);
                break;
            case GemmTile::Direct: if constexpr (WF) launch_direct<EPI, DIST>(part, s); break;
            case GemmTile::Persistent: launch_persistent<EPI, DIST, WF>(part, s); break;
        }
        r += c.rows;
    }
}

template <int EPI, int DIST, bool WF>
static hipError_t launch_bf16(const void* a, const void* wt, const void* bias, const void* res,
                              void* out, float* partials, const void* ref, bool post, GemmLnFold ln,
                              int64_t M, int N, int K, int ld, int ldo, hipStream_t s) {
    const GemmArgs g{(const bf16raw*)a, (const bf16raw*)wt, (const bf16raw*)bias, (const bf16raw*)res,
                     (const bf16raw*)ref, (bf16raw*)out, partials, post ? 1 : 0, ln, M, N, K, ld, ldo, M};
    const int variant = gemm_variant();
    if (variant == 1) launch_persistent<EPI, DIST, WF>(g, s);
    else if (variant == 2) launch_slim<4, 2, 2, 3, EPI, DIST, WF>(g, s);
    else if (variant == 3) launch_ring<128, 128, EPI, DIST, WF>(g, s);
    else if (variant == 4) {
        if constexpr (WF) launch_direct<EPI, DIST>(g, s);
        else launch_ring<128, 256, EPI, DIST, WF>(g, s);
    } else launch_by_shape<EPI, DIST, WF>(g, s);
    return hipGetLastError();
}

#define RS_STR2(...) #__VA_ARGS__
#define RS_STR(...) RS_STR2(__VA_ARGS__)
const char* gemm_build_info() {
    return "bf16 gemm, block: weights in fragments; slim tiles 64x64, 128x64, 128x128, 256x128 up to one workgroup per CU (256x128 to two"
           " where the direct tiles are more), direct tiles 128x256 beyond, ring tiles 128x128x32 or slim to 128 features; persistent tiles"
           " (BM,BN,BK,stages,waves m,waves n) " RS_STR(RS_GEMM_CFG) ", three activation stages when K >= 2048, when K >= 1536 and the last"
           " round is more than 0.5 full (0.6 below K = 3072), and for the whole rounds when K >= 2048 and it is at most 1/6 full, the rows"
           " behind them apart; rs_linear_fwd: weights in rows; slim (256x128 up to 1.45 rounds of 256x256 when K < 2048), persistent, ring"
           " tiles 128x128x32 and 128x256x32 beyond one round when K <= 384, rows behind whole rounds apart when K >= 2048 and the last round"
           " is at most 0.5 full";
}

// `count` independent products out_p[M, N] = a_p[M, K] @ wt_p[N, K]^T (bf16, no bias), problem p at
// element offsets p * stride from the base pointers; 128 x 128 tiles, grid.y = problem.
hipError_t launch_gemm_batched(const void* a, const void* wt, void* out, int count, int64_t stride_a,
                               int64_t stride_w, int64_t stride_out, int M, int N, int K, hipStream_t s) {
    if (count == 0 || M == 0) return hipSuccess;
    const GemmBatch gb{stride_a, stride_w, stride_out};
    if (N <= 64) {  // one 64-wide wave column: 256 x 64 tiles, four waves along the rows
        const int tiles_m = (M + 255) / 256;
        hipLaunchKernelGGL((gemm_bf16_ring_kernel<256, 64, 4, 1, EPI_BIAS, 0, false>), dim3(8 * ((tiles_m + 7) / 8), count), dim3(256), 0, s,
                           (const bf16raw*)a, (const bf16raw*)wt, (const bf16raw*)nullptr, (const bf16raw*)nullptr,
                           (bf16raw*)out, (float*)nullptr, (const bf16raw*)nullptr, 0, GemmLnFold{}, M, N, K, K, N, tiles_m, 1,
                           1, (int64_t)0, RS_GEMM_GM, gb);
    } else {
        const int tiles_m = (M + 127) / 128, tiles_n = (N + 127) / 128;
        const int nblk = tiles_m * tiles_n;
        hipLaunchKernelGGL((gemm_bf16_ring_kernel<128, 128, 2, 2, EPI_BIAS, 0, false>), dim3(8 * ((nblk + 7) / 8), count), dim3(256), 0, s,
                           (const bf16raw*)a, (const bf16raw*)wt, (const bf16raw*)nullptr, (const bf16raw*)nullptr,
                           (bf16raw*)out, (float*)nullptr, (const bf16raw*)nullptr, 0, GemmLnFold{}, M, N, K, K, N, tiles_m,
                           tiles_n, (N + 63) / 64, (int64_t)0, RS_GEMM_GM, gb);
    }
    return hipGetLastError();
}

int gemm_shift_slots(rs_dtype dt, int N) {
    (void)dt;
    return (N + 63) / 64;  // one slot per 64 features, whatever the type and the tile variant
}

hipError_t launch_gemm(rs_dtype dt, GemmEpilogue epi, rs_dist dist, const void* a, const void* w,
                       const void* bias, const void* res, void* out, float* partials, const void* ref,
                       bool post, int64_t M, int N, int K, hipStream_t s, bool frag, int ld, int ldo) {
    if (M == 0) return hipSuccess;
    if (dt == RS_F32) return launch_gemm_f32(epi, dist, a, w, bias, res, out, partials, ref, post, M, N, K, s);
    const GemmLnFold ln{};
    ld = ld ? ld : K;
    ldo = ldo ? ldo : N;
#define RS_GEMM_GO(EPI_, DIST_, WF_) return launch_bf16<EPI_, DIST_, WF_>(a, w, bias, res, out, partials, ref, post, ln, M, N, K, ld, ldo, s)
    if (!frag) {
        if (epi == EPI_BIAS) RS_GEMM_GO(EPI_BIAS, 0, false);
        if (epi == EPI_BIAS_GELU) RS_GEMM_GO(EPI_BIAS_GELU, 0, false);
        if (epi == EPI_BIAS_RES) RS_GEMM_GO(EPI_BIAS_RES, 0, false);
    } else {  // the block's layers; those behind a LayerNorm go through launch_gemm_ln
        if (epi == EPI_BIAS_RES) RS_GEMM_GO(EPI_BIAS_RES, 0, true);
        if (epi == EPI_BIAS_RES_SHIFT) {
            if (dist == RS_DIST_L2) RS_GEMM_GO(EPI_BIAS_RES_SHIFT, RS_DIST_L2, true);
            if (dist == RS_DIST_L1) RS_GEMM_GO(EPI_BIAS_RES_SHIFT, RS_DIST_L1, true);
            RS_GEMM_GO(EPI_BIAS_RES_SHIFT, RS_DIST_COS, true);
        }
    }
#undef RS_GEMM_GO
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_ln(GemmEpilogue epi, const void* x, const void* w_folded, GemmLnFold ln, void* out,
                          int64_t M, int N, int K, hipStream_t s, int ld, int ldo) {
    if (M == 0) return hipSuccess;
    ld = ld ? ld : K;
    ldo = ldo ? ldo : N;
    if (epi == EPI_LN_BIAS)
        return launch_bf16<EPI_LN_BIAS, 0, true>(x, w_folded, nullptr, nullptr, out, nullptr, nullptr, false, ln, M, N, K, ld, ldo, s);
    if (epi == EPI_LN_BIAS_GELU)
        return launch_bf16<EPI_LN_BIAS_GELU, 0, true>(x, w_folded, nullptr, nullptr, out, nullptr, nullptr, false, ln, M, N, K, ld, ldo, s);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Weight re-layout for the bf16 path: [K, N] row-major -> [N, K] row-major (rs_pack_linear), or into the
// fragment order of the block's kernels, there optionally with row k scaled by gamma[k] (a LayerNorm
// scale folded into the weights; the product is rounded to bf16).  64 x 64 tiles through LDS, coalesced on both sides.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bf16raw fold_gamma(bf16raw w, const bf16raw* gamma, int k) {
    return gamma ? f2bf(bf2f(gamma[k]) * bf2f(w)) : w;
}

__global__ __launch_bounds__(256) void transpose_bf16_kernel(const bf16raw* __restrict__ w, bf16raw* __restrict__ wt, int K, int N) {
    __shared__ bf16raw tile[64][66];
    const int k0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int r = ty; r < 64; r += 4) {
        const int k = k0 + r, n = n0 + tx;
        tile[r][tx] = (k < K && n < N) ? w[(int64_t)k * N + n] : (bf16raw)0;
    }
    __syncthreads();
    for (int r = ty; r < 64; r += 4) {
        const int n = n0 + r, k = k0 + tx;
        if (n < N && k < K) wt[(int64_t)n * K + k] = tile[tx][r];
    }
}

hipError_t launch_pack_transpose(const void* w, void* wt, int K, int N, hipStream_t s) {
    dim3 grid((N + 63) / 64, (K + 63) / 64);
    hipLaunchKernelGGL(transpose_bf16_kernel, grid, dim3(256), 0, s, (const bf16raw*)w, (bf16raw*)wt, K, N);
    return hipGetLastError();
}

// [K, N] row-major -> fragment order (frag_off), optionally with row k scaled by gamma[k]; N and K are multiples of 64.  A
// workgroup takes 64 x 64 elements through LDS: 2 x 4 fragments, written 16 bytes per lane.  `tail` elements behind the
// last fragment are written as zeros (the buffer's size does not depend on how it is laid out).
__global__ __launch_bounds__(256) void pack_frag_kernel(const bf16raw* __restrict__ w, const bf16raw* __restrict__ gamma,
                                                        bf16raw* __restrict__ wf, int K, int N, int64_t tail) {
    __shared__ bf16raw tile[64][66];
    const int k0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int r = ty; r < 64; r += 4) tile[r][tx] = fold_gamma(w[(int64_t)(k0 + r) * N + n0 + tx], gamma, k0 + r);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int f = h, kk = ty, n = f * 32 + (tx & 31), k = kk * 16 + (tx >> 5) * 8;
        uint32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = tile[k + 2 * e][n] | (uint32_t)tile[k + 2 * e + 1][n] << 16;
        const int64_t at = ((int64_t)(n0 / 32 + f) * (K / 16) + k0 / 16 + kk) * 512 + tx * 8;
        *reinterpret_cast<uint4*>(wf + at) = make_uint4(v[0], v[1], v[2], v[3]);
    }
    if (tail > 0) {
        const int64_t id = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x, step = (int64_t)gridDim.x * gridDim.y * 256;
        for (int64_t i = id; i < tail; i += step) wf[(int64_t)N * K + i] = 0;
    }
}

hipError_t launch_pack_frag(const void* w, const void* gamma, void* wf, int K, int N, int64_t tail, hipStream_t s) {
    hipLaunchKernelGGL(pack_frag_kernel, dim3(N / 64, K / 64), dim3(256), 0, s, (const bf16raw*)w, (const bf16raw*)gamma,
                       (bf16raw*)wf, K, N, tail);
    return hipGetLastError();
}

// Column vectors of a LayerNorm folded into the linear layer behind it:
//   colsum[n] = sum_k bf16(gamma_k w_kn)   -- over exactly the values pack_frag_kernel stores,
//                                             so that mean * colsum cancels the mean's share of acc
//   bias_out[n] = sum_k beta_k w_kn + bias[n]
// One thread per column, 4 row groups per workgroup reduced through LDS; fp64 sums (one-off work).
__global__ __launch_bounds__(256) void ln_fold_kernel(const bf16raw* __restrict__ w, const bf16raw* __restrict__ gamma,
                                                      const bf16raw* __restrict__ beta, const bf16raw* __restrict__ bias,
                                                      float* __restrict__ colsum, float* __restrict__ bias_out,
                                                      int K, int N) {
    __shared__ double s_cs[4][64], s_bb[4][64];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int n = blockIdx.x * 64 + tx;
    double cs = 0.0, bb = 0.0;
    if (n < N)
        for (int k = ty; k < K; k += 4) {
            const bf16raw wv = w[(int64_t)k * N + n];
            cs += (double)bf2f(fold_gamma(wv, gamma, k));
            if (beta) bb += (double)bf2f(beta[k]) * (double)bf2f(wv);
        }
    s_cs[ty][tx] = cs;
    s_bb[ty][tx] = bb;
    __syncthreads();
    if (ty == 0 && n < N) {
        cs = ((s_cs[0][tx] + s_cs[1][tx]) + s_cs[2][tx]) + s_cs[3][tx];
        bb = ((s_bb[0][tx] + s_bb[1][tx]) + s_bb[2][tx]) + s_bb[3][tx];
        if (bias) bb += (double)bf2f(bias[n]);
        colsum[n] = (float)cs;
        bias_out[n] = (float)bb;
    }
}

hipError_t launch_pack_ln_fold(const void* w, const void* gamma, const void* beta, const void* bias,
                               float* colsum, float* bias_out, int K, int N, hipStream_t s) {
    hipLaunchKernelGGL(ln_fold_kernel, dim3((N + 63) / 64), dim3(256), 0, s, (const bf16raw*)w,
                       (const bf16raw*)gamma, (const bf16raw*)beta, (const bf16raw*)bias, colsum, bias_out, K, N);
    return hipGetLastError();
}

}  // namespace rs
