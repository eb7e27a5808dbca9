// Representation-shift score, token selection and compaction
// (Eq. (4) of Sec. 3.2; "Distance metrics", Sec. 3.3; pruning of the lowest-score
// tokens, Secs. 3.1 and 3.2).  All of it is HBM-bound: the score pass streams F(x)
// and x once, the selection works on N floats per image, the gather copies K rows.
#include <type_traits>

#include "common.hpp"

namespace rs {

// ---------------------------------------------------------------------------
// scores[row] = D(f_out[row, :], f_in[row, :]); one wavefront per row, 8 elements per
// lane per step, butterfly reduction in a fixed order (bit-reproducible).
// ---------------------------------------------------------------------------
template <typename T, int DIST>
__global__ __launch_bounds__(256) void shift_scores_kernel(const T* __restrict__ f_out,
                                                           const T* __restrict__ f_in,
                                                           float* __restrict__ scores, int64_t M,
                                                           int D) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= M) return;
    const T* a = f_out + row * D;
    const T* b = f_in + row * D;
    float p0 = 0.f, p1 = 0.f, p2 = 0.f;
    for (int c = lane * 8; c < D; c += 64 * 8) {
        float x[8], y[8];
        Elem<T>::load8(a + c, x);
        Elem<T>::load8(b + c, y);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (DIST == RS_DIST_L2) { float d = x[i] - y[i]; p0 = fmaf(d, d, p0); }
            else if (DIST == RS_DIST_L1) { p0 += fabsf(x[i] - y[i]); }
            else { p0 = fmaf(x[i], y[i], p0); p1 = fmaf(x[i], x[i], p1); p2 = fmaf(y[i], y[i], p2); }
        }
    }
    p0 = wave_sum(p0);
    if (DIST == RS_DIST_COS) { p1 = wave_sum(p1); p2 = wave_sum(p2); }
    if (lane == 0) {
        float s;
        if (DIST == RS_DIST_L2) s = sqrtf(p0);
        else if (DIST == RS_DIST_L1) s = p0;
        else s = 1.0f - p0 / (sqrtf(p1) * sqrtf(p2));
        scores[row] = s;
    }
}

// One value's share of the three sums a distance is made of, and the distance from the sums.
template <int DIST>
__device__ __forceinline__ void dist_term(float x, float y, float& p0, float& p1, float& p2) {
    if (DIST == RS_DIST_L2) { const float d = x - y; p0 = fmaf(d, d, p0); }
    else if (DIST == RS_DIST_L1) { p0 += fabsf(x - y); }
    else { p0 = fmaf(x, y, p0); p1 = fmaf(x, x, p1); p2 = fmaf(y, y, p2); }
}
template <int DIST>
__device__ __forceinline__ float dist_value(float p0, float p1, float p2) {
    if (DIST == RS_DIST_L2) return sqrtf(p0);
    if (DIST == RS_DIST_L1) return p0;
    return 1.0f - p0 / (sqrtf(p1) * sqrtf(p2));
}

// Score of the row a group of G consecutive lanes holds, lane `sub` of the group elements 8 sub .. 8 sub + 7
// (zeros past the row's end): the same additions as shift_scores_kernel's, whose missing lanes add
// zeros, hence the same bits.
template <int DIST, int G>
__device__ __forceinline__ float group_score(const float (&x)[8], const float (&y)[8]) {
    float p0 = 0.f, p1 = 0.f, p2 = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) dist_term<DIST>(x[i], y[i], p0, p1, p2);
    p0 = lanes_sum<G>(p0);
    if (DIST == RS_DIST_COS) { p1 = lanes_sum<G>(p1); p2 = lanes_sum<G>(p2); }
    return dist_value<DIST>(p0, p1, p2);
}

// Narrow rows (D <= 8 G, G = 8, 16 or 32 lanes): 64 / G rows per wave and four such groups of rows per
// thread, all requested before the first is summed.  With one wave per row a 64-channel map kept 8 of
// 64 lanes busy with one 16-byte request each.
template <typename T, int DIST, int G>
__global__ __launch_bounds__(256) void shift_scores_narrow_kernel(const T* __restrict__ f_out,
                                                                  const T* __restrict__ f_in,
                                                                  float* __restrict__ scores, int64_t M, int D) {
    constexpr int U = 4, RPG = 256 / G;  // row groups per thread, rows per workgroup and group
    const int sub = threadIdx.x % G;
    const int64_t row0 = (int64_t)blockIdx.x * (RPG * U) + threadIdx.x / G;
    const bool on = sub * 8 < D;
    float x[U][8], y[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t row = row0 + u * RPG;
        if (on && row < M) {
            Elem<T>::load8(f_out + row * D + sub * 8, x[u]);
            Elem<T>::load8(f_in + row * D + sub * 8, y[u]);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[u][i] = y[u][i] = 0.f;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t row = row0 + u * RPG;
        const float sc = group_score<DIST, G>(x[u], y[u]);
        if (sub == 0 && row < M) scores[row] = sc;
    }
}

template <typename T>
static hipError_t launch_scores_t(rs_dist dist, const void* f_out, const void* f_in, float* scores,
                                  int64_t M, int D, hipStream_t s) {
    const T* a = (const T*)f_out;
    const T* b = (const T*)f_in;
#define RS_SCORES(KERNEL_, ROWS_)                                                                                \
    hipLaunchKernelGGL(KERNEL_, dim3((unsigned)((M + (ROWS_) - 1) / (ROWS_))), dim3(256), 0, s, a, b, scores, M, D)
#define RS_SCORES_D(DIST_)                                                                                       \
    if (D <= 64) RS_SCORES((shift_scores_narrow_kernel<T, DIST_, 8>), 128);                                      \
    else if (D <= 128) RS_SCORES((shift_scores_narrow_kernel<T, DIST_, 16>), 64);                                \
    else if (D <= 256) RS_SCORES((shift_scores_narrow_kernel<T, DIST_, 32>), 32);                                \
    else RS_SCORES((shift_scores_kernel<T, DIST_>), 4);
    if (dist == RS_DIST_L2) { RS_SCORES_D(RS_DIST_L2) }
    else if (dist == RS_DIST_L1) { RS_SCORES_D(RS_DIST_L1) }
    else { RS_SCORES_D(RS_DIST_COS) }
#undef RS_SCORES_D
#undef RS_SCORES
    return hipGetLastError();
}

hipError_t launch_shift_scores(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in,
                               float* scores, int64_t M, int D, hipStream_t s) {
    if (M == 0) return hipSuccess;
    return dt == RS_F32 ? launch_scores_t<float>(dist, f_out, f_in, scores, M, D, s)
                        : launch_scores_t<bf16raw>(dist, f_out, f_in, scores, M, D, s);
}

// ---------------------------------------------------------------------------
// scores from the GEMM epilogue's per-row partial slots ([kShiftLanes][slots][M]), summed in slot order.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float score_from_partials(const float* __restrict__ partials, int slots, int64_t M, int64_t row,
                                                     int dist) {
    const float* p = partials + row;
    float p0 = 0.f, p1 = 0.f, p2 = 0.f;
#pragma unroll 4
    for (int s = 0; s < slots; ++s) p0 += p[s * M];
    if (dist == RS_DIST_COS) {
#pragma unroll 4
        for (int s = 0; s < slots; ++s) { p1 += p[(slots + s) * M]; p2 += p[(2 * slots + s) * M]; }
        return dist_value<RS_DIST_COS>(p0, p1, p2);
    }
    return dist == RS_DIST_L2 ? dist_value<RS_DIST_L2>(p0, p1, p2) : p0;
}

__global__ __launch_bounds__(256) void finalize_scores_kernel(const float* __restrict__ partials,
                                                              int slots, int dist,
                                                              float* __restrict__ scores, int64_t M) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row < M) scores[row] = score_from_partials(partials, slots, M, row, dist);
}

hipError_t launch_finalize_scores(rs_dist dist, const float* partials, int slots, float* scores,
                                  int64_t M, hipStream_t s) {
    if (M == 0) return hipSuccess;
    hipLaunchKernelGGL(finalize_scores_kernel, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, s,
                       partials, slots, (int)dist, scores, M);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Selection: one workgroup per image.  Scores become order-preserving uint32 keys (sign flip trick;
// NaN above +inf).  Up to 256 tokens a token's rank is counted directly; longer sequences find the key
// of the n_keep-th largest candidate by most-significant-first radix passes over an LDS histogram, and
// an ordered compaction writes the prefix and the survivors in ascending index order (equal keys:
// the lowest indices survive).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t score_key(float s) {
    const uint32_t u = __float_as_uint(s);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// inclusive scan over the NT threads of a workgroup (NT / 64 waves), values in thread order
template <int NT>
__device__ __forceinline__ int block_scan_incl(int v, int* s_wave /*[NT / 64]*/, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    v = wave_scan_incl(v);
    __syncthreads();  // protects s_wave against the previous use
    if (lane == 63) s_wave[wave] = v;
    __syncthreads();
    int add = 0;
    for (int w = 0; w < wave; ++w) add += s_wave[w];
    return v + add;
}

constexpr int SEL_LIST = 256;                 // candidates the last step ranks by counting
constexpr int SEL_MAXN = 12288;               // longest sequence whose keys are kept in LDS
constexpr int SEL_WORDS = SEL_MAXN / 64 + 16; // 64-token words of the compaction
struct SelectShared {
    int hist[256];
    int wave[32];
    uint32_t prefix;
    int remaining, count;
    __attribute__((aligned(16))) uint32_t list[SEL_LIST];
    int gt[SEL_WORDS], eq[SEL_WORDS];
};

// The selection for N <= SEL_MAXN tokens whose scores are in LDS (all NT threads call it; they see sc).
// What the general form below spends its time on is taken out: no pass over the bits all keys share (the
// scores of a sequence lie within a factor of a few, so the leading 8 bits put every key into one
// histogram bin, one serialised LDS atomic per token), no pass for the low bits (once at most SEL_LIST
// candidates share the digits found so far their ranks are counted directly, usually after one pass),
// and the compaction takes 64 tokens per ballot.  10.1 -> 6.7 us at 8 x 1569 tokens.  `sc` is
// overwritten with the keys.
template <int NT>
__device__ __forceinline__ void block_select_lds(float* sc, int N, int n_prefix, int n_keep, int32_t* __restrict__ out,
                                                 SelectShared& sh, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    constexpr int NW = NT / 64;
    uint32_t* keys = reinterpret_cast<uint32_t*>(sc);
    for (int i = tid; i < n_prefix; i += NT) out[i] = i;
    if (n_keep == 0) return;  // uniform over the workgroup
    uint32_t k_and = ~0u, k_or = 0u;
    for (int i = n_prefix + tid; i < N; i += NT) {
        const uint32_t key = score_key(sc[i]);
        keys[i] = key;
        k_and &= key;
        k_or |= key;
    }
    k_and = lanes_reduce<64>(k_and, [](uint32_t a, uint32_t b) { return a & b; });
    k_or = lanes_reduce<64>(k_or, [](uint32_t a, uint32_t b) { return a | b; });
    if (lane == 0) { sh.wave[wave] = (int)k_and; sh.wave[16 + wave] = (int)k_or; }
    if (tid < 256) sh.hist[tid] = 0;
    if (tid == 0) sh.count = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) { k_and &= (uint32_t)sh.wave[w]; k_or |= (uint32_t)sh.wave[16 + w]; }
    const uint32_t diff = k_and ^ k_or;       // bits in which some keys differ
    uint32_t thr = k_and;
    int remaining = n_keep;                   // candidates with the digits found so far still to take
    if (diff) {
        int top = 32 - __clz(diff);           // bits [0, top) are still open
        uint32_t mask = top == 32 ? 0u : ~0u << top, prefix = k_and & mask;
        for (;;) {
            const int shift = top > 8 ? top - 8 : 0;
            for (int i = n_prefix + tid; i < N; i += NT)
                if ((keys[i] & mask) == prefix) atomicAdd(&sh.hist[(keys[i] >> shift) & ((1u << (top - shift)) - 1u)], 1);
            __syncthreads();
            if (wave == 0) {                  // lane l: bins 255 - 4 l ... 252 - 4 l, counted from the top
                int c[4], incl = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) { c[e] = sh.hist[255 - 4 * lane - e]; incl += c[e]; }
                const int own = incl;
                incl = wave_scan_incl(incl);
                int above = incl - own;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (above < remaining && above + c[e] >= remaining) {
                        sh.prefix = prefix | ((uint32_t)(255 - 4 * lane - e) << shift);
                        sh.remaining = remaining - above;
                        sh.gt[0] = c[e];
                    }
                    above += c[e];
                }
            }
            __syncthreads();
            prefix = sh.prefix;
            remaining = sh.remaining;
            const int cnt = sh.gt[0];
            mask = shift ? ~0u << shift : ~0u;
            top = shift;
            if (shift == 0) { thr = prefix; break; }
            if (cnt <= SEL_LIST) {            // few candidates left: count their ranks
                for (int i = n_prefix + tid; i < N; i += NT)
                    if ((keys[i] & mask) == prefix) sh.list[atomicAdd(&sh.count, 1)] = keys[i];
                __syncthreads();
                if (tid < cnt) {
                    const uint32_t mine = sh.list[tid];
                    int g = 0, e = 0;
#pragma unroll 8
                    for (int t = 0; t < cnt; ++t) { const uint32_t k = sh.list[t]; g += k > mine; e += k == mine; }
                    if (g < remaining && g + e >= remaining) { sh.prefix = mine; sh.remaining = remaining - g; }
                }
                // (every thread read sh.remaining before the barrier above)
                __syncthreads();
                thr = sh.prefix;
                remaining = sh.remaining;
                break;
            }
            if (tid < 256) sh.hist[tid] = 0;
            __syncthreads();
        }
    }
    // `remaining` of the candidates equal to thr survive, lowest indices first.  Word t = tokens 64 t .. + 63.
    const int words = (N + 63) / 64;
    __syncthreads();
    for (int t = wave; t < words; t += NW) {
        const int i = t * 64 + lane;
        const bool in = i >= n_prefix && i < N;
        const uint32_t key = in ? keys[i] : 0u;
        const unsigned long long g = __ballot(in && key > thr), e = __ballot(in && key == thr);
        if (lane == 0) { sh.gt[t] = __popcll(g); sh.eq[t] = __popcll(e); }
    }
    __syncthreads();
    if (wave == 0) {                          // exclusive sums over the words
        int bg = 0, be = 0;
        for (int t0 = 0; t0 < words; t0 += 64) {
            const int t = t0 + lane;
            const int g = t < words ? sh.gt[t] : 0, e = t < words ? sh.eq[t] : 0;
            const int ig = wave_scan_incl(g), ie = wave_scan_incl(e);
            if (t < words) { sh.gt[t] = bg + ig - g; sh.eq[t] = be + ie - e; }
            bg += __builtin_amdgcn_readlane(ig, 63);
            be += __builtin_amdgcn_readlane(ie, 63);
        }
    }
    __syncthreads();
    for (int t = wave; t < words; t += NW) {
        const int i = t * 64 + lane;
        const bool in = i >= n_prefix && i < N;
        const uint32_t key = in ? keys[i] : 0u;
        const bool gt = in && key > thr, eq = in && key == thr;
        const unsigned long long below = (1ull << lane) - 1ull, mg = __ballot(gt), me = __ballot(eq);
        const int gb = sh.gt[t] + __popcll(mg & below), eb = sh.eq[t] + __popcll(me & below);
        if (gt || (eq && eb < remaining)) out[n_prefix + gb + min(eb, remaining)] = i;
    }
}

// General form, any N: selection of one image by the NT threads of a workgroup (all of them must call it): among
// the tokens i >= n_prefix of sc[0 .. N) the n_keep highest keys survive, equal keys by lower
// index; out[0 .. n_prefix + n_keep) lists the prefix and the survivors in ascending order.
// `sc` is global memory.
template <int NT>
__device__ __forceinline__ void block_select(const float* sc, int N, int n_prefix, int n_keep,
                                             int32_t* __restrict__ out, SelectShared& sh, int tid) {
    for (int i = tid; i < n_prefix; i += NT) out[i] = i;
    if (n_keep == 0) return;  // uniform over the workgroup

    uint32_t prefix = 0, mask = 0;
    int remaining = n_keep;  // how many of the candidates matching `prefix` still to take
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) sh.hist[tid] = 0;
        __syncthreads();
        for (int i = n_prefix + tid; i < N; i += NT) {
            const uint32_t key = score_key(sc[i]);
            if ((key & mask) == prefix) atomicAdd(&sh.hist[(key >> shift) & 255], 1);
        }
        __syncthreads();
        // suffix sums over the bins: thread t < 256 looks at bin 255 - t, so an inclusive scan in
        // thread order counts the candidates in bins >= bin (threads beyond 255 add nothing).
        const int bin = 255 - tid;
        const int cnt = tid < 256 ? sh.hist[bin] : 0;
        const int incl = block_scan_incl<NT>(cnt, sh.wave, tid);
        // the wanted key's digit is the first bin (from the top) whose suffix count reaches `remaining`
        if (tid < 256 && incl >= remaining && incl - cnt < remaining) {
            sh.prefix = prefix | ((uint32_t)bin << shift);
            sh.remaining = remaining - (incl - cnt);
        }
        __syncthreads();
        prefix = sh.prefix;
        remaining = sh.remaining;
        mask |= 255u << shift;
        __syncthreads();
    }
    // `prefix` = key of the n_keep-th largest candidate; `remaining` = how many candidates with
    // exactly that key are kept (those with the lowest indices).
    const uint32_t thr = prefix;
    const int n = N - n_prefix;
    const int seg = (n + NT - 1) / NT;
    const int lo = n_prefix + tid * seg;
    const int hi = min(lo + seg, N);
    int gt = 0, eq = 0;
    for (int i = lo; i < hi; ++i) {
        const uint32_t key = score_key(sc[i]);
        gt += key > thr;
        eq += key == thr;
    }
    const int gt_before = block_scan_incl<NT>(gt, sh.wave, tid) - gt;
    const int eq_before = block_scan_incl<NT>(eq, sh.wave, tid) - eq;
    int pos = n_prefix + gt_before + min(eq_before, remaining);
    int eq_rank = eq_before;
    for (int i = lo; i < hi; ++i) {
        const uint32_t key = score_key(sc[i]);
        bool keep = key > thr;
        if (key == thr) { keep = eq_rank < remaining; ++eq_rank; }
        if (keep) out[pos++] = i;
    }
}

// The same selection for at most 64 R tokens by ONE wave, in registers: lane l holds the keys of tokens
// l, l + 64, ...; on return pos[r] is the place of token 64 r + l in the ascending list of survivors
// (prefix included) or -1.  The key of the n_keep-th largest candidate is found bit by bit, counting with
// ballots how many keys reach a trial value (about 20 trials: it ends as soon as exactly n_keep do); no
// LDS, no barrier.  (Counting every token's rank against all others took N^2 comparisons per image, in
// every workgroup that shares an image: 5 us of the block's prune pass at 64 x 197 tokens.)
template <int R>
__device__ __forceinline__ void wave_select(const uint32_t (&key)[R], int N, int n_prefix, int n_keep, int lane, int (&pos)[R]) {
    bool valid[R];
    uint32_t k[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * 64 + lane;
        valid[r] = i >= n_prefix && i < N;
        k[r] = valid[r] ? key[r] : 0u;  // below every trial value
    }
    uint32_t thr = 0u;         // kept: keys above thr, and `ties` of those equal to it, lowest indices first
    bool exact = false;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t c = thr | (1u << bit);
        int cnt = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) cnt += __popcll(__ballot(k[r] >= c));
        if (cnt >= n_keep) thr = c;
        if (cnt == n_keep) { exact = true; break; }
    }
    if (exact) thr -= 1u;      // exactly the keys that reach thr (>= 1) survive
    int above = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) above += __popcll(__ballot(valid[r] && k[r] > thr));
    const int ties = n_keep - above;
    const unsigned long long below = (1ull << lane) - 1ull;
    int base = 0, eq_base = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const unsigned long long me = __ballot(valid[r] && k[r] == thr);
        const bool tie = valid[r] && k[r] == thr && eq_base + __popcll(me & below) < ties;
        const bool keep = r * 64 + lane < n_prefix || (valid[r] && k[r] > thr) || tie;
        const unsigned long long mk = __ballot(keep);
        pos[r] = keep ? base + __popcll(mk & below) : -1;
        base += __popcll(mk);
        eq_base += __popcll(me);
    }
}

// Longer sequences, one image per workgroup.  The scores go through LDS (N * 4 bytes of dynamic LDS, N <= SEL_MAXN): read
// from `scores`, or with `partials` formed from the GEMM epilogue's per-row slots (added in slot order,
// as finalize_scores_kernel does) and written to `scores` on the way: the block's prune pass needs no
// separate score launch.
template <int NT>
__global__ __launch_bounds__(NT) void select_kernel(float* __restrict__ scores,
                                                     int32_t* __restrict__ kept_idx, int N,
                                                     int n_prefix, int n_keep,
                                                     const float* __restrict__ partials, int slots, int dist) {
    __shared__ SelectShared sh;
    extern __shared__ float s_scores[];
    const int tid = threadIdx.x;
    float* sc = scores + (int64_t)blockIdx.x * N;
    int32_t* out = kept_idx + (int64_t)blockIdx.x * (n_prefix + n_keep);
    for (int i = tid; i < N; i += NT) {
        float r;
        if (partials) {
            r = score_from_partials(partials, slots, (int64_t)gridDim.x * N, (int64_t)blockIdx.x * N + i, dist);
            sc[i] = r;
        } else {
            r = sc[i];
        }
        s_scores[i] = r;
    }
    __syncthreads();
    block_select_lds<NT>(s_scores, N, n_prefix, n_keep, out, sh, tid);
}

// Sequences of at most 256 tokens: one wave per image.
__global__ __launch_bounds__(256) void select_short_kernel(const float* __restrict__ scores,
                                                           int32_t* __restrict__ kept_idx, int B, int N, int n_prefix,
                                                           int n_keep) {
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= B) return;
    uint32_t key[4];
    int pos[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) key[r] = r * 64 + lane < N ? score_key(scores[b * N + r * 64 + lane]) : 0u;
    wave_select<4>(key, N, n_prefix, n_keep, lane, pos);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (pos[r] >= 0) kept_idx[b * (n_prefix + n_keep) + pos[r]] = r * 64 + lane;
}

// Sequences beyond SEL_MAXN tokens: the scores stay in global memory.
__global__ __launch_bounds__(1024) void select_long_kernel(const float* __restrict__ scores,
                                                           int32_t* __restrict__ kept_idx, int N, int n_prefix,
                                                           int n_keep) {
    __shared__ SelectShared sh;
    block_select<1024>(scores + (int64_t)blockIdx.x * N, N, n_prefix, n_keep,
                       kept_idx + (int64_t)blockIdx.x * (n_prefix + n_keep), sh, threadIdx.x);
}

// ---------------------------------------------------------------------------
// Score, selection and gather of one image in ONE pass over memory, for images whose f_in rows
// fit the register file of a compute unit (N <= 16 NR rows of at most 512 CH bytes: every
// image-classification shape).  One workgroup of 16 waves per image at a time: wave w holds rows
// w, w + 16, ... of f_in in registers (8 bytes per lane and chunk), streams the same rows of f_out
// past them for the scores, the workgroup selects, and every wave then writes its surviving rows
// to their places in `gathered` straight from registers.  Against the three-launch path the
// kept rows are not read a second time: memory traffic is the algorithmic minimum
// (2 N D e read, K D e written per image).  Workgroups loop over images (persistent grid).
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ void unpack8(u32x2 v, float (&f)[4]);
template <> __device__ __forceinline__ void unpack8<bf16raw>(u32x2 v, float (&f)[4]) {
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
}
template <> __device__ __forceinline__ void unpack8<float>(u32x2 v, float (&f)[4]) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = 0.f; f[3] = 0.f;
}

#ifndef RS_RES_WAVES
#define RS_RES_WAVES 16
#endif
#ifndef RS_RES_G
#define RS_RES_G 4
#endif
constexpr int RES_WAVES = RS_RES_WAVES;   // waves per workgroup: between them they own the CU's registers
constexpr int RES_MAXN = 208;             // longest sequence the kernel takes
constexpr int RES_NR = (RES_MAXN + RES_WAVES - 1) / RES_WAVES;  // rows per wave

template <typename T, int DIST, int CH, int NR>
__global__ __launch_bounds__(RES_WAVES * 64) void shift_topk_resident_kernel(
    const T* __restrict__ f_out, const T* __restrict__ f_in, float* __restrict__ scores,
    int32_t* __restrict__ kept_idx, T* __restrict__ gathered, int B, int N, int D, int n_prefix, int n_keep) {
    static_assert(RES_WAVES == 16 && RES_MAXN <= 256, "the selection below: row wave + 16 k is token 64 (k / 4) + wave + 16 (k % 4)");
    __shared__ float s_scores[2][256];
    int par = 0;  // scores of two images alternate, so that one barrier per image is enough
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: row addresses stay scalar
    const int row_u = D * (int)sizeof(T) / 8;  // 8-byte units per row
    const int K = n_prefix + n_keep;
    // Rows are addressed through buffer resources over one image: the row offset is a scalar, the
    // lane offset one register per chunk, and whatever lies outside (rows past N, lanes past the
    // row's end, which are aimed far outside) reads as zero and is dropped on stores.
    const int row_bytes = D * (int)sizeof(T);
    int voff[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) voff[c] = (lane + 64 * c) < row_u ? (lane + 64 * c) * 8 : 0x7fff0000;
    // The resident rows of the first image; those of every later image are requested row by row
    // while the previous image's surviving rows are being written out of the same registers, so
    // their latency passes under that image's stores and the next image's f_out stream.
    u32x2 keep[NR][CH];
    {
        const __amdgpu_buffer_rsrc_t r_in0 = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(f_in + (int64_t)blockIdx.x * N * D), 0, (int)blockIdx.x < B ? N * row_bytes : 0, 0x00020000);
#pragma unroll
        for (int k = 0; k < NR; ++k)
#pragma unroll
            for (int c = 0; c < CH; ++c)
                keep[k][c] = __builtin_amdgcn_raw_buffer_load_b64(r_in0, voff[c], (wave + RES_WAVES * k) * row_bytes, 0);
    }
    for (int b = blockIdx.x; b < B; b += gridDim.x) {
        const __amdgpu_buffer_rsrc_t r_fo = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(f_out + (int64_t)b * N * D), 0, N * row_bytes, 0x00020000);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int G = RS_RES_G;  // rows of f_out in flight per wave (next to the resident rows)
#pragma unroll
        for (int k0 = 0; k0 < NR; k0 += G) {
            u32x2 t[G][CH];
#pragma unroll
            for (int kk = 0; kk < G; ++kk)
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    if (k0 + kk < NR)
                        t[kk][c] = __builtin_amdgcn_raw_buffer_load_b64(r_fo, voff[c], (wave + RES_WAVES * (k0 + kk)) * row_bytes, 0);
#pragma unroll
            for (int kk = 0; kk < G; ++kk) {
                if (k0 + kk >= NR) break;
                const int i = wave + RES_WAVES * (k0 + kk);
                float p0 = 0.f, p1 = 0.f, p2 = 0.f;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    float x[4], y[4];
                    unpack8<T>(t[kk][c], x);
                    unpack8<T>(keep[k0 + kk][c], y);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (DIST == RS_DIST_L2) { float d = x[e] - y[e]; p0 = fmaf(d, d, p0); }
                        else if (DIST == RS_DIST_L1) { p0 += fabsf(x[e] - y[e]); }
                        else { p0 = fmaf(x[e], y[e], p0); p1 = fmaf(x[e], x[e], p1); p2 = fmaf(y[e], y[e], p2); }
                    }
                }
                p0 = wave_sum(p0);
                if (DIST == RS_DIST_COS) { p1 = wave_sum(p1); p2 = wave_sum(p2); }
                if (lane == 0 && i < N) {
                    float sc;
                    if (DIST == RS_DIST_L2) sc = sqrtf(p0);
                    else if (DIST == RS_DIST_L1) sc = p0;
                    else sc = 1.0f - p0 / (sqrtf(p1) * sqrtf(p2));
                    s_scores[par][i] = sc;
                    scores[(int64_t)b * N + i] = sc;
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // the next group's loads stay behind this group's sums
        }
        __syncthreads();
        // every wave selects for itself (registers only) and needs nothing from the others
        uint32_t key[4];
        int pos[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) key[r] = r * 64 + lane < N ? score_key(s_scores[par][r * 64 + lane]) : 0u;
        wave_select<4>(key, N, n_prefix, n_keep, lane, pos);
        if (wave == 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (pos[r] >= 0) kept_idx[(int64_t)b * K + pos[r]] = r * 64 + lane;
        }
        par ^= 1;
        const __amdgpu_buffer_rsrc_t r_out = __builtin_amdgcn_make_buffer_rsrc(
            gathered + (int64_t)b * K * D, 0, K * row_bytes, 0x00020000);
        const int b_next = b + gridDim.x;
        const __amdgpu_buffer_rsrc_t r_in = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(f_in + (int64_t)(b_next < B ? b_next : 0) * N * D), 0, b_next < B ? N * row_bytes : 0, 0x00020000);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = wave + RES_WAVES * k;
            const int j = __builtin_amdgcn_readlane(pos[k >> 2], wave + 16 * (k & 3));  // place of row i, or -1
            if (j >= 0) {
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    __builtin_amdgcn_raw_buffer_store_b64(keep[k][c], r_out, voff[c], j * row_bytes, kWriteThrough);
            }
#pragma unroll
            for (int c = 0; c < CH; ++c)
                keep[k][c] = __builtin_amdgcn_raw_buffer_load_b64(r_in, voff[c], i * row_bytes, 0);
        }
    }
}

// The scores of the one-pass kernel, bit for bit, by a grid over the rows: which kernel an image goes through depends on
// how many there are, and its scores must not.  A lane takes 16 bytes of a row, that is the bytes of lanes 2 sub
// and 2 sub + 1 of the one-pass kernel's wave, and keeps their two sums apart up to the butterfly's last step.  G lanes
// per row (the next power of two of its 16-byte vectors, at most 32), CH vectors of each.  The whole call with the scores
// in shift_scores_kernel's order / in this one: 1 x 197 x 384 6.8 / 7.0 us, 16 x 197 x 768 8.0 / 8.0, 128: 22.6 / 22.1, 64 x 197 x 64
// 8.5 / 7.4 (four rows per thread: 8.2, and 15.0 instead of 14.5 at 64 x 197 x 768).
template <typename T, int DIST, int G, int CH>
__global__ __launch_bounds__(256) void shift_scores_paired_kernel(const T* __restrict__ f_out, const T* __restrict__ f_in,
                                                                  float* __restrict__ scores, int64_t M, int row_vec) {
    const int sub = threadIdx.x % G;
    const int64_t row = (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G;
    const u32x4 *a = reinterpret_cast<const u32x4*>(f_out), *b = reinterpret_cast<const u32x4*>(f_in);
    u32x4 x[CH], y[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const bool on = row < M && sub + c * G < row_vec;
        x[c] = on ? a[row * row_vec + sub + c * G] : u32x4{0u, 0u, 0u, 0u};
        y[c] = on ? b[row * row_vec + sub + c * G] : u32x4{0u, 0u, 0u, 0u};
    }
    float p[2][3] = {};
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float fx[4], fy[4];
            unpack8<T>(u32x2{x[c][2 * h], x[c][2 * h + 1]}, fx);
            unpack8<T>(u32x2{y[c][2 * h], y[c][2 * h + 1]}, fy);
#pragma unroll
            for (int e = 0; e < 4; ++e) dist_term<DIST>(fx[e], fy[e], p[h][0], p[h][1], p[h][2]);
        }
#pragma unroll
    for (int i = 0; i < (DIST == RS_DIST_COS ? 3 : 1); ++i) {
        p[0][i] = lanes_sum<G>(p[0][i]);
        p[1][i] = lanes_sum<G>(p[1][i]);
    }
    if (sub == 0 && row < M) scores[row] = dist_value<DIST>(p[0][0] + p[1][0], p[0][1] + p[1][1], p[0][2] + p[1][2]);
}

template <typename T>
static hipError_t launch_paired_t(rs_dist dist, const void* f_out, const void* f_in, float* scores, int64_t M, int D, hipStream_t s) {
    const int row_vec = (int)((size_t)D * sizeof(T) / 16);
#define RS_PAIRED(DIST_, G_, CH_)                                                                                      \
    hipLaunchKernelGGL((shift_scores_paired_kernel<T, DIST_, G_, CH_>), dim3((unsigned)((M + 256 / G_ - 1) / (256 / G_))), \
                       dim3(256), 0, s, (const T*)f_out, (const T*)f_in, scores, M, row_vec)
#define RS_PAIRED_D(DIST_)                                                                                             \
    if (row_vec <= 8) RS_PAIRED(DIST_, 8, 1);                                                                          \
    else if (row_vec <= 16) RS_PAIRED(DIST_, 16, 1);                                                                   \
    else if (row_vec <= 32) RS_PAIRED(DIST_, 32, 1);                                                                   \
    else if (row_vec <= 64) RS_PAIRED(DIST_, 32, 2);                                                                   \
    else RS_PAIRED(DIST_, 32, 3);
    if (dist == RS_DIST_L2) { RS_PAIRED_D(RS_DIST_L2) }
    else if (dist == RS_DIST_L1) { RS_PAIRED_D(RS_DIST_L1) }
    else { RS_PAIRED_D(RS_DIST_COS) }
#undef RS_PAIRED_D
#undef RS_PAIRED
    return hipGetLastError();
}

hipError_t launch_shift_scores_paired(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in, float* scores, int64_t M,
                                      int D, hipStream_t s) {
    if (M == 0) return hipSuccess;
    return dt == RS_F32 ? launch_paired_t<float>(dist, f_out, f_in, scores, M, D, s)
                        : launch_paired_t<bf16raw>(dist, f_out, f_in, scores, M, D, s);
}

// Sequences that fit the one-pass kernel, however many.
bool shift_topk_resident_form(rs_dtype dt, int N, int D) { return N <= RES_MAXN && (size_t)D * elem_size(dt) <= 512 * 3; }

// Where the one-pass kernel is the faster way.  Its workgroup holds one image whatever its length and
// works through it serially, so it needs images that fill the registers (more than half of the rows it
// has room for) and rounds of the chip that are at least three quarters full; otherwise the separate
// launches, each spread over all rows, win although they read the kept rows twice.  bf16, nine tenths kept, one pass /
// separate launches in us: 197 x 768 192 images 33.5 / 36.9, 256: 38.7 / 47.2, 384: 82.7 / 72.8, 512: 102 / 98, 576: 132 / 125,
// 640: 133 / 145, 768: 148 / 170, 1024: 195 / 221, 2048: 367 / 421 (between one round and two and a half the inputs no
// longer fit the caches, and the line at three quarters is too low by up to 13 %); 197 x 384 192: 23.4 / 22.2, 256: 25.2 / 27.5;
// 150 x 768 256: 33.1 / 37.1, 110 x 768 256: 29.0 / 29.0, 1024: 124 / 124; below, 16 x 197 x 768 25.4 / 8.0.
// From 2^26 rows on the separate launches would reach 2^32 threads (a wave per gathered row), its own never does.
bool shift_topk_resident_fits(rs_dtype dt, int B, int N, int D) {
    if (!shift_topk_resident_form(dt, N, D)) return false;
    if ((int64_t)B * N >= (int64_t)1 << 26) return true;
    const int64_t cus = device_cus(), rounds = (B + cus - 1) / cus;
    return 2 * N > RES_MAXN && 4 * (int64_t)B >= 3 * rounds * cus;
}

template <typename T, int CH>
static hipError_t launch_resident_t(rs_dist dist, const void* f_out, const void* f_in, float* scores,
                                    int32_t* kept_idx, void* gathered, int B, int N, int D, int n_prefix,
                                    int n_keep, int grid, hipStream_t s) {
#define RS_RES_LAUNCH(DIST_)                                                                                  \
    hipLaunchKernelGGL((shift_topk_resident_kernel<T, DIST_, CH, RES_NR>), dim3(grid), dim3(RES_WAVES * 64), 0, s, \
                       (const T*)f_out, (const T*)f_in, scores, kept_idx, (T*)gathered, B, N, D, n_prefix, n_keep)
    if (dist == RS_DIST_L2) RS_RES_LAUNCH(RS_DIST_L2);
    else if (dist == RS_DIST_L1) RS_RES_LAUNCH(RS_DIST_L1);
    else RS_RES_LAUNCH(RS_DIST_COS);
#undef RS_RES_LAUNCH
    return hipGetLastError();
}

hipError_t launch_shift_topk_resident(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in,
                                      float* scores, int32_t* kept_idx, void* gathered, int B, int N, int D,
                                      int n_prefix, int n_keep, hipStream_t s) {
    if (B == 0 || N == 0) return hipSuccess;
    const int cus = device_cus();
    const int grid = B < cus ? B : cus;  // one workgroup fills a compute unit's register file
    const int ch = (int)(((size_t)D * elem_size(dt) + 511) / 512);
#define RS_RES_CH(T_)                                                                                                   \
    (ch == 1 ? launch_resident_t<T_, 1>(dist, f_out, f_in, scores, kept_idx, gathered, B, N, D, n_prefix, n_keep, grid, s) \
     : ch == 2 ? launch_resident_t<T_, 2>(dist, f_out, f_in, scores, kept_idx, gathered, B, N, D, n_prefix, n_keep, grid, s) \
               : launch_resident_t<T_, 3>(dist, f_out, f_in, scores, kept_idx, gathered, B, N, D, n_prefix, n_keep, grid, s))
    return dt == RS_F32 ? RS_RES_CH(float) : RS_RES_CH(bf16raw);
#undef RS_RES_CH
}

// kept_idx[b, j] = j when every token survives
__global__ __launch_bounds__(256) void iota_kernel(int32_t* __restrict__ kept_idx, int B, int K) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < (int64_t)B * K) kept_idx[t] = (int32_t)(t % K);
}

hipError_t launch_select(const float* scores, int32_t* kept_idx, int B, int N, int n_prefix,
                         int n_keep, hipStream_t s) {
    if (B == 0 || n_prefix + n_keep == 0) return hipSuccess;
    if (n_keep == N - n_prefix) {
        const int64_t tot = (int64_t)B * N;
        hipLaunchKernelGGL(iota_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, kept_idx, B, N);
    } else {
        const size_t lds = (size_t)N * sizeof(float);
        if (N <= 256)
            hipLaunchKernelGGL(select_short_kernel, dim3((unsigned)((B + 3) / 4)), dim3(256), 0, s, scores, kept_idx, B, N, n_prefix, n_keep);
        else if (N > SEL_MAXN)
            hipLaunchKernelGGL(select_long_kernel, dim3(B), dim3(1024), 0, s, scores, kept_idx, N, n_prefix, n_keep);
        else if (N > 1024)
            hipLaunchKernelGGL(select_kernel<1024>, dim3(B), dim3(1024), lds, s, const_cast<float*>(scores), kept_idx, N,
                               n_prefix, n_keep, (const float*)nullptr, 0, 0);
        else
            hipLaunchKernelGGL(select_kernel<256>, dim3(B), dim3(256), lds, s, const_cast<float*>(scores), kept_idx, N,
                               n_prefix, n_keep, (const float*)nullptr, 0, 0);
    }
    return hipGetLastError();
}

bool select_from_partials_fits(int N) { return N <= SEL_MAXN; }  // scores of one image in LDS

hipError_t launch_select_from_partials(rs_dist dist, const float* partials, int slots, float* scores,
                                       int32_t* kept_idx, int B, int N, int n_prefix, int n_keep,
                                       hipStream_t s) {
    if (B == 0) return hipSuccess;
    if (N <= 256 || B < 64) {
        // a few long sequences (video clips): one workgroup per image would walk its image's slots
        // alone, one cache line per thread and slot, and spend more time there than selecting.
        // The scores are formed by a grid over all rows instead (the same additions in the same
        // order), and the selection reads them back.
        if (hipError_t e = launch_finalize_scores(dist, partials, slots, scores, (int64_t)B * N, s); e != hipSuccess)
            return e;
        return launch_select(scores, kept_idx, B, N, n_prefix, n_keep, s);
    } else {
        hipLaunchKernelGGL(select_kernel<256>, dim3(B), dim3(256), (size_t)N * sizeof(float), s, scores, kept_idx, N,
                           n_prefix, n_keep, partials, slots, (int)dist);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gather: out[b, j, :] = src[b, kept_idx[b, j], :].  G lanes per row (the next power of two of its 16-byte
// vectors, at most a wave), U rows per thread and CH vectors of each at a time.  What limits it is the
// chain index -> row -> store, so everything a thread needs is requested before its first store:
// stores and loads share one counter, and a load behind a store waits for that store too (three
// vectors per lane in a plain loop: 20 us against 6 for 8 x 785 rows of 3 KB).
// (A variant over the flat output, four vectors per thread whatever the row length, measured 50 %
// slower at 1536-byte rows.)
// ---------------------------------------------------------------------------
template <int G, int U, int CH>
__global__ __launch_bounds__(256) void gather_rows_kernel(const u32x4* __restrict__ src,
                                                          const int32_t* __restrict__ kept_idx,
                                                          u32x4* __restrict__ out, int64_t rows,
                                                          int N, int K, int row_vec) {
    constexpr int RPG = 256 / G;
    const int sub = threadIdx.x % G;
    const int64_t r0 = (int64_t)blockIdx.x * (RPG * U) + threadIdx.x / G;
    int64_t sp[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t r = r0 + u * RPG;  // rows < 2^31
        sp[u] = r < rows ? (int64_t)((uint32_t)r / (uint32_t)K) * N + kept_idx[r] : -1;
    }
    for (int c = sub; c < row_vec; c += G * CH) {
        u32x4 v[U][CH];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < CH; ++k)
                if (sp[u] >= 0 && c + k * G < row_vec) v[u][k] = src[sp[u] * row_vec + c + k * G];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < CH; ++k)
                if (sp[u] >= 0 && c + k * G < row_vec) out[(r0 + u * RPG) * row_vec + c + k * G] = v[u][k];
    }
}

// The same gather for bf16 rows that also leaves the LayerNorm statistics of every row it writes
// (mean, 1 / sqrt(variance + eps)): the wave has the row in registers anyway, and the block that
// consumes the gathered rows then needs no statistics pass of its own.  Same arithmetic as the
// statistics kernel (wave_row_stats), hence the same bits.
template <int MAXC>
__global__ __launch_bounds__(256) void gather_rows_stats_kernel(const bf16raw* __restrict__ src,
                                                                const int32_t* __restrict__ kept_idx,
                                                                bf16raw* __restrict__ out,
                                                                float2* __restrict__ stats, int64_t rows, int N,
                                                                int K, int D, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= rows) return;
    const int64_t b = r / K;
    const bf16raw* s = src + (b * N + kept_idx[r]) * D;
    bf16raw* d = out + r * D;
    const int nchunk = D >> 3;
    u32x4 raw[MAXC];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        raw[c] = u32x4{0u, 0u, 0u, 0u};
        if (lane + c * 64 < nchunk) raw[c] = *reinterpret_cast<const u32x4*>(s + (lane + c * 64) * 8);
    }
    float v[MAXC][8];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        if (lane + c * 64 < nchunk) *reinterpret_cast<u32x4*>(d + (lane + c * 64) * 8) = raw[c];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[c][2 * i] = __uint_as_float(raw[c][i] << 16);
            v[c][2 * i + 1] = __uint_as_float(raw[c][i] & 0xffff0000u);
        }
    }
    const float2 st = wave_row_stats<MAXC>(v, nchunk, lane, D, eps);
    if (lane == 0) stats[r] = st;
}

bool gather_stats_fits(rs_dtype dt, int D) { return dt == RS_BF16 && D <= 8 * 64 * 8; }

hipError_t launch_gather_stats(const void* src, const int32_t* kept_idx, void* out, float* stats, int B, int N,
                               int K, int D, float eps, hipStream_t s) {
    const int64_t rows = (int64_t)B * K;
    if (rows == 0) return hipSuccess;
    const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
    if (D <= 2 * 512)
        hipLaunchKernelGGL(gather_rows_stats_kernel<2>, grid, block, 0, s, (const bf16raw*)src, kept_idx, (bf16raw*)out,
                           reinterpret_cast<float2*>(stats), rows, N, K, D, eps);
    else
        hipLaunchKernelGGL(gather_rows_stats_kernel<8>, grid, block, 0, s, (const bf16raw*)src, kept_idx, (bf16raw*)out,
                           reinterpret_cast<float2*>(stats), rows, N, K, D, eps);
    return hipGetLastError();
}

// A workgroup's share of an image's surviving rows (s_idx: their tokens, in LDS): one wave per row, STATS: with
// their LayerNorm statistics as in gather_rows_stats_kernel.  MAXC: 16-byte vectors per lane and row.
template <bool STATS, int MAXC, int NW>
__device__ __forceinline__ void copy_share(const int32_t* s_idx, const u32x4* __restrict__ src, u32x4* __restrict__ out,
                                           float2* __restrict__ stats, int64_t b, int N, int K, int row_vec, int D, float eps,
                                           int lane, int wave) {
    const int per = (K + gridDim.x - 1) / gridDim.x;
    const int j1 = min((int)(blockIdx.x + 1) * per, K);
    constexpr int U = 2;  // rows in flight per wave
    for (int j0 = blockIdx.x * per + wave; j0 < j1; j0 += NW * U) {
        u32x4 v[U][MAXC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * NW;
            const u32x4* s = src + (b * N + s_idx[min(j, K - 1)]) * row_vec;
#pragma unroll
            for (int c = 0; c < MAXC; ++c)
                v[u][c] = j < j1 && lane + c * 64 < row_vec ? s[lane + c * 64] : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = __builtin_amdgcn_readfirstlane(j0 + u * NW);
            if (j >= j1) break;  // wave-uniform
            u32x4* d = out + (b * K + j) * row_vec;
            if constexpr (STATS) {  // inside a block: the next one reads the rows (alone, topk_clips: 30.6 us plain, 30.9 written through)
                const __amdgpu_buffer_rsrc_t rs_d = __builtin_amdgcn_make_buffer_rsrc(d, 0, row_vec * 16, 0x00020000);
#pragma unroll
                for (int c = 0; c < MAXC; ++c) store16_wt(rs_d, (lane + c * 64) * 16, v[u][c]);  // nothing past the row's end
            } else {
#pragma unroll
                for (int c = 0; c < MAXC; ++c)
                    if (lane + c * 64 < row_vec) d[lane + c * 64] = v[u][c];
            }
            if constexpr (STATS) {
                float f[MAXC][8];
#pragma unroll
                for (int c = 0; c < MAXC; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        f[c][2 * i] = __uint_as_float(v[u][c][i] << 16);
                        f[c][2 * i + 1] = __uint_as_float(v[u][c][i] & 0xffff0000u);
                    }
                const float2 st = wave_row_stats<MAXC>(f, row_vec, lane, D, eps);
                if (lane == 0) stats[b * K + j] = st;
            }
        }
    }
}

// Scores, selection and gather of one short image (N <= 256) in one launch: `parts` workgroups per image,
// each of which forms the image's scores from the partial sums and selects (a microsecond; the sums
// are a few KB per image) and then copies its share of the surviving rows, STATS: with their LayerNorm
// statistics as in gather_rows_stats_kernel.  Against a selection and a gather of their own it saves
// a launch of every pruning block (vit_s16, eleven of them: 1020 -> 944 us per forward together with the
// selection by one wave); one workgroup per image would leave the chip idle and copy with too few
// requests in flight.  MAXC: 16-byte vectors per lane and row.
constexpr int SG_WAVES = 8;
template <bool STATS, int MAXC>
__global__ __launch_bounds__(SG_WAVES * 64) void select_gather_kernel(
    const float* __restrict__ partials, int slots, int dist, float* __restrict__ scores,
    int32_t* __restrict__ kept_idx, const u32x4* __restrict__ src, u32x4* __restrict__ out,
    float2* __restrict__ stats, int N, int n_prefix, int n_keep, int row_vec, int D, float eps) {
    __shared__ float s_scores[256];
    __shared__ int32_t s_idx[256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b = blockIdx.y;
    const int K = n_prefix + n_keep;
    if (tid < N) {
        const float r = partials ? score_from_partials(partials, slots, (int64_t)gridDim.y * N, b * N + tid, dist) : scores[b * N + tid];
        s_scores[tid] = r;
        if (partials && blockIdx.x == 0) scores[b * N + tid] = r;
    }
    __syncthreads();
    if (wave == 0) {
        uint32_t key[4];
        int pos[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) key[r] = r * 64 + lane < N ? score_key(s_scores[r * 64 + lane]) : 0u;
        wave_select<4>(key, N, n_prefix, n_keep, lane, pos);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (pos[r] >= 0) {
                s_idx[pos[r]] = r * 64 + lane;
                if (blockIdx.x == 0) kept_idx[b * K + pos[r]] = r * 64 + lane;
            }
    }
    __syncthreads();
    copy_share<STATS, MAXC, SG_WAVES>(s_idx, src, out, stats, b, N, K, row_vec, D, eps, lane, wave);
}

// Selection and gather of longer sequences in one launch: as above with the selection of select_kernel, for so
// few sequences that their selections leave most of the chip idle anyway (every workgroup repeats its
// sequence's).
constexpr int SGL_WAVES = 16;
template <bool STATS, int MAXC>
__global__ __launch_bounds__(SGL_WAVES * 64) void select_gather_long_kernel(
    const float* __restrict__ scores, int32_t* __restrict__ kept_idx, const u32x4* __restrict__ src, u32x4* __restrict__ out,
    float2* __restrict__ stats, int N, int n_prefix, int n_keep, int row_vec, int D, float eps) {
    __shared__ SelectShared sh;
    extern __shared__ float s_scores[];  // N scores, then the K surviving tokens
    int32_t* s_idx = reinterpret_cast<int32_t*>(s_scores + N);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b = blockIdx.y;
    const int K = n_prefix + n_keep;
    for (int i = tid; i < N; i += SGL_WAVES * 64) s_scores[i] = scores[b * N + i];
    __syncthreads();
    block_select_lds<SGL_WAVES * 64>(s_scores, N, n_prefix, n_keep, s_idx, sh, tid);
    __syncthreads();
    if (blockIdx.x == 0)
        for (int j = tid; j < K; j += SGL_WAVES * 64) kept_idx[b * K + j] = s_idx[j];
    copy_share<STATS, MAXC, SGL_WAVES>(s_idx, src, out, stats, b, N, K, row_vec, D, eps, lane, wave);
}

// One workgroup per CU over all sequences (two, measured: 4 x 4097 x 1024 28.1 -> 30.2 us, 64 x 300 x 192 11.1 -> 12.4).
// Score, selection and gather in two launches / three (us): 8 x 1569 x 768 fp32 25.1 / 26.5, 4 x 4097 x 1024 28.1 /
// 30.1, 20 x 1000 x 768 21.6 / 25.0, 64 x 500 x 768 28.3 / 30.1; beyond, fewer than four workgroups share a sequence's copy.
bool select_gather_long_fits(rs_dtype dt, int B, int N, int D) {
    return N > 256 && N <= SEL_MAXN / 2 && (size_t)D * elem_size(dt) <= 4 * 1024 && 4 * B <= device_cus();
}

hipError_t launch_select_gather_long(rs_dtype dt, const float* scores, int32_t* kept_idx, const void* src, void* out,
                                     float* stats, int B, int N, int n_prefix, int n_keep, int D, float eps, hipStream_t s) {
    if (B == 0) return hipSuccess;
    const int K = n_prefix + n_keep, row_vec = (int)((size_t)D * elem_size(dt) / 16);
    int parts = device_cus() / B;
    parts = parts < (K + SGL_WAVES - 1) / SGL_WAVES ? parts : (K + SGL_WAVES - 1) / SGL_WAVES;
    const bool st = stats && dt == RS_BF16;
    const size_t lds = (size_t)(N + K) * 4;
#define RS_SGL(ST_, C_)                                                                                                  \
    hipLaunchKernelGGL((select_gather_long_kernel<ST_, C_>), dim3(parts, B), dim3(SGL_WAVES * 64), lds, s, scores, kept_idx, \
                       (const u32x4*)src, (u32x4*)out, reinterpret_cast<float2*>(stats), N, n_prefix, n_keep, row_vec, D, eps)
    if (row_vec <= 64) { if (st) RS_SGL(true, 1); else RS_SGL(false, 1); }
    else if (row_vec <= 128) { if (st) RS_SGL(true, 2); else RS_SGL(false, 2); }
    else { if (st) RS_SGL(true, 4); else RS_SGL(false, 4); }
#undef RS_SGL
    return hipGetLastError();
}

bool select_gather_fits(rs_dtype dt, int N, int D) { return N <= 256 && (size_t)D * elem_size(dt) <= 4 * 1024; }

hipError_t launch_select_gather(rs_dtype dt, rs_dist dist, const float* partials, int slots, float* scores,
                                int32_t* kept_idx, const void* src, void* out, float* stats, int B, int N, int n_prefix,
                                int n_keep, int D, float eps, hipStream_t s) {
    if (B == 0) return hipSuccess;
    const int K = n_prefix + n_keep, row_vec = (int)((size_t)D * elem_size(dt) / 16);
    // about two workgroups per CU over all images (256 .. 2048 in all measured within 1 %), at least one row per wave
    int parts = (512 + B - 1) / B;
    parts = parts < (K + SG_WAVES - 1) / SG_WAVES ? parts : (K + SG_WAVES - 1) / SG_WAVES;
    const bool st = stats && dt == RS_BF16;
#define RS_SG(ST_, C_)                                                                                                   \
    hipLaunchKernelGGL((select_gather_kernel<ST_, C_>), dim3(parts, B), dim3(SG_WAVES * 64), 0, s, partials, slots, (int)dist, \
                       scores, kept_idx, (const u32x4*)src, (u32x4*)out, reinterpret_cast<float2*>(stats), N, n_prefix,      \
                       n_keep, row_vec, D, eps)
    if (row_vec <= 64) { if (st) RS_SG(true, 1); else RS_SG(false, 1); }
    else if (row_vec <= 128) { if (st) RS_SG(true, 2); else RS_SG(false, 2); }
    else { if (st) RS_SG(true, 4); else RS_SG(false, 4); }
#undef RS_SG
    return hipGetLastError();
}

// lanes that share one row of `vec` 16-byte vectors in the gathers: the next power of two, at most a wave
static int gather_lanes(int vec) {
    int g = 1;
    while (g < vec && g < 64) g *= 2;
    return g;
}

#define RS_GATHER_LANES(g_, CALL_)                                                     \
    switch (g_) {                                                                      \
        case 1: case 2: case 4: case 8: CALL_(8); break;                               \
        case 16: CALL_(16); break;                                                     \
        case 32: CALL_(32); break;                                                     \
        default: CALL_(64); break;                                                     \
    }

hipError_t launch_gather(rs_dtype dt, const void* src, const int32_t* kept_idx, void* out, int B,
                         int N, int K, int D, hipStream_t s) {
    const int64_t rows = (int64_t)B * K;
    if (rows == 0) return hipSuccess;
    const int row_vec = (int)((size_t)D * elem_size(dt) / 16);
#define RS_CALL(G_)                                                                                              \
    {                                                                                                            \
        constexpr int U_ = G_ == 64 ? 1 : 4, CH_ = G_ == 64 ? 4 : 1, RPW_ = 256 / G_ * U_;  /* rows per workgroup */ \
        hipLaunchKernelGGL((gather_rows_kernel<G_, U_, CH_>), dim3((unsigned)((rows + RPW_ - 1) / RPW_)), dim3(256), 0, \
                           s, (const u32x4*)src, kept_idx, (u32x4*)out, rows, N, K, row_vec);                    \
    }
    RS_GATHER_LANES(gather_lanes(row_vec), RS_CALL)
#undef RS_CALL
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Pruning of a 2-D token grid (Sec. 4.2, "CNN and SSM").  Feature maps are narrow (64-512 channels) and
// their lines short (7-56 positions), so what costs time is launches, idle lanes and the fixed work
// of a selection: the kernels below take several positions per wave, and lines of at most
// GRID_LINE positions are selected by counting inside the kernel that has their scores.  Longer lines
// go through separate selection launches.
// ---------------------------------------------------------------------------
constexpr int GRID_LINE = 256;

// Linear workgroup id -> item of [0, n): ids go round-robin to the 8 XCDs, XCD x takes a contiguous range
// (neighbouring lines write neighbouring bytes: they should meet in one L2).  -1: no item.
__device__ __forceinline__ int xcd_item(unsigned bid, int n) {
    const int x = bid & 7, j = bid >> 3, q = n >> 3, r = n & 7;
    if (j >= q + (x < r ? 1 : 0)) return -1;
    return x * q + (x < r ? x : r) + j;
}

// Line-wise variant: the per-position shift averaged along each row and along each column; thread h sums
// row h over w in index order and thread w sums column w over h in index order (fixed order:
// bit-reproducible).
__global__ __launch_bounds__(256) void grid_line_scores_kernel(const float* __restrict__ scores,
                                                               float* __restrict__ row_scores,
                                                               float* __restrict__ col_scores, int H, int W) {
    const float* s = scores + (int64_t)blockIdx.x * H * W;
    for (int h = threadIdx.x; h < H; h += 256) {
        float a = 0.f;
        for (int w = 0; w < W; ++w) a += s[h * W + w];
        row_scores[(int64_t)blockIdx.x * H + h] = a / (float)W;
    }
    for (int w = threadIdx.x; w < W; w += 256) {
        float a = 0.f;
        for (int h = 0; h < H; ++h) a += s[h * W + w];
        col_scores[(int64_t)blockIdx.x * W + w] = a / (float)H;
    }
}

hipError_t launch_grid_line_scores(const float* scores, float* row_scores, float* col_scores, int B, int H,
                                   int W, hipStream_t s) {
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(grid_line_scores_kernel, dim3(B), dim3(256), 0, s, scores, row_scores, col_scores, H, W);
    return hipGetLastError();
}

// The same sums (same order) from a copy of the image's scores in LDS, followed by both selections:
// one launch for the three of the general path.  H, W <= GRID_LINE, H * W * 4 bytes of dynamic LDS.
constexpr size_t GRID_LDS = 64 * 1024;
__global__ __launch_bounds__(512) void grid_line_select_kernel(const float* __restrict__ scores,
                                                               float* __restrict__ row_scores,
                                                               float* __restrict__ col_scores,
                                                               int32_t* __restrict__ kept_rows,
                                                               int32_t* __restrict__ kept_cols, int H, int W, int R,
                                                               int Q) {
    __shared__ float s_row[GRID_LINE], s_col[GRID_LINE];
    extern __shared__ float s_map[];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    const float* s = scores + b * H * W;
    for (int i = tid; i < H * W; i += 512) s_map[i] = s[i];
    __syncthreads();
    if (tid < 256) {
        if (tid < H) {
            float a = 0.f;
            for (int w = 0; w < W; ++w) a += s_map[tid * W + w];
            row_scores[b * H + tid] = s_row[tid] = a / (float)W;
        }
    } else if (tid - 256 < W) {
        const int w = tid - 256;
        float a = 0.f;
        for (int h = 0; h < H; ++h) a += s_map[h * W + w];
        col_scores[b * W + w] = s_col[w] = a / (float)H;
    }
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63;
    if (wave > 1) return;
    // wave 0: rows, wave 1: columns
    const float* sc = wave == 0 ? s_row : s_col;
    const int n = wave == 0 ? H : W, n_keep = wave == 0 ? R : Q;
    int32_t* out = wave == 0 ? kept_rows + b * R : kept_cols + b * Q;
    if (n_keep == 0) return;
    uint32_t key[4];
    int pos[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) key[r] = r * 64 + lane < n ? score_key(sc[r * 64 + lane]) : 0u;
    wave_select<4>(key, n, 0, n_keep, lane, pos);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (pos[r] >= 0) out[pos[r]] = r * 64 + lane;
}

// A launch holds less than 2^32 threads (one beyond that is refused or, worse, runs modulo 2^32): 2^23 workgroups of 512.
bool grid_line_select_fits(int B, int H, int W) {
    return H <= GRID_LINE && W <= GRID_LINE && (size_t)H * W * sizeof(float) <= GRID_LDS - 4096 && B < 1 << 23;
}

hipError_t launch_grid_line_select(const float* scores, float* row_scores, float* col_scores, int32_t* kept_rows,
                                   int32_t* kept_cols, int B, int H, int W, int R, int Q, hipStream_t s) {
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(grid_line_select_kernel, dim3(B), dim3(512), (size_t)H * W * sizeof(float), s, scores, row_scores,
                       col_scores, kept_rows, kept_cols, H, W, R, Q);
    return hipGetLastError();
}

// out[b, i, j, :] = src[b, kept_rows[b, i], kept_cols[b, j], :]; G lanes per output position, four
// positions per thread, all requested before the first is stored
template <int G>
__global__ __launch_bounds__(256) void grid_gather_kernel(const u32x4* __restrict__ src,
                                                          const int32_t* __restrict__ kept_rows,
                                                          const int32_t* __restrict__ kept_cols,
                                                          u32x4* __restrict__ out, int64_t positions, int H, int W,
                                                          int R, int Q, int vec) {
    constexpr int U = 4, PPG = 256 / G;
    const int sub = threadIdx.x % G;
    const int64_t p0 = (int64_t)blockIdx.x * (PPG * U) + threadIdx.x / G;
    int64_t sp[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t p = p0 + u * PPG;
        if (p < positions) {
            const uint32_t pu = (uint32_t)p;  // positions < 2^31
            const uint32_t b = pu / (uint32_t)(R * Q), ij = pu - b * (uint32_t)(R * Q);
            const uint32_t i = ij / (uint32_t)Q, j = ij - i * Q;
            sp[u] = ((int64_t)b * H + kept_rows[(int64_t)b * R + i]) * W + kept_cols[(int64_t)b * Q + j];
        } else {
            sp[u] = -1;
        }
    }
    for (int c = sub; c < vec; c += G) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (sp[u] >= 0) v[u] = src[sp[u] * vec + c];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (sp[u] >= 0) out[(p0 + u * PPG) * vec + c] = v[u];
    }
}

hipError_t launch_grid_gather(rs_dtype dt, const void* src, const int32_t* kept_rows, const int32_t* kept_cols,
                              void* out, int B, int H, int W, int R, int Q, int C, hipStream_t s) {
    const int64_t positions = (int64_t)B * R * Q;
    if (positions == 0) return hipSuccess;
    const int vec = (int)((size_t)C * elem_size(dt) / 16);
#define RS_CALL(G_)                                                                                                  \
    hipLaunchKernelGGL(grid_gather_kernel<G_>, dim3((unsigned)((positions + 1024 / G_ - 1) / (1024 / G_))), dim3(256), 0, s, \
                       (const u32x4*)src, kept_rows, kept_cols, (u32x4*)out, positions, H, W, R, Q, vec)
    RS_GATHER_LANES(gather_lanes(vec), RS_CALL)
#undef RS_CALL
    return hipGetLastError();
}

// Token-wise variant: every row first keeps its Q highest-shift positions, the rows close up, and every
// column of the compacted H x Q grid then keeps its R highest-shift positions.
//
// First half, lines of at most GRID_LINE positions: one workgroup per grid row forms the scores of its W
// positions (G lanes per position while rows of C elements fit, else a wave per position), selects
// by counting and writes the survivors' scores to their places in the compacted grid.
template <typename T, int DIST, int G>
__global__ __launch_bounds__(256) void grid_row_select_kernel(const T* __restrict__ f_out, const T* __restrict__ f_in,
                                                              float* __restrict__ scores, int32_t* __restrict__ kept_cols,
                                                              float* __restrict__ col_scores, int rows, int H, int W,
                                                              int C, int Q) {
    __shared__ float s_sc[GRID_LINE];
    const int row = xcd_item(blockIdx.x, rows);
    if (row < 0) return;  // whole workgroup, before any barrier
    const int tid = threadIdx.x, sub = tid % G;
    const int64_t base = (int64_t)row * W * C;
    constexpr int PPG = 256 / G;
    if (G < 64 || C <= 512) {
        constexpr int U = 2;
        const bool on = sub * 8 < C;
        for (int w0 = tid / G; w0 < W; w0 += PPG * U) {
            float x[U][8], y[U][8];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int w = w0 + u * PPG;
                if (on && w < W) {
                    Elem<T>::load8(f_out + base + (int64_t)w * C + sub * 8, x[u]);
                    Elem<T>::load8(f_in + base + (int64_t)w * C + sub * 8, y[u]);
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[u][i] = y[u][i] = 0.f;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float sc = group_score<DIST, G>(x[u], y[u]);
                if (sub == 0 && w0 + u * PPG < W) s_sc[w0 + u * PPG] = sc;
            }
        }
    } else {
        for (int w = tid / 64; w < W; w += 4) {
            float p0 = 0.f, p1 = 0.f, p2 = 0.f;
            for (int c = sub * 8; c < C; c += 512) {
                float x[8], y[8];
                Elem<T>::load8(f_out + base + (int64_t)w * C + c, x);
                Elem<T>::load8(f_in + base + (int64_t)w * C + c, y);
#pragma unroll
                for (int i = 0; i < 8; ++i) dist_term<DIST>(x[i], y[i], p0, p1, p2);
            }
            p0 = wave_sum(p0);
            if (DIST == RS_DIST_COS) { p1 = wave_sum(p1); p2 = wave_sum(p2); }
            if (sub == 0) s_sc[w] = dist_value<DIST>(p0, p1, p2);
        }
    }
    __syncthreads();
    if (tid >= 64) {  // waves 1 .. 3 write the scores while wave 0 selects
        for (int w = tid - 64; w < W; w += 192) scores[(int64_t)row * W + w] = s_sc[w];
        return;
    }
    const int b = row / H, h = row - b * H;
    auto select = [&](auto regs) {
        constexpr int R = decltype(regs)::value;
        uint32_t key[R];
        int pos[R];
#pragma unroll
        for (int r = 0; r < R; ++r) key[r] = r * 64 + tid < W ? score_key(s_sc[r * 64 + tid]) : 0u;
        wave_select<R>(key, W, 0, Q, tid, pos);
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (pos[r] >= 0) {
                kept_cols[(int64_t)row * Q + pos[r]] = r * 64 + tid;
                if (col_scores) col_scores[((int64_t)b * Q + pos[r]) * H + h] = s_sc[r * 64 + tid];
            }
    };
    if (W <= 64) select(std::integral_constant<int, 1>{});
    else select(std::integral_constant<int, 4>{});
}

// Both launches round their workgroups of 256 (a grid row each; four columns each) up to a multiple of 8 and hold less
// than 2^32 threads.
bool grid_token_fused_fits(int64_t B, int H, int W, int Q) {
    constexpr int64_t most = ((int64_t)1 << 24) - 8;
    return H <= GRID_LINE && W <= GRID_LINE && B * H <= most && B * ((Q + 3) / 4) <= most;
}

template <typename T, int DIST>
static hipError_t launch_grid_row_select_t(const void* f_out, const void* f_in, float* scores, int32_t* kept_cols,
                                           float* col_scores, int B, int H, int W, int C, int Q, hipStream_t s) {
    const int rows = B * H;
#define RS_CALL(G_)                                                                                                  \
    hipLaunchKernelGGL((grid_row_select_kernel<T, DIST, G_>), dim3(8 * (unsigned)((rows + 7) / 8)), dim3(256), 0, s, \
                       (const T*)f_out, (const T*)f_in, scores, kept_cols, col_scores, rows, H, W, C, Q)
    RS_GATHER_LANES(gather_lanes(C / 8), RS_CALL)
#undef RS_CALL
    return hipGetLastError();
}

hipError_t launch_grid_row_select(rs_dtype dt, rs_dist dist, const void* f_out, const void* f_in, float* scores,
                                  int32_t* kept_cols, float* col_scores, int B, int H, int W, int C, int Q, hipStream_t s) {
    if (B == 0) return hipSuccess;
#define RS_CALL(T_)                                                                                                       \
    (dist == RS_DIST_L2 ? launch_grid_row_select_t<T_, RS_DIST_L2>(f_out, f_in, scores, kept_cols, col_scores, B, H, W, C, Q, s) \
     : dist == RS_DIST_L1 ? launch_grid_row_select_t<T_, RS_DIST_L1>(f_out, f_in, scores, kept_cols, col_scores, B, H, W, C, Q, s) \
                          : launch_grid_row_select_t<T_, RS_DIST_COS>(f_out, f_in, scores, kept_cols, col_scores, B, H, W, C, Q, s))
    return dt == RS_F32 ? RS_CALL(float) : RS_CALL(bf16raw);
#undef RS_CALL
}

// Second half: one wave per column of the compacted grid selects R of its H positions by counting and
// copies them, four neighbouring columns per workgroup (their positions are neighbours in `out`).
//   out[b, i, j, :] = src[b, r, kept_cols[b, r, j], :] with r = kept_rows[b, j, i]
template <int G>
__global__ __launch_bounds__(256) void grid_col_gather_kernel(const u32x4* __restrict__ src,
                                                              const int32_t* __restrict__ kept_cols,
                                                              const float* __restrict__ col_scores,
                                                              int32_t* __restrict__ kept_rows, u32x4* __restrict__ out,
                                                              int items, int groups, int H, int W, int R, int Q, int vec) {
    __shared__ int s_pos[4][GRID_LINE];  // source position (r * W + c) of the column's i-th survivor
    const int item = xcd_item(blockIdx.x, items);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (item < 0) return;
    const int b = item / groups, j = (item - b * groups) * 4 + wave;
    if (j >= Q) return;  // whole wave; no workgroup barrier below
    const int64_t bj = (int64_t)b * Q + j;
    auto select = [&](auto regs) {
        constexpr int RG = decltype(regs)::value;
        uint32_t key[RG];
        int pos[RG];
#pragma unroll
        for (int r = 0; r < RG; ++r) key[r] = r * 64 + lane < H ? score_key(col_scores[bj * H + r * 64 + lane]) : 0u;
        wave_select<RG>(key, H, 0, R, lane, pos);
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            const int h = r * 64 + lane;
            if (pos[r] >= 0) {
                kept_rows[bj * R + pos[r]] = h;
                s_pos[wave][pos[r]] = h * W + kept_cols[((int64_t)b * H + h) * Q + j];
            }
        }
    };
    if (H <= 64) select(std::integral_constant<int, 1>{});
    else select(std::integral_constant<int, 4>{});
    if (!out) return;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    constexpr int U = 4, PPG = 64 / G;
    const int sub = lane % G;
    const u32x4* sb = src + (int64_t)b * H * W * vec;
    u32x4* ob = out + (int64_t)b * R * Q * vec;
    for (int i0 = lane / G; i0 < R; i0 += PPG * U)
        for (int c = sub; c < vec; c += G) {
            u32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * PPG < R) v[u] = sb[(int64_t)s_pos[wave][i0 + u * PPG] * vec + c];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * PPG < R) ob[((int64_t)(i0 + u * PPG) * Q + j) * vec + c] = v[u];
        }
}

hipError_t launch_grid_col_gather(rs_dtype dt, const void* src, const int32_t* kept_cols, const float* col_scores,
                                  int32_t* kept_rows, void* out, int B, int H, int W, int R, int Q, int C, hipStream_t s) {
    if (B == 0 || R == 0 || Q == 0) return hipSuccess;
    const int vec = (int)((size_t)C * elem_size(dt) / 16);
    const int groups = (Q + 3) / 4, items = B * groups;
#define RS_CALL(G_)                                                                                                   \
    hipLaunchKernelGGL(grid_col_gather_kernel<G_>, dim3(8 * (unsigned)((items + 7) / 8)), dim3(256), 0, s, (const u32x4*)src, \
                       kept_cols, col_scores, kept_rows, (u32x4*)out, items, groups, H, W, R, Q, vec)
    RS_GATHER_LANES(gather_lanes(vec), RS_CALL)
#undef RS_CALL
    return hipGetLastError();
}

// Longer lines: the selections are launches of their own (select_kernel, one line as one "image").
// col_scores[b, j, h] = scores[b, h, kept_cols[b, h, j]] feeds the second one.
__global__ __launch_bounds__(256) void grid_compact_scores_kernel(const float* __restrict__ scores,
                                                                  const int32_t* __restrict__ kept_cols,
                                                                  float* __restrict__ col_scores, int64_t total,
                                                                  int H, int W, int Q) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;  // index into [B, Q, H]
    if (t >= total) return;
    const int h = (int)(t % H);
    const int64_t bj = t / H;
    const int j = (int)(bj % Q);
    const int64_t b = bj / Q;
    col_scores[t] = scores[(b * H + h) * W + kept_cols[(b * H + h) * Q + j]];
}

// out[b, i, j, :] = src[b, r, kept_cols[b, r, j], :] with r = kept_rows[b, j, i]; one wavefront per position
__global__ __launch_bounds__(256) void grid_token_gather_kernel(const uint4* __restrict__ src,
                                                                const int32_t* __restrict__ kept_cols,
                                                                const int32_t* __restrict__ kept_rows,
                                                                uint4* __restrict__ out, int64_t positions, int H,
                                                                int W, int R, int Q, int vec) {
    const int lane = threadIdx.x & 63;
    const int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (p >= positions) return;
    const int64_t b = p / ((int64_t)R * Q);
    const int ij = (int)(p - b * R * Q);
    const int i = ij / Q, j = ij - i * Q;
    const int r = kept_rows[(b * Q + j) * R + i];
    const int c = kept_cols[(b * H + r) * Q + j];
    const int64_t sp = (b * H + r) * W + c;
    for (int v = lane; v < vec; v += 64) out[p * vec + v] = src[sp * vec + v];
}

hipError_t launch_grid_compact_scores(const float* scores, const int32_t* kept_cols, float* col_scores, int B, int H,
                                      int W, int Q, hipStream_t s) {
    const int64_t total = (int64_t)B * Q * H;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(grid_compact_scores_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, scores,
                       kept_cols, col_scores, total, H, W, Q);
    return hipGetLastError();
}

hipError_t launch_grid_token_gather(rs_dtype dt, const void* src, const int32_t* kept_cols, const int32_t* kept_rows,
                                    void* out, int B, int H, int W, int R, int Q, int C, hipStream_t s) {
    const int64_t positions = (int64_t)B * R * Q;
    if (positions == 0) return hipSuccess;
    const int vec = (int)((size_t)C * elem_size(dt) / 16);
    hipLaunchKernelGGL(grid_token_gather_kernel, dim3((unsigned)((positions + 3) / 4)), dim3(256), 0, s,
                       (const uint4*)src, kept_cols, kept_rows, (uint4*)out, positions, H, W, R, Q, vec);
    return hipGetLastError();
}

}  // namespace rs
