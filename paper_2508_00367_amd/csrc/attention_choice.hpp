// Which kernel of the bf16 attention of long sequences takes which query rows: host arithmetic only, no HIP.
#pragma once

#include <stdint.h>

namespace rs {

constexpr int ATT_BM = 256;        // query rows per workgroup of 8 waves; one of 4 waves has half of them
constexpr int ATT_TAIL_ROWS = 64;  // at most so many rows beyond the last full tile may go to the tail kernel

// Workgroups of `rows` query rows, `q_tiles` of them per (image, head); tail: the rows behind these to the tail kernel.
struct AttentionPlan {
    int rows, q_tiles;
    bool tail;
};

// By what the busiest CU of an XCD gets, in workgroups of 4 waves (it holds four of them, or two of 8 waves; a head
// stays on one XCD; the tail kernel costs about 0.6 per head of a CU and 8 us).  us, 8 waves / 4 waves / 8 waves + tail:
// 8 x 1569 x 12 heads 92 / 82 / 105, 4 x 1407 x 16 53 / 46, 20 x 785 x 12 64 / 57 / 65, 3 x 1569 x 12 55 / 45 / 49, 1 x 1569 x 12
// 31.5 / 23.6 / 46, 4 x 4097 x 16 312 / 324 / 311, 1 x 4097 x 16 127 / 104 / 97, and with the same number on both sides
// 4 x 2869 x 16 153 / 160, 4 x 2009 x 16 79 / 83, 2 x 2353 x 12 46.5 / 48.6: the larger tile, which copies K and V half as often.
inline AttentionPlan attention_plan(int64_t BH, int N, int64_t all_cus) {
    const int64_t heads = (BH + 7) / 8, cus = all_cus / 8;
    auto busiest = [&](int64_t tiles) { return (heads * tiles + cus - 1) / cus; };
    const int rem = N % ATT_BM;
    const int64_t c8 = 20 * busiest((N + ATT_BM - 1) / ATT_BM), c4 = 10 * busiest((N + ATT_BM / 2 - 1) / (ATT_BM / 2));
    const int64_t c_tail = 20 * busiest(N / ATT_BM) + 6 * busiest(1) + 9000 / N;
    if (rem > 0 && rem <= ATT_TAIL_ROWS && N > ATT_BM && c_tail < c8 && c_tail < c4) return {ATT_BM, N / ATT_BM, true};
    const int rows = c8 <= c4 ? ATT_BM : ATT_BM / 2;
    return {rows, (N + rows - 1) / rows, false};
}

}  // namespace rs
