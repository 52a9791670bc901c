// dtw_bnb.h -- what happens to a pair between the rounds of early termination
// (kernels in dtw_bnb.hip).
#pragma once

#include <math.h>

#include "internal.h"

namespace ra {

// Monotone encoding of doubles as unsigned 64-bit keys (larger double ->
// larger key), so the per-read best can be raised with an integer atomicMax.
RA_HOST_DEV inline uint64_t order_key(double d) {
    const uint64_t b = __builtin_bit_cast(uint64_t, d);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
RA_HOST_DEV inline double order_value(uint64_t k) {
    const uint64_t b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    return __builtin_bit_cast(double, b);
}

// The next round's part of pair p: rows [from, to), or none (from < 0).
RA_HOST_DEV inline void bnb_part(const BnbArgs &b, int64_t p, int from, int to) {
    b.s.part_off[p] = b.a.q_off[p] + (from < 0 ? 0 : from);
    b.s.part_len[p] = from < 0 ? -1 : to - from;   // a negative length is skipped
    b.s.part_first[p] = from == 0;
    b.s.part_row[p] = from;
}

// After a round: the result of a pair that it completed, or whose sweep was
// given up (NaN, kGaveUp: the resident row is only partly the pair's, so there
// is nothing to go on from).  Returns the read whose best Score the pair may
// raise (to `key`), or -1.
RA_HOST_DEV inline int bnb_finish(const BnbArgs &b, int64_t p, uint64_t &key) {
    if (b.s.status[p] == kBnbDone || b.s.part_row[p] < 0) return -1;
    const bool lost = b.s.part_end[p] == kGaveUp;
    if (!lost && b.s.part_row[p] + b.s.part_len[p] < b.a.q_len[p]) return -1;
    const float cost = b.s.part_score[p];
    b.a.out_score[p] = cost;
    b.a.out_end[p] = b.s.part_end[p];
    b.s.status[p] = kBnbDone;
    const int k = lost ? -1 : b.s.read_of[p];
    if (k >= 0) key = order_key(b.b_match * (double)b.n_events[k] - (double)cost);
    return k;
}

// The open pairs' next round (every pair here has one read: the others were
// aligned whole), or their end.  A pair is dropped in the row where its
// minimum reaches `need`; at min / rows a row that is need / min times the rows
// so far, and 5 % are added for rows that cost less.  Steps of a fixed length
// or ratio instead sweep a pair up to half further and take more rounds, each
// 63 steps of skew per pair and 45 us of launches: 11.8 ms against 7.8 on 20,000
// pairs of the uneven batch (82 % of them dropped).
RA_HOST_DEV inline void bnb_advance(const BnbArgs &b, int64_t p, int block_rows, bool whole) {
    if (b.s.status[p] == kBnbDone) {
        bnb_part(b, p, -1, 0);
        return;
    }
    const int k = b.s.read_of[p];
    const double most = b.b_match * (double)b.n_events[k], best = order_value(b.s.best[k]);
    const double cost = b.s.part_score[p];
    if (most - cost < best) {
        b.a.out_score[p] = __builtin_inff();   // cannot win: treated as unmapped by the decision
        b.a.out_end[p] = -3;
        b.s.status[p] = kBnbDone;
        bnb_part(b, p, -1, 0);
        return;
    }
    const int n = b.a.q_len[p], from = b.s.part_row[p] + b.s.part_len[p], least = block_rows / 4;
    const double to = fmax(1.05 * (double)from * ((most - best) / cost), (double)from) + (double)least;
    bnb_part(b, p, from, !whole && to < (double)(n - least) ? (int)to : n);
}

}  // namespace ra
