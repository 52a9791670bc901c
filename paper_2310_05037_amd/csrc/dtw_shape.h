// dtw_shape.h -- how the stripe sweep cuts a pair into work items: the rule
// alone, which the planner (dtw_plan.hip) and host code read.
#pragma once

#include <math.h>

#include "internal.h"

namespace ra {

// Work items of a pair in the stripe sweep: each sweeps k stripes of 64 c
// columns one after another.  lim = 0: one item.  Else lim is what one item
// may cost, in cells per lane (a share of the batch's cells per resident
// wave): a longer one would end after the rest of the batch, so the pair is
// cut into items of one stripe that run beside each other (an item of several
// would hold up its right neighbour until its last).  Items narrower than 64
// sqrt(26 m / n) columns, or 64 kSweepMinC, do not pay: each starts about 166
// rows after its left neighbour, and a row of c columns costs a lone wave about
// 52 + 5.2 c ns, so (n + 166 m / (64 c)) (52 + 5.2 c) is least there.  A query
// longer than an edge column (kEdgeCap) is not cut: a ring slot holds the column,
// its corner and two words of the running minimum, and nothing past its end is
// this pair's.
RA_HOST_DEV inline void sweep_shape(int n, int m, float lim, int &items, int &k, int &c) {
    const int stripes = m > kSweepStripe ? (m + kSweepStripe - 1) / kSweepStripe : 1;
    items = 1;
    if (lim > 0.0f && n <= kEdgeCap) {
        const float rows = (float)(n < 1 ? 1 : n), cols = (float)m;
        const float want = ceilf(rows * cols / (64.0f * lim));
        const float most = ceilf(cols / (64.0f * fmaxf((float)kSweepMinC, sqrtf(26.0f * cols / rows))));
        const int more = (int)fminf(want, most);
        if (want > 1.0f) items = more > stripes ? more : stripes;
    }
    k = items > 1 ? 1 : stripes;
    c = (m + 64 * items * k - 1) / (64 * items * k);
    if (c < 1) c = 1;
    if (items > 1) items = (m + 64 * c - 1) / (64 * c);   // every item starts inside the region
}

// Work items a pair of at most n events and m levels can have, whatever lim.
RA_HOST_DEV inline int64_t most_items(int64_t n, int64_t m) {
    const float rows = (float)(n < 1 ? 1 : n < kEdgeCap ? n : kEdgeCap), cols = (float)(m < 1 ? 1 : m < kMaxRegion ? m : kMaxRegion);
    const float most = cols / (64.0f * fmaxf((float)kSweepMinC, sqrtf(26.0f * cols / rows)));
    return (int64_t)fmaxf(most, cols / (float)kSweepStripe) + 2;   // rounded up, and what rounding may add
}
// Many long pairs, twelve for each of `few` workgroups (16 per CU) and a million
// cells a pair: those take all items, and the fifth wave of each SIMD is left out.
// The sweep is bound by issue then, which four waves reach as five do, and the
// clock stays higher.  Uneven pairs, time with 16 per CU over time with 20, on
// 4,096 workgroups:
//     pairs                8,192  16,384  24,576  32,768  49,152  65,536  98,304
//     0.4 M cells a pair    0.99    1.02    0.97    0.99    1.01    1.02    1.03
//     1.7 M                 1.01    1.02    1.00    0.97    0.96    0.97    1.00
//     3.4 M                 1.02    1.03    1.04    1.02    0.97    0.96    0.98
//     6.8 M                 1.05    1.03    0.99    1.06    1.00    0.98
// (100,000 pairs of 9.2 M: 50.7 ms against 53.3).  Fewer pairs need the fifth wave
// to hide the others' waits, shorter ones to hide their starts and ends.
RA_HOST_DEV inline bool few_waves(int64_t n_pairs, double cells, int few) {
    return few > 0 && n_pairs >= 12 * (int64_t)few && cells >= (double)(1 << 20) * (double)n_pairs;
}

static_assert(kEdgeCap + 3 <= kSlotFloats, "an edge column fits its slot");

}  // namespace ra
