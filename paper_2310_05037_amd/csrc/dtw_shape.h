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
static_assert(kEdgeCap + 3 <= kSlotFloats, "an edge column fits its slot");

}  // namespace ra
