// dtw_band.h -- stripes of the banded pairs that are cut (kernels in dtw_band.hip).
#pragma once

#include "dtw_device.h"

namespace ra {

// Stripes of a banded pair: c columns per lane, so that a stripe is a quarter
// to two thirds of the band wide (a stripe meets (64 c + W) n / m rows, of which
// the 64 c part has cells outside the band; narrower ones cost more per step
// and per start: 8.1 ms on 10,000 uneven regions, 8.9 with half the band), and
// one item per stripe where the pair costs more than lim.  All rows pass
// through the stripes' waves one after another, so such a pair takes narrower
// stripes down to n c = lim.  Pairs that fit a moving frame are swept faster
// there and cut only above four times the share (40,000 chains: 3.34 ms, 3.51
// at twice, 3.40 at once, 3.34 uncut but for the widest).  False: it is not cut, and needs no stripes unless
// it is too wide for the other classes.
RA_DEV float band_cost(int n, int m, int w, int &c) {
    const int W = 2 * w + 1 < m ? 2 * w + 1 : m;
    c = W <= 1024 ? 4 : W <= 1536 ? 8 : 16;
    const int cols = W + 64 * c < m ? W + 64 * c : m;
    return (float)n * (float)cols / 64.0f;
}
RA_DEV bool band_shape(int n, int m, int w, float lim, int &items, int &c) {
    items = 1;
    if (m <= n && 2 * w + 1 <= kBandMaxFrame) lim *= 4.0f;
    if (!(band_cost(n, m, w, c) > lim) || n > kEdgeCap) return false;
    while (c > 4 && (float)n * (float)c > lim) c /= 2;
    items = (m + 64 * c - 1) / (64 * c);
    return items > 1;
}
static_assert(kMaxRegion / (64 * 4) < 512, "item fields");

}  // namespace ra
