// The planner's shape rules (csrc/dtw_shape.h) and limits, for the host tests.
#include "dtw_shape.h"

extern "C" {

void sweep_shape(int n, int m, float lim, int *out) { ra::sweep_shape(n, m, lim, out[0], out[1], out[2]); }

int few_waves(long long pairs, double cells, int few) { return ra::few_waves(pairs, cells, few); }
long long most_items(long long n, long long m) { return ra::most_items(n, m); }

int limit(int which) {
    const int v[] = {ra::kEdgeCap, ra::kSlotFloats, ra::kSweepStripe, ra::kSingleMaxRegion, ra::kMaxItems, ra::kSweepMaxC};
    return v[which];
}
}
