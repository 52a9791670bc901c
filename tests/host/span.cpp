// Starts and path intervals of pairs (csrc/internal.h, csrc/dtw_path.h).
#include "dtw_path.h"

extern "C" {
int span_start(int end, int rev_end) { return ra::span_start(end, rev_end); }

// path_interval of a pair of n events and m levels with room for its codes.
int interval(int n, int m, int start, int end) {
    const int64_t off = 0;
    ra::PathArgs pa{};
    pa.q_size = n;
    pa.r_size = m;
    pa.q_off = pa.r_off = pa.dir_off = &off;
    pa.q_len = &n;
    pa.r_len = &m;
    pa.start = &start;
    pa.end = &end;
    pa.dir_size = (int64_t)1 << 40;
    int a, b, c;
    return ra::path_interval(pa, 0, a, b, c);
}
}
