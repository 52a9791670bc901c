// dtw_path.h -- warping path of an alignment (kernels in dtw_path.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace ra {

// Widest stripe of the direction pass: 64 lanes x 32 columns.
constexpr int kPathStripeCols = 64 * 32;
// Direction words per query row and 2,048 columns: 2 bits per column.
constexpr int kPathWordsPerRow = 64;

// Workspace words pair p needs for an interval of L levels: per stripe and
// row one word per lane, plus one word per row for the stripe edge.
__host__ __device__ inline int64_t path_words(int64_t n, int64_t L) {
    const int64_t S = (L + kPathStripeCols - 1) / kPathStripeCols;
    return n * (kPathWordsPerRow * S + 1);
}

// Bytes from one row's codes to the next.
__host__ __device__ inline int64_t path_pitch(int64_t L) {
    return (L + kPathStripeCols - 1) / kPathStripeCols * kPathWordsPerRow * 8;
}

struct PathArgs {
    const float *q;
    int64_t q_size;
    const int64_t *q_off;
    const int32_t *q_len;
    const float *r;
    int64_t r_size;
    const int64_t *r_off;
    const int32_t *r_len;
    const int32_t *start;   // per pair, from the start-of-alignment pass
    const int32_t *end;
    int64_t n_pairs;
    const int64_t *dir_off;   // per pair: first workspace word
    uint64_t *dirs;           // caller's workspace
    int64_t dir_size;         // words
    const int64_t *path_off;
    int32_t *path_lo;
    int32_t *path_hi;
    int64_t path_size;
};

// Directions (the items of the chained queue that launch_path_plan wrote), then
// the paths.
hipError_t launch_path_plan(const PathArgs &pa, int grid, const PlanScratch &s, const SweepScratch &sw,
                            hipStream_t stream);
hipError_t launch_path(const PathArgs &pa, int grid, const SweepScratch &sw, hipStream_t stream);
int path_blocks_per_cu();

// Interval of pair p, or a sentinel: -1 / -2 from the start pass (empty
// query or region / invalid slice), kGaveUp where one of its passes was given
// up, -4 when the pair's workspace range is missing or too small.
__host__ __device__ __forceinline__ int path_interval(const PathArgs &pa, int64_t p, int &n, int &s, int &L) {
    n = pa.q_len[p];
    const int e = pa.end[p];
    s = pa.start[p];
    if (e < 0) return e;
    if (s == kGaveUp) return s;
    const int m = pa.r_len[p];
    const int64_t qo = pa.q_off[p], ro = pa.r_off[p];
    if (n < 1 || s < 0 || s > e || e >= m || qo < 0 || ro < 0 || qo + n > pa.q_size || ro + m > pa.r_size)
        return -2;
    L = e - s + 1;
    const int64_t off = pa.dir_off[p];
    if (off < 0 || off > pa.dir_size || path_words(n, L) > pa.dir_size - off) return -4;
    return 0;
}

// Work items of a pair's n x L direction table: one per stripe of 64 c columns,
// c = 4, 8, 16 or 32, where the pair costs more than lim (see sweep_shape);
// else, and where a ring slot or an item's fields are too small, one for all.
__host__ __device__ __forceinline__ void path_shape(int n, int L, float lim, int &items, int &c) {
    const float cost = (float)n * (float)L / 64.0f;
    const bool split = n <= kEdgeCap && L <= kMaxRegion && cost > lim;
    const int want = split ? (int)fminf(ceilf(cost / lim), 1024.0f) : 1;
    const int cols = split || L < kPathStripeCols ? L : kPathStripeCols;
    const int least = (cols + 64 * want - 1) / (64 * want);
    c = least <= 4 ? 4 : least <= 8 ? 8 : least <= 16 ? 16 : 32;
    items = split ? (L + 64 * c - 1) / (64 * c) : 1;
}
// A wait of the direction pass was given up (`failed`) and the pair is one of
// those that were cut: its table is in doubt.
__host__ __device__ __forceinline__ bool path_lost(int n, int L, float lim, bool failed) {
    int items = 1, c;
    if (failed) path_shape(n, L, lim, items, c);
    return items > 1;
}
static_assert(kMaxRegion / (64 * 4) < 512, "item fields");

}  // namespace ra
