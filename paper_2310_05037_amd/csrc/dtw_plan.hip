// dtw_plan.hip -- device-side planning (routing, longest-first ordering,
// sentinels for degenerate or invalid pairs) and the mapping decision.
#include "dtw_band.h"
#include "dtw_path.h"

namespace ra {

struct PlanArgs {
    PairArrays a;
    int64_t n_pairs;
    int buckets;      // 1: single bucket (plain), kBuckets: LPT buckets
    int extend;
    int single_max;   // widest region of the single-stripe routes
    int chain;        // the sweep's pairs are listed stripe by stripe (sw)
    float lim_scale;  // share of the batch's cells that one item may have, per lane
    PlanScratch s;
    SweepScratch sw;
    const int32_t *band;   // banded planning (band half-width per pair), else null
    int paths;             // planning of the direction pass (path), whose intervals are the regions
    PathArgs path;
    int few;               // workgroups of the sweep for many long pairs (see few_waves)
    int chain_route;       // the list whose counters the chained queue's items have
};

// Banded pairs (dtw_band.hip): class 0 for frames of at most kBandLoMaxH*128
// columns, class 1 for wider ones, longest first by the frame cells swept;
// for the shapes the band-relative frame does not take (more levels than
// events, or a band wider than one wave's frame), class 2 when the whole
// region fits one wave's frame and class 3 (stripes) above that.  Pairs
// that need no kernel get their result here: NaN/-2 for an invalid slice
// or a negative band, (0, -1) for an empty query, (+inf, -1) for an empty
// region, NaN/-4 for the one shape left: a query longer than a stripe edge
// column (kEdgeCap) against more than 2048 levels with a band wider than
// 2048 columns.
RA_DEV int band_classify(const PlanArgs &pa, int64_t p, float lim, int &bucket, float &score, int &end) {
    const PairArrays &a = pa.a;
    const int n = a.q_len[p];
    const int m = a.r_len[p];
    const int wraw = pa.band[p];
    if (!slices_ok(a, p, false) || wraw < 0) {
        score = __builtin_nanf("");
        end = -2;
        return -1;
    }
    if (n == 0 || m == 0) {
        score = n == 0 ? 0.0f : kInf;
        end = -1;
        return -1;
    }
    const int w = wraw < m - 1 ? wraw : m - 1;
    const int W = 2 * w + 1;
    int items, c;
    if (pa.chain && band_shape(n, m, w, lim, items, c)) {
        // In the order of the time they take: rows in turn, and 190 rows from
        // one stripe's start to the next one's.
        const int b = (int)(4.0f * __log2f(((float)n + 190.0f * (float)items) * (float)(64 * c) + 1.0f));
        bucket = kBuckets - 1 - (b >= kBuckets ? kBuckets - 1 : b);
        return 3;
    }
    if (m > n || W > kBandMaxFrame) {
        if (m <= kBandMaxFrame) {
            const float work = (float)(n + 64) * (float)(128 * ((m + 127) / 128)) + 1.0f;
            int b = (int)(4.0f * __log2f(work));
            b = b < 0 ? 0 : (b >= kBuckets ? kBuckets - 1 : b);
            bucket = kBuckets - 1 - b;
            return 2;
        }
        if (n <= kEdgeCap) {
            // stripes of the band's rows only: about the rows the band
            // spends in each stripe times its width
            int S, h;
            const int cols = stripe_shape(m, S, h, false);
            const float rows = fminf((float)n, (float)(cols + W) * (float)n / (float)m + 64.0f);
            const float work = rows * (float)(S * cols) + 1.0f;
            int b = (int)(4.0f * __log2f(work));
            b = b < 0 ? 0 : (b >= kBuckets ? kBuckets - 1 : b);
            bucket = kBuckets - 1 - b;
            return 3;
        }
        score = __builtin_nanf("");
        end = -4;
        return -1;
    }
    const int h = (W + 127) / 128;
    const float work = (float)(n + 64) * (float)(128 * h) + 1.0f;
    int b = (int)(4.0f * __log2f(work));
    b = b < 0 ? 0 : (b >= kBuckets ? kBuckets - 1 : b);
    bucket = kBuckets - 1 - b;
    return h <= kBandLoMaxH ? 0 : 1;
}

// Route of pair p.  Returns -1 when the pair needs no kernel; then
// (score, end) is its result: a sentinel for invalid slices (NaN, -2) or the
// value of a degenerate pair (empty query or empty region).  Returns -2 for
// a global pair that the one-pair-per-lane kernel aligns (no output here).
RA_DEV int classify(const PlanArgs &pa, int64_t p, float lim, int &bucket, float &score, int &end) {
    if (pa.paths) {
        int n = 0, s = 0, L = 0;
        if (path_interval(pa.path, p, n, s, L) != 0) return -2;   // the trace writes its sentinel
        const int b = (int)(4.0f * __log2f((float)n * (float)(L + 64) + 1.0f));
        bucket = kBuckets - 1 - (b >= kBuckets ? kBuckets - 1 : b);
        return kRouteSingleLo;
    }
    if (pa.band) return band_classify(pa, p, lim, bucket, score, end);
    const PairArrays &a = pa.a;
    const int n = a.q_len[p];
    const int m = a.r_len[p];
    const bool ok = slices_ok(a, p, pa.extend != 0);
    const bool fresh = pa.extend ? a.first_chunk[p] != 0 : true;
    if (!ok) {
        score = __builtin_nanf("");
        end = -2;
        return -1;
    }
    if (a.bound == kBoundGlobal) {
        // Anchors touching diagonally cost 0; a gap with events but no
        // levels (or levels but no events) has no path: +inf.
        if (n == 0 || m == 0) {
            score = (n == 0 && m == 0) ? 0.0f : kInf;
            end = -1;
            return -1;
        }
        if (m <= kTinyMaxCols && !a.reverse) return -2;
    }
    if (n == 0 && fresh) {
        score = 0.0f;
        end = -1;
        return -1;
    }
    if (m == 0) {
        score = n == 0 ? 0.0f : kInf;
        end = -1;
        return -1;
    }
    // Single-stripe routes up to the cut-off; regions up to the widest
    // single stripe whose query is too long for a stripe edge column keep
    // one stripe whatever the cut-off, so the result never depends on it.
    int route;
    if (pa.chain) route = m > kSweepStripe && n > kEdgeCap ? kRouteSingleHi : kRouteSingleLo;
    else if (m <= kSingleLoMaxRegion) route = kRouteSingleLo;
    else if (m <= pa.single_max || (m <= kSingleMaxRegion && n > kEdgeCap)) route = kRouteSingleHi;
    else route = kRouteMulti;
    bucket = 0;
    if (pa.buckets > 1) {
        // Longest-processing-time order: quarter-octave buckets of the swept
        // cells (n + 64 steps per stripe x the stripe's padded columns),
        // bucket 0 holding the largest pairs.
        int S, h;
        const int cols = stripe_shape(m, S, h, route != kRouteMulti);
        const float work = (float)(n + 64) * (float)(S * cols) + 1.0f;
        int b = (int)(4.0f * __log2f(work));
        b = b < 0 ? 0 : (b >= pa.buckets ? pa.buckets - 1 : b);
        bucket = pa.buckets - 1 - b;
    }
    return route;
}

// Pair p is on no list, as its width alone tells: a gap that the one-pair-per-lane
// kernel aligns, or one that needs no kernel.  (Of a million gaps nearly all
// are, and the scatter reads 4 bytes of each instead of 24, twice.)
RA_DEV bool never_listed(const PlanArgs &pa, int64_t p) {
    return !pa.paths && !pa.band && pa.a.bound == kBoundGlobal && !pa.a.reverse && pa.a.r_len[p] <= kTinyMaxCols;
}

// 1024 threads: each thread classifies a few pairs of a million-pair batch,
// one after another; at 256 threads that chain of dependent loads set the
// planning time.
constexpr int kPlanBlock = 1024;
constexpr int kBins = kNumRoutes * kBuckets;

RA_DEV void plan_range(int64_t n_pairs, int64_t &lo, int64_t &hi) {
    const int64_t per = ((n_pairs + gridDim.x - 1) / gridDim.x + kPlanBlock - 1) / kPlanBlock * kPlanBlock;
    lo = (int64_t)blockIdx.x * per;
    hi = lo + per < n_pairs ? lo + per : n_pairs;
}

// Sum over the workgroup, for every thread.
RA_DEV double block_sum(double v) {
    __shared__ double part[kPlanBlock / 64];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < kPlanBlock / 64; ++i) t += part[i];
    return t;
}

// What a pair takes of its route's list: one entry, or its work items.
RA_DEV int list_slots(const PlanArgs &pa, int64_t p, int route, float lim, int &k, int &c) {
    if (!pa.chain || route != pa.chain_route) return 1;
    int items;
    if (pa.band) {
        const int m = pa.a.r_len[p], w = pa.band[p] < m - 1 ? pa.band[p] : m - 1;
        k = 1;
        (void)band_shape(pa.a.q_len[p], m, w, lim, items, c);
        return items;
    }
    if (pa.paths) {
        int n = 0, s = 0, L = 0;
        (void)path_interval(pa.path, p, n, s, L);
        k = 1;
        path_shape(n, L, lim, items, c);
        return items;
    }
    sweep_shape(pa.a.q_len[p], pa.a.r_len[p], lim, items, k, c);
    return items;
}

RA_DEV void write_slots(const PlanArgs &pa, int64_t p, int route, int slots, int k, int c, int at) {
    if (!pa.chain || route != pa.chain_route) {
        pa.s.list[route * pa.s.capacity + at] = (int32_t)p;
        return;
    }
    for (int i = 0; i < slots; ++i)
        if (at + i < pa.sw.item_cap) pa.sw.items[at + i] = pack_item({(int)p, c, k, i, slots});
}

// Phase 0 of a planning workgroup: cells of the pairs [lo, hi).
RA_DEV double plan_cells(const PlanArgs &pa, int64_t lo, int64_t hi) {
    double cells = 0.0;
    if (pa.paths) {
        for (int64_t p = lo + threadIdx.x; p < hi; p += kPlanBlock) {
            int n = 0, s = 0, L = 0;
            if (path_interval(pa.path, p, n, s, L) == 0) cells += (double)n * (double)L;
        }
    } else if (pa.chain && pa.band) {   // the wider pairs are costed at the band's stripes
        for (int64_t p = lo + threadIdx.x; p < hi; p += kPlanBlock) {
            const int n = pa.a.q_len[p], m = pa.a.r_len[p];
            int c;
            if (slices_ok(pa.a, p, false) && n > 0 && m > 0 && pa.band[p] >= 0)
                cells += 64.0 * (double)band_cost(n, m, pa.band[p] < m - 1 ? pa.band[p] : m - 1, c);
        }
    } else if (pa.chain) {
        for (int64_t p = lo + threadIdx.x; p < hi; p += kPlanBlock)
            if (slices_ok(pa.a, p, pa.extend != 0)) cells += (double)pa.a.q_len[p] * (double)pa.a.r_len[p];
    }
    return block_sum(cells);
}

// Clears the sweep's slot counters and, after a call with a wait that timed
// out, refills its ring; every thread of the grid takes part.
RA_DEV void reset_ring(const PlanArgs &pa) {
    const int64_t i0 = (int64_t)blockIdx.x * kPlanBlock + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * kPlanBlock;
    for (int64_t i = i0; i < pa.sw.ring_slots; i += step) pa.sw.done[i] = 0;
    if (*pa.sw.failed) {
        const int64_t words = (int64_t)pa.sw.ring_slots * kSlotFloats;
        for (int64_t i = i0; i < words; i += step) reinterpret_cast<uint32_t *>(pa.sw.ring)[i] = 0xffffffffu;
    }
}

// Counts the pairs [lo, hi) per (route, bucket) into h; pairs that need no
// kernel get their result here.
RA_DEV void plan_count(const PlanArgs &pa, int64_t lo, int64_t hi, float lim, int *h) {
    for (int64_t p = lo + threadIdx.x; p < hi; p += kPlanBlock) {
        int b = 0, e = 0, k = 0, c = 0;
        float sc = 0.0f;
        const int route = classify(pa, p, lim, b, sc, e);
        if (route >= 0) {
            atomicAdd(&h[route * kBuckets + b], list_slots(pa, p, route, lim, k, c));
        } else if (route == -1) {
            pa.a.out_score[p] = sc;
            if (pa.a.out_end) pa.a.out_end[p] = e;
        }
    }
}

// Writes the pairs [lo, hi) to their lists; next[bin] is the bin's cursor.
RA_DEV void plan_scatter(const PlanArgs &pa, int64_t lo, int64_t hi, float lim, const int *base, int *next) {
    for (int64_t p = lo + threadIdx.x; p < hi; p += kPlanBlock) {
        if (never_listed(pa, p)) continue;
        int b = 0, e = 0, k = 0, c = 0;
        float sc = 0.0f;
        const int route = classify(pa, p, lim, b, sc, e);
        if (route >= 0) {
            const int bin = route * kBuckets + b;
            const int slots = list_slots(pa, p, route, lim, k, c);
            write_slots(pa, p, route, slots, k, c, (base ? base[bin] : 0) + atomicAdd(&next[bin], slots));
        }
    }
}

// Exclusive scan of each route's bins (bucket 0 first), one wave per route:
// three buckets per lane.
RA_DEV void plan_scan(const PlanArgs &pa, int *hist) {
    static_assert(kBuckets == 3 * 64, "three buckets per lane");
    const int route = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (route >= kNumRoutes) return;
    int *h = hist + route * kBuckets + 3 * lane;
    const int a0 = h[0], a1 = h[1], a2 = h[2];
    int run = a0 + a1 + a2;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int x = __shfl_up(run, off, 64);
        if (lane >= off) run += x;
    }
    const int excl = run - (a0 + a1 + a2);
    h[0] = excl;
    h[1] = excl + a0;
    h[2] = excl + a0 + a1;
    if (lane == 63) {
        pa.s.counts[route] = run;
        pa.s.queue[route] = 0;
        if (pa.chain && route == pa.chain_route) {
            *pa.sw.n_items = run < pa.sw.item_cap ? run : (int)pa.sw.item_cap;
            pa.sw.n_items[2] = live_workgroups(run, pa.sw.n_items[2]);   // (no others need to ask for items)
            for (int x = 0; x < kQueues; ++x) pa.sw.queue[x * kQueueStride] = 0;
            *pa.sw.failed = 0;
        }
    }
}

// Clears the histogram; chained sweep: cells of each workgroup's range.
__global__ __launch_bounds__(kPlanBlock) void k_plan_start(PlanArgs pa) {
    const int i = blockIdx.x * kPlanBlock + threadIdx.x;
    if (i < kBins) pa.s.hist[i] = 0;
    if (!pa.chain) return;
    reset_ring(pa);
    int64_t lo, hi;
    plan_range(pa.n_pairs, lo, hi);
    const double cells = plan_cells(pa, lo, hi);
    if (threadIdx.x == 0) pa.sw.partial[blockIdx.x] = cells;
}

// Total cells of the batch -> what one item may cost (see sweep_shape).
RA_DEV float plan_lim(const PlanArgs &pa, double cells) {
    const float lim = (float)cells * pa.lim_scale;
    return pa.chain ? fmaxf(lim, 1.0f) : 0.0f;
}
RA_DEV float plan_lim_of_grid(const PlanArgs &pa) {
    if (!pa.chain) return 0.0f;
    return plan_lim(pa, block_sum(threadIdx.x < gridDim.x ? pa.sw.partial[threadIdx.x] : 0.0));
}

// The sweep's workgroups and, for the trace of paths, the share that decides
// which pairs are cut.
RA_DEV void plan_waves(const PlanArgs &pa, float lim) {
    const double cells = (double)lim / (double)pa.lim_scale;
    pa.sw.n_items[2] = !pa.extend && few_waves(pa.n_pairs, cells, pa.few) ? pa.few : 0x7fffffff;
    pa.sw.n_items[3] = __builtin_bit_cast(int, lim);
}

// Each workgroup counts its pairs per (route, bucket) in LDS and adds the
// non-zero bins to the global histogram: one global atomic per bin per
// workgroup instead of one per pair.
__global__ __launch_bounds__(kPlanBlock) void k_plan_count(PlanArgs pa) {
    __shared__ int h[kBins];
    for (int i = threadIdx.x; i < kBins; i += kPlanBlock) h[i] = 0;
    const float lim = plan_lim_of_grid(pa);
    if (pa.chain && blockIdx.x == 0 && threadIdx.x == 0) plan_waves(pa, lim);
    __syncthreads();
    int64_t lo, hi;
    plan_range(pa.n_pairs, lo, hi);
    plan_count(pa, lo, hi, lim, h);
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += kPlanBlock)
        if (h[i]) atomicAdd(&pa.s.hist[i], h[i]);
}

__global__ __launch_bounds__(64 * kNumRoutes) void k_plan_scan(PlanArgs pa) { plan_scan(pa, pa.s.hist); }

// Each workgroup counts its range per bin in LDS, reserves one contiguous
// range per bin with a single global atomic on the bin's cursor, then ranks
// its pairs in LDS again and writes them there (in plain mode, one bin per
// route: workgroups keep their order of arrival at the cursor, pairs inside
// a workgroup their LDS rank).
__global__ __launch_bounds__(kPlanBlock) void k_plan_scatter(PlanArgs pa) {
    __shared__ int cnt[kBins];
    __shared__ int base[kBins];
    for (int i = threadIdx.x; i < kBins; i += kPlanBlock) cnt[i] = 0;
    const float lim = plan_lim_of_grid(pa);
    __syncthreads();
    int64_t lo, hi;
    plan_range(pa.n_pairs, lo, hi);
    for (int64_t p = lo + threadIdx.x; p < hi; p += kPlanBlock) {
        if (never_listed(pa, p)) continue;
        int b = 0, e = 0, k = 0, c = 0;
        float sc = 0.0f;
        const int route = classify(pa, p, lim, b, sc, e);
        if (route >= 0) atomicAdd(&cnt[route * kBuckets + b], list_slots(pa, p, route, lim, k, c));
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += kPlanBlock) {
        if (cnt[i]) base[i] = atomicAdd(&pa.s.hist[i], cnt[i]);
        cnt[i] = 0;
    }
    __syncthreads();
    plan_scatter(pa, lo, hi, lim, base, cnt);
}

// Small batches: the same phases in one workgroup, one launch instead of
// four (a launch between dependent kernels costs more than planning a few
// thousand pairs).
constexpr int64_t kPlanSmall = 4096;
__global__ __launch_bounds__(kPlanBlock) void k_plan_small(PlanArgs pa) {
    __shared__ int h[kBins];
    for (int i = threadIdx.x; i < kBins; i += kPlanBlock) h[i] = 0;
    float lim = 0.0f;
    if (pa.chain) {
        reset_ring(pa);
        lim = plan_lim(pa, plan_cells(pa, 0, pa.n_pairs));
        if (threadIdx.x == 0) plan_waves(pa, lim);
    }
    __syncthreads();
    plan_count(pa, 0, pa.n_pairs, lim, h);
    __syncthreads();
    plan_scan(pa, h);
    __syncthreads();
    plan_scatter(pa, 0, pa.n_pairs, lim, nullptr, h);
}

static hipError_t run_plan(const PlanArgs &pa, hipStream_t stream) {
    const int64_t n_pairs = pa.n_pairs;
    if (n_pairs <= kPlanSmall) {
        hipLaunchKernelGGL(k_plan_small, dim3(1), dim3(kPlanBlock), 0, stream, pa);
        return hipGetLastError();
    }
    const int64_t g64 = (n_pairs + kPlanBlock - 1) / kPlanBlock;
    const unsigned g = (unsigned)(g64 < kPlanGrid ? g64 : kPlanGrid);
    static_assert(kPlanGrid <= kPlanBlock && kBins <= kPlanBlock * (kPlanSmall / kPlanBlock), "start kernel covers both");
    const unsigned g0 = pa.chain ? g : (kBins + kPlanBlock - 1) / kPlanBlock;   // without a queue it only clears the bins
    hipLaunchKernelGGL(k_plan_start, dim3(g0), dim3(kPlanBlock), 0, stream, pa);
    hipLaunchKernelGGL(k_plan_count, dim3(g), dim3(kPlanBlock), 0, stream, pa);
    hipLaunchKernelGGL(k_plan_scan, dim3(1), dim3(64 * kNumRoutes), 0, stream, pa);
    hipLaunchKernelGGL(k_plan_scatter, dim3(g), dim3(kPlanBlock), 0, stream, pa);
    return hipGetLastError();
}

// One item's share of the batch, in what every resident wave would get.  On
// the 4,096-pair batch 0.91 ms (1.08 at half the share, 0.97 at twice), the
// 10,000-pair uneven batch with starts 10.7 ms (11.8, 12.4).
constexpr float kItemShare = 1.0f;

hipError_t launch_plan(const PairArrays &a, int64_t n_pairs, const LaunchCfg &cfg, const PlanScratch &s,
                       const SweepScratch *sw, hipStream_t stream) {
    PlanArgs pa{};
    pa.a = a;
    pa.n_pairs = n_pairs;
    pa.buckets = cfg.persistent ? kBuckets : 1;
    pa.extend = a.rows != nullptr;
    pa.single_max = cfg.single_max;
    pa.chain = cfg.chain;
    pa.few = cfg.sweep_few;
    pa.chain_route = kRouteSingleLo;
    pa.lim_scale = kItemShare / (64.0f * (float)(cfg.sweep_share > 0 ? cfg.sweep_share : 1));
    pa.s = s;
    if (cfg.chain) pa.sw = *sw;
    pa.band = nullptr;
    return run_plan(pa, stream);
}

hipError_t launch_path_plan(const PathArgs &path, int share, const PlanScratch &s, const SweepScratch &sw,
                            hipStream_t stream) {
    PlanArgs pa{};
    pa.n_pairs = path.n_pairs;
    pa.buckets = kBuckets;
    pa.chain = 1;
    pa.chain_route = kRouteSingleLo;
    pa.lim_scale = kItemShare / (64.0f * (float)share);
    pa.s = s;
    pa.sw = sw;
    pa.paths = 1;
    pa.path = path;
    return run_plan(pa, stream);
}

hipError_t launch_band_plan(const PairArrays &a, const int32_t *band, int64_t n_pairs, const PlanScratch &s,
                            const SweepScratch *sw, int grid, hipStream_t stream) {
    PlanArgs pa{};
    pa.a = a;
    pa.n_pairs = n_pairs;
    pa.buckets = kBuckets;
    pa.extend = 0;
    pa.s = s;
    pa.band = band;
    if (sw) {
        pa.chain = 1;
        pa.chain_route = 3;
        pa.sw = *sw;
        pa.lim_scale = kItemShare / (64.0f * (float)grid);
    }
    return run_plan(pa, stream);
}

// ---- alignment start -------------------------------------------------------------

// The reverse pass aligns the reversed query against the reversed region
// prefix r[0 .. end]: end + 1 levels (none for a pair without an end).
__global__ void k_span_prep(const int32_t *__restrict__ end, int64_t n_pairs, int32_t *__restrict__ rev_len) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n_pairs) rev_len[p] = end[p] >= 0 ? end[p] + 1 : 0;
}

// Starts from the reverse pass's best ends (smallest on ties).
__global__ void k_span_finish(const int32_t *__restrict__ end, const int32_t *__restrict__ rev_end, int64_t n_pairs,
                              int32_t *__restrict__ out_start) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n_pairs) out_start[p] = span_start(end[p], rev_end[p]);
}

hipError_t launch_span_prep(const int32_t *end, int64_t n_pairs, int32_t *rev_len, hipStream_t stream) {
    const unsigned g = (unsigned)((n_pairs + 255) / 256);
    hipLaunchKernelGGL(k_span_prep, dim3(g), dim3(256), 0, stream, end, n_pairs, rev_len);
    return hipGetLastError();
}

hipError_t launch_span_finish(const int32_t *end, const int32_t *rev_end, int64_t n_pairs, int32_t *out_start,
                              hipStream_t stream) {
    const unsigned g = (unsigned)((n_pairs + 255) / 256);
    hipLaunchKernelGGL(k_span_finish, dim3(g), dim3(256), 0, stream, end, rev_end, n_pairs, out_start);
    return hipGetLastError();
}

// ---- mapping decision (Sec. 2.3) ----------------------------------------------

// One wave per read.  Score = B_Match * N_Read - C_DTW; the highest wins,
// the smallest candidate index on ties.  Anchored chains count the events
// each chain aligns.  A NaN cost (the sentinel of a pair that was not
// aligned: invalid slice, unsupported shape) is no candidate at all, so it
// can neither win nor block a later candidate.  Lane l scans candidates l,
// l + 64, ... in order and keeps its first highest; the wave then keeps the
// highest score and, among equal scores, the smallest index.  With B_Match
// finite (checked by every entry point) no score is NaN, so this is the
// candidate a sequential first-highest scan picks.
__global__ __launch_bounds__(256) void k_decide(const float *__restrict__ score, int64_t n_pairs,
                                                const int64_t *__restrict__ cand_off,
                                                const int32_t *__restrict__ cand_cnt,
                                                const int32_t *__restrict__ n_events, int64_t n_reads,
                                                double b_match, double threshold, int32_t *out_best,
                                                double *out_score, uint8_t *out_mapped, bool per_candidate) {
    const int lane = __lane_id();
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; k < n_reads; k += waves) {
        const int64_t p0 = cand_off[k];   // wave-uniform from here on
        const int cnt = cand_cnt[k];
        if (cnt < 0 || p0 < 0 || p0 + cnt > n_pairs) {   // candidate range outside the score array
            if (lane == 0) {
                out_best[k] = -2;
                out_score[k] = __builtin_nan("");
                out_mapped[k] = 0;
            }
            continue;
        }
        const double bonus = per_candidate ? 0.0 : b_match * (double)n_events[k];
        int32_t best = -1;
        double bs = -__builtin_inf();
        for (int c = lane; c < cnt; c += 64) {
            const float cost = score[p0 + c];
            if (cost != cost) continue;
            const double s = (per_candidate ? b_match * (double)n_events[p0 + c] : bonus) - (double)cost;
            if (best < 0 || s > bs) {
                best = (int32_t)(p0 + c);
                bs = s;
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const double os = __shfl_xor(bs, off, 64);
            const int32_t ob = __shfl_xor(best, off, 64);
            if (ob >= 0 && (best < 0 || os > bs || (os == bs && ob < best))) {
                best = ob;
                bs = os;
            }
        }
        if (lane == 0) {
            out_best[k] = best;
            out_score[k] = bs;
            out_mapped[k] = (best >= 0 && bs >= threshold) ? 1 : 0;
        }
    }
}

hipError_t launch_decide(const float *score, int64_t n_pairs, const int64_t *cand_off, const int32_t *cand_cnt,
                         const int32_t *n_events, int64_t n_reads, double b_match, double threshold,
                         int32_t *out_best, double *out_score, uint8_t *out_mapped, bool per_candidate,
                         hipStream_t stream) {
    // four waves (one read each at a time) per workgroup
    const int64_t g64 = (n_reads + 3) / 4;
    const unsigned g = (unsigned)(g64 < (1 << 20) ? g64 : (1 << 20));
    hipLaunchKernelGGL(k_decide, dim3(g), dim3(256), 0, stream, score, n_pairs, cand_off, cand_cnt, n_events,
                       n_reads, b_match, threshold, out_best, out_score, out_mapped, per_candidate);
    return hipGetLastError();
}

}  // namespace ra
