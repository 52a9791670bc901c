// dtw_bnb.hip -- early termination of hopeless candidates (branch and bound).
//
// RawAlign outputs at most one mapping per read and prunes DTW work that
// cannot beat the best candidate found so far; candidates are visited in
// chaining-score order so that a good one comes first (Sec. 2.4.1).  Here the
// call aligns in rounds, each a streaming extension of its pairs' resident
// rows by the stripe sweep (dtw_sweep.hip), whose items spread every round
// over the chip however uneven its pairs are:
//   * round 0: every read's first candidate (and pairs no single read owns),
//     whole, and the first block_rows events of the others, which nothing can
//     drop earlier;
//   * the later rounds: the pairs still open, each up to the row where, its
//     minimum growing on as it has, it is dropped; in the last one whole.
// After a round that ended at row i the sweep knows min_j D(i, j); every path
// reaches row n-1 through row i and costs never decrease along a path (each
// cell adds |q - r| >= 0), so C_DTW >= min_j D(i, j) and the pair's Score is
// at most B_Match * N_Read - min_j D(i, j).  When that is strictly below the
// best Score its read has reached so far the pair cannot win (nor tie) and is
// dropped; a pair that completes raises its read's best.  The best only grows,
// so every drop is justified by the final best: the read's decision (argmax
// Score, smallest index on ties, threshold) is the one of the full
// computation.  Between the rounds: two small kernels and the planner.
//
// A persistent kernel with one wave per pair, which did all of this in one
// launch, took as long as its largest first candidate: 31 ms for 20,000 pairs
// of the uneven batch.
#include "dtw_bnb.h"
#include "dtw_device.h"

namespace ra {

// Pair checks: the same rules as the batch entry point (slices inside q and
// r, region and query limits) plus the row slot and the caller's longest
// query.
RA_DEV bool bnb_valid(const BnbArgs &b, int64_t p) {
    const PairArrays &a = b.a;
    const int n = a.q_len[p];
    const int m = a.r_len[p];
    const int64_t qo = a.q_off[p];
    const int64_t ro = a.r_off[p];
    const int64_t wo = a.row_off[p];
    return n >= 0 && m >= 0 && qo >= 0 && ro >= 0 && qo + n <= a.q_size && ro + m <= a.r_size &&
           m <= kMaxRegion && n <= kMaxQuery && (m <= kSingleMaxRegion || n <= kEdgeCap) && n <= b.max_query &&
           wo >= 0 && wo + m <= a.rows_size;
}

__global__ void k_bnb_clear(BnbArgs b) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < b.n_pairs) {
        b.s.read_of[p] = -1;
        b.s.status[p] = kBnbWaiting;
    }
    if (p < b.n_reads) b.s.best[p] = order_key(-__builtin_inf());
}

// Read of every pair, through the reads' candidate ranges.
__global__ void k_bnb_claim(BnbArgs b) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= b.n_reads) return;
    const int64_t p0 = b.cand_off[k];
    const int cnt = b.cand_cnt[k];
    if (cnt <= 0 || p0 < 0 || p0 + cnt > b.n_pairs) return;   // rawalign_decide flags such reads
    for (int c = 0; c < cnt; ++c) {
        // A pair claimed by two reads is never pruned (it has no single bound).
        if (atomicCAS(&b.s.read_of[p0 + c], -1, (int32_t)k) != -1) atomicExch(&b.s.read_of[p0 + c], -2);
    }
    b.s.status[p0] = kBnbFirst;
}

// Round 0, and the results of pairs that need no DTW.
__global__ void k_bnb_start(BnbArgs b, int block_rows) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= b.n_pairs) return;
    const PairArrays &a = b.a;
    float sc = 0.0f;
    int e = -1;
    bool settled = true;
    if (!bnb_valid(b, p)) {
        sc = __builtin_nanf("");
        e = -2;
    } else if (a.q_len[p] != 0) {
        sc = kInf;
        settled = a.r_len[p] == 0;
    }
    if (settled) {
        a.out_score[p] = sc;
        a.out_end[p] = e;
        b.s.status[p] = kBnbDone;
    }
    const bool whole = b.s.status[p] == kBnbFirst || b.s.read_of[p] < 0 || a.q_len[p] < block_rows;
    bnb_part(b, p, settled ? -1 : 0, whole ? a.q_len[p] : block_rows);
}

__global__ void k_bnb_finish(BnbArgs b) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= b.n_pairs) return;
    uint64_t key;
    const int k = bnb_finish(b, p, key);
    if (k >= 0) atomicMax((unsigned long long *)&b.s.best[k], (unsigned long long)key);
}

__global__ void k_bnb_advance(BnbArgs b, int block_rows, bool whole) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < b.n_pairs) bnb_advance(b, p, block_rows, whole);
}

static unsigned grid_of(int64_t n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_bnb_start(const BnbArgs &b, int block_rows, hipStream_t stream) {
    const int64_t mx = b.n_pairs > b.n_reads ? b.n_pairs : b.n_reads;
    hipLaunchKernelGGL(k_bnb_clear, dim3(grid_of(mx)), dim3(256), 0, stream, b);
    if (b.n_reads > 0) hipLaunchKernelGGL(k_bnb_claim, dim3(grid_of(b.n_reads)), dim3(256), 0, stream, b);
    hipLaunchKernelGGL(k_bnb_start, dim3(grid_of(b.n_pairs)), dim3(256), 0, stream, b, block_rows);
    return hipGetLastError();
}

hipError_t launch_bnb_next(const BnbArgs &b, int block_rows, int left, hipStream_t stream) {
    hipLaunchKernelGGL(k_bnb_finish, dim3(grid_of(b.n_pairs)), dim3(256), 0, stream, b);
    if (left > 0)
        hipLaunchKernelGGL(k_bnb_advance, dim3(grid_of(b.n_pairs)), dim3(256), 0, stream, b, block_rows, left == 1);
    return hipGetLastError();
}

}  // namespace ra
