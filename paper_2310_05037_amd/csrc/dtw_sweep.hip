// dtw_sweep.hip -- the stripe sweep: the pairs of the batch, streaming,
// start-of-alignment and early-termination calls.
//
// A region is cut into S stripes of 64 C columns (C <= 32 per lane).  One
// wave sweeps one stripe over all query rows, lane-striped and skewed: lane k
// owns C consecutive columns and at step t computes rows 2(t-k) and
// 2(t-k)+1 (rows2 in dtw_rows.h).  The values a lane needs from its left
// neighbour (two query events, two west values) arrive with four DPP
// wave_shr:1 moves per step; lane 0 gets them from a 64-row block in LDS, one
// broadcast ds_read_b128 per step, read a step ahead.  Lane 63's last column
// goes to LDS and leaves the wave as one coalesced 256-byte store per block.
// A block costs the wave about 110 instructions; a step costs 6 C + 12 vector
// instructions and about ten others.
//
// A work item is one stripe of a long pair or one whole short pair.  The
// planner lists the stripes of a pair one after another, pairs longest first,
// and resident waves take items in that order.  Stripe s reads the edge column
// of stripe s - 1 while that is still being swept by another wave anywhere on
// the chip, about 190 rows behind it, so a batch is spread over the chip
// whether it has ten pairs or a hundred thousand: with one wave per pair a
// batch took as long as its largest pair (start-of-alignment of 10,000 pairs:
// 52 ms, now 10.5; 1,024 regions of 20,000 levels: 28, now 14.7).  How the
// columns travel: dtw_chain.h.  An item that costs less than its share of the
// batch takes all of its pair's stripes, edges through the wave's own column.
//
// What bounds it: instruction issue.  3.5 vector instructions per cell, a SIMD
// issuing one in 2.2 cycles at most: 50.3 to 52.5 ms for 100,000 uneven pairs
// (0.96 T cells, 18.2 to 19.0 T cells/s; 55 before), memory far from busy.  Few or short pairs
// wait for one wave's chain of dependent instructions instead.
#include "dtw_chain.h"
#include "dtw_rows.h"

namespace ra {

// Per-wave LDS: 64 rows of (query event, west value) for lane 0, lane 63's
// last column of 64 rows, and room for the other lanes' writes beside it (no
// execution-mask change per step).
struct WaveBuf {
    float feed[(64 + 2) * 2];   // (a step reads one pair of rows ahead)
    float out[64];
    float sink[63 * 2 + 64];
};

// A stripe and where its edge columns are.  Between items they go through the
// ring (chain_in, chain_out), within one through the wave's own column.
struct Stripe {
    int s;
    bool ein, eout;             // there is a stripe to the left, to the right
    bool chain_in, chain_out;
    const float *in;
    float *out;
    int block;                  // steps per block, a multiple of 4 up to 32
    float corner;               // within an item: D(-1, last column of stripe s - 1)
    int32_t *failed;            // a wave has given up
};

// One stripe of a pair.  best / bj: the minimum of the pair's last row so far,
// with this stripe's on return; between items they travel behind the edge
// column.  False when a wait was given up.
template <int C, bool EXT>
RA_DEV bool sweep_stripe(const PairView &pv, Stripe &it, WaveBuf *wb, float &best, int &bj) {
    const int lane = opaque_lane();
    const int n = pv.n;
    const int col0 = (it.s * 64 + lane) * C;
    const bool chain_in = it.chain_in, chain_out = it.chain_out;
    float rv[C], A[C];
    bool ok = true;
    {
        float B[C];
        load_lane<C, EXT>(pv, col0, rv, A, B);
    }
    // In the ring, element 0 of an edge column is the corner D(-1, last
    // column), the rows follow.
    if (chain_out && lane == 63) store_agent(it.out, stored(A[C - 1]));
    float corner = pv.corner ? 0.0f : kInf;   // left of the region: see load_lane
    const int nm1 = n - 1;
    float qn, en;   // the next block's rows, one per lane
    if (chain_in) {
        corner = load_agent(it.in);
        ok = take(it.in, it.failed, 0, lane == 0, corner);
    } else if (it.ein) {
        corner = it.corner;
    }
    it.corner = __shfl(A[C - 1], 63, 64);
    // Where there is no stripe to the left the loads below go to q and their
    // values to nothing: a block's data moves without branches, of which a
    // lone wave takes one in about 50 cycles.
    const float *const in = it.ein ? it.in + (chain_in ? 1 : 0) : pv.q;
    float *const out = it.out + (chain_out ? 1 : 0);
    auto fetch = [&](int row0) {
        const int row = row0 + lane < n ? row0 + lane : nm1;
        qn = pv.q[pv.reverse ? nm1 - row : row];
        en = load_agent(in + row);
    };
    if (n > 0) {
        fetch(0);
        float xl = 0.0f;
        typedef float quad __attribute__((ext_vector_type(4)));
        const quad *feed = reinterpret_cast<const quad *>(wb->feed);
        // (event, west) of the two rows of the previous step (P) and of this one
        quad P{0.0f, kInf, 0.0f, corner}, Q;
        float *const mine = lane == 63 ? wb->out : wb->sink + 2 * lane;
        typedef float pairf __attribute__((ext_vector_type(2)));
        const int steps = (n + 1) / 2 + 63;
        const bool odd = (n & 1) != 0;
        const int block = it.block;
        const bool in_block = lane < 2 * block;   // this lane moves a row of each block
        const bool sends = it.eout && in_block, takes = chain_in && in_block;
        // The block that ended at step t0 brought lane 63's rows from 2 t0 -
        // 2 block - 126 on, two a step.  They leave after the next block's
        // rows have come in (see arrived).
        auto flush = [&](int t0) {
            const int row = 2 * (t0 - block) - 126 + lane;
            const float v = stored(wb->out[lane]);
            if (sends && (unsigned)row < (unsigned)n) store_agent(out + row, v);
        };
        int t0 = 0;
        for (; t0 < steps; t0 += block) {
            const int row0 = 2 * t0;
            arrived(qn);
            arrived(en);
            ok = take(in, it.failed, row0 + lane, takes && ok && row0 + lane < n, en) && ok;
            reinterpret_cast<pairf *>(wb->feed)[lane] = pairf{qn, it.ein ? en : kInf};
            flush(t0);
            fetch(row0 + 2 * block);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            Q = feed[0];
            // Lanes before their first row or after their last keep their
            // registers as they are.  The last row of an odd query is swept
            // in the second loop's blocks, which follow the first loop's.
            const int plain = odd && row0 + 2 * block >= n ? 0 : block;
            const quad *f = feed + 1;
            pairf *o = reinterpret_cast<pairf *>(mine);
            int x = row0 - 2 * lane;
#define RA_STEP(P, Q, u, ODD)                                                                        \
    {                                                                                                \
        const float q0 = dpp_shr1(Q[0], P[0]), q1 = dpp_shr1(Q[2], P[2]);                            \
        const float w0 = dpp_shr1(Q[1], xl), w1 = dpp_shr1(Q[3], A[C - 1]);                          \
        const float nw = P[3];                                                                       \
        P = f[u];                                                                                    \
        if ((unsigned)(x + 2 * u) < (unsigned)n)                                                     \
            rows2<C, ODD>(x + 2 * u < nm1, q0, q1, nw, w0, w1, rv, A, xl);                           \
        Q = quad{q0, w0, q1, w1};                                                                    \
        o[u] = pairf{xl, A[C - 1]};                                                                  \
    }
            // Four steps a turn where registers allow it.
#define RA_STEPS(FROM, TO, ODD)                                                                      \
    _Pragma("unroll 1") for (int u = FROM; u < TO; u += U, f += U, o += U, x += 2 * U) {             \
        RA_STEP(P, Q, 0, ODD)                                                                        \
        RA_STEP(Q, P, 1, ODD)                                                                        \
        if constexpr (U == 4) {                                                                      \
            RA_STEP(P, Q, 2, ODD)                                                                    \
            RA_STEP(Q, P, 3, ODD)                                                                    \
        }                                                                                            \
    }
            constexpr int U = C <= 8 ? 4 : 2;
            RA_STEPS(0, plain, false)
            RA_STEPS(plain, block, true)
#undef RA_STEPS
#undef RA_STEP
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        flush(t0);
    }
    float b;
    int j;
    finish_lane<C, EXT>(pv, col0, A, b, j);
    wave_min(b, j);
    if (chain_in) {   // the items to the left: their minimum is behind the rows
        float v = lane < 2 ? load_agent(in + n + lane) : 0.0f;
        if (ok) ok = take(in, it.failed, n + lane, lane < 2, v);
        take_min(b, j, __shfl(v, 0, 64), __builtin_bit_cast(int, __shfl(v, 1, 64)));
    }
    take_min(best, bj, b, j);
    if (chain_out && lane < 2) store_agent(out + n + lane, lane == 0 ? stored(best) : __builtin_bit_cast(float, bj));
    return ok;
}

// Columns per lane 1 .. kSweepMaxC, halving.
template <int LO, int HI, bool EXT>
RA_DEV bool sweep_dispatch(int c, const PairView &pv, Stripe &it, WaveBuf *wb, float &best, int &bj) {
    if constexpr (LO == HI) {
        return sweep_stripe<LO, EXT>(pv, it, wb, best, bj);
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (c <= MID) return sweep_dispatch<LO, MID, EXT>(c, pv, it, wb, best, bj);
        return sweep_dispatch<MID + 1, HI, EXT>(c, pv, it, wb, best, bj);
    }
}

RA_DEV void write_result(const PairArrays &a, int p, float best, int bj) {
    if (__lane_id() == 0) {
        a.out_score[p] = best;
        if (a.out_end) a.out_end[p] = bj;
    }
}

// Stripes [s0, s1) of a pair by one wave.
template <bool EXT>
RA_DEV bool sweep_item(int c, const PairView &pv, int s0, int s1, Stripe &it, const float *in, float *out, float *own,
                       WaveBuf *wb, float &best, int &bj) {
    bool ok = true;
    const bool last = (s1 - 1) * 64 * c + 64 * c >= pv.m;   // the item ends with the region
    for (int s = s0; s < s1; ++s) {
        it.s = s;
        it.ein = s > 0;
        it.eout = s + 1 < s1 || !last;
        it.chain_in = s == s0 && s > 0;
        it.chain_out = s + 1 == s1 && !last;
        it.in = it.chain_in ? in : own;
        it.out = it.chain_out ? out : own;
        ok = sweep_dispatch<1, kSweepMaxC, EXT>(c, pv, it, wb, best, bj) && ok;
        stores_done();   // before the next stripe's loads
    }
    return ok;
}

// Five waves per SIMD: 96 VGPRs.
template <bool EXT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kSweepWaves, kSweepWaves)))
void k_sweep(PairArrays a, SweepScratch sw) {
    __shared__ __align__(16) WaveBuf wb;
    const int n_items = *sw.n_items;
    if ((int)blockIdx.x >= sw.n_items[2]) return;   // more waves than are of use
    for (int t = next_item(sw.queue); t < n_items; t = next_item(sw.queue)) {
        const ItemCode x = load_item(sw, t);
        const bool last = x.i + 1 == x.items;
        bool ok = open_slots(sw, t, x);
        float best = kInf;
        int bj = 0x7fffffff;
        if (ok) {
            const PairView pv = pair_view<EXT>(a, x.p);
            const int S = (pv.m + 64 * x.c - 1) / (64 * x.c);
            const int s0 = x.i * x.k, s1 = s0 + x.k < S ? s0 + x.k : S;
            Stripe it;
            it.failed = sw.failed;
            // Few items: short blocks, so that an item trails its left
            // neighbour by about 96 steps instead of 160.
            it.block = n_items * 4 <= kLoneItems ? 16 : 32;
            it.corner = 0.0f;
            ok = sweep_item<EXT>(x.c, pv, s0, s1 > s0 ? s1 : s0 + 1, it, slot_of(sw, t - 1), slot_of(sw, t),
                                 sw.own + (size_t)blockIdx.x * kOwnFloats, &wb, best, bj);
            // (every kEmpty is back: sweep_item waits for its stores)
            if (x.i > 0) slot_done(sw, t - 1);
        }
        // After a wait that was given up anywhere no pair of several items is trusted.
        if (last) {
            if (!ok || (x.items > 1 && gave_up(sw))) {
                best = __builtin_nanf("");
                bj = kGaveUp;
            }
            write_result(a, x.p, best, bj);
        }
    }
}

hipError_t launch_sweep(const PairArrays &a, int grid, const SweepScratch &sw, hipStream_t stream) {
    if (a.rows)
        hipLaunchKernelGGL(k_sweep<true>, dim3((unsigned)grid), dim3(64), 0, stream, a, sw);
    else
        hipLaunchKernelGGL(k_sweep<false>, dim3((unsigned)grid), dim3(64), 0, stream, a, sw);
    return hipGetLastError();
}

template <class K>
static int occupancy(K kernel) {
    int nb = 0;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, 64, 0);
    return nb > 0 ? nb : 1;
}

int sweep_blocks_per_cu(bool extend) {
    static const int plain = occupancy(k_sweep<false>), ext = occupancy(k_sweep<true>);
    return extend ? ext : plain;
}

}  // namespace ra
