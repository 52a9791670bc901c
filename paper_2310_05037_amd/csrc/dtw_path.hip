// dtw_path.hip -- the warping path of each alignment (RawAlign, arXiv
// 2310.05037, Sec. 2.4: the path can be added to the output).
//
// Given an alignment's start s and end e (the start-of-alignment pass), its
// path is an optimal global path from (0, s) to (n-1, e): global DTW of the
// whole query against r[s..e], entered from the corner D(-1, s-1) = 0.
//
// k_path_dirs sweeps the n x L table (L = e - s + 1) in stripes of 64 C
// columns, lane k computing row t - k at step t, query events and west values
// arriving from lane k-1 by DPP and from a block in LDS for lane 0.  Stripes
// are work items of the chained queue (dtw_chain.h, dtw_sweep.hip): with one
// wave per pair the longest of 500 uneven pairs held up the pass, 9.5 ms for
// 2.1 (2 waves a SIMD by their registers, issue-bound).  Every cell also records which neighbour gave
// its minimum, north-west before north before west on ties, as 2 bits.  C is 4,
// 8, 16 or 32, so a lane's codes of a row fill 1 to 8 bytes and the row is one
// bit string, column j at bit 2j, whatever C.  Per cell: v_sub, v_min3, v_add,
// two compares and two selects for the code, and its insertion into the word.
//
// k_path_trace: one wave per pair follows the codes back from (n-1, L-1) to
// (0, 0) and writes, for every query row i, the region columns lo[i] .. hi[i]
// that the path visits (a monotone path covers a contiguous range of every
// row).  Lane k holds 32 columns of row i - k; the walk itself is scalar and
// reads a code with v_readlane, so it waits for memory once in 64 rows or 32
// columns (1.1 ms; one thread per pair, a dependent load per step: 4.5).
#include "dtw_path.h"

#include <type_traits>

#include "dtw_chain.h"

namespace ra {

constexpr int kPathNW = 0, kPathN = 1, kPathW = 2;

// Per-wave LDS: 32 rows of (query event, west value) for lane 0, lane 63's last
// column of 32 rows, and room for the other lanes' writes beside it.
struct PathBuf {
    float feed[64 * 2];
    float out[32];
    float sink[63 + 32];
};
constexpr int kPathBlock = 32;

// One stripe of 64 C columns from column a on.  in / out: edge columns (null at
// the ends).  chain_in: in is a slot of the ring.  Else it is the pair's own
// column and so is out: a row is read at least 64 steps before it is written.
template <int C>
RA_DEV bool path_stripe(const PathArgs &pa, int64_t p, int n, int s, int L, int a, const float *in, bool chain_in,
                        float *out, int32_t *failed, PathBuf *pb) {
    using word = std::conditional_t<C == 4, uint8_t, std::conditional_t<C == 8, uint16_t,
                 std::conditional_t<C == 16, uint32_t, uint64_t>>>;
    const int lane = opaque_lane();
    const float *rp = pa.r + pa.r_off[p] + s;
    const __amdgpu_buffer_rsrc_t rrs = make_rsrc(rp, L);
    const float *qp = pa.q + pa.q_off[p];
    const int col0 = a + lane * C;
    float rv[C], A[C];
#pragma unroll
    for (int v = 0; v < C; ++v) {
        const int j = col0 + v;
        const float lv = bload(rrs, j < L ? j : L - 1);
        rv[v] = j < L ? lv : kInf;
        A[v] = kInf;   // row -1: +inf except the corner D(-1, -1) (first stripe, lane 0)
    }
    char *const rows = reinterpret_cast<char *>(pa.dirs + pa.dir_off[p]) + col0 / 4;
    const int64_t pitch = path_pitch(L);
    // West value of this step (ecur) and of the previous one (eprev): lane
    // k-1's last column of rows i and i-1; for lane 0 column -1 of the stripe:
    // +inf in the first stripe (whose first previous value is the corner, 0),
    // the previous stripe's edge otherwise (row -1: +inf).
    float ecur = in ? kInf : 0.0f, eprev, qv = 0.0f;
    float qn, en;
    const float *const west = in ? in : qp;   // no stripe to the left: loads of no use
    const bool takes = chain_in && lane < kPathBlock, sends = out && lane < kPathBlock;
    auto fetch = [&](int row0) {
        const int row = row0 + lane < n ? row0 + lane : n - 1;
        qn = qp[row];
        en = load_agent(west + row);
    };
    auto flush = [&](int t0) {   // the block that ended at step t0: rows t0 - 32 - 63 and on
        const int row = t0 - kPathBlock - 63 + lane;
        const float v = stored(pb->out[lane & (kPathBlock - 1)]);
        if (sends && (unsigned)row < (unsigned)n) store_agent(out + row, v);
    };
    typedef float pairf __attribute__((ext_vector_type(2)));
    const pairf *feed = reinterpret_cast<const pairf *>(pb->feed);
    float *const mine = lane == 63 ? pb->out : pb->sink + lane;
    bool ok = true;
    fetch(0);
    int t0 = 0;
    for (; t0 < n + 63; t0 += kPathBlock) {
        arrived(qn);
        arrived(en);
        if (chain_in) ok = take(west, failed, t0 + lane, takes && ok && t0 + lane < n, en) && ok;
        reinterpret_cast<pairf *>(pb->feed)[lane] = pairf{qn, in ? en : kInf};
        flush(t0);
        fetch(t0 + kPathBlock);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 2
        for (int u = 0; u < kPathBlock; ++u) {
            const pairf f = feed[u];
            qv = dpp_shr1(f[0], qv);
            eprev = ecur;
            ecur = dpp_shr1(f[1], A[C - 1]);
            const int i = t0 + u - lane;
            const bool valid = (unsigned)i < (unsigned)n;
            float diag = eprev, left = ecur;
            uint64_t code = 0;
#pragma unroll
            for (int v = 0; v < C; ++v) {
                const float up = A[v];
                const float mn = fminf(fminf(diag, up), left);
                const uint32_t c = diag == mn ? kPathNW : (up == mn ? kPathN : kPathW);
                code |= (uint64_t)c << (2 * v);
                const float nv = fabsf(qv - rv[v]) + mn;
                diag = up;
                left = nv;
                A[v] = valid ? nv : A[v];
            }
            if (valid) *reinterpret_cast<word *>(rows + i * pitch) = (word)code;
            mine[u] = A[C - 1];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    flush(t0);
    return ok;
}

template <int C>
RA_DEV bool path_item(const PathArgs &pa, int64_t p, int n, int s, int L, const ItemCode &x, const float *in, float *out,
                      int32_t *failed, PathBuf *pb) {
    if (x.items > 1)   // one stripe, columns through the ring
        return path_stripe<C>(pa, p, n, s, L, x.i * 64 * C, x.i > 0 ? in : nullptr, x.i > 0,
                              x.i + 1 < x.items ? out : nullptr, failed, pb);
    // The whole interval: stripes in turn, columns in the workspace behind the codes.
    float *own = reinterpret_cast<float *>(reinterpret_cast<char *>(pa.dirs + pa.dir_off[p]) + n * path_pitch(L));
    for (int a = 0; a < L; a += 64 * C) {
        (void)path_stripe<C>(pa, p, n, s, L, a, a > 0 ? own : nullptr, false, a + 64 * C < L ? own : nullptr, failed, pb);
        stores_done();
    }
    return true;
}

RA_DEV bool path_dispatch(const PathArgs &pa, const ItemCode &x, int n, int s, int L, const float *in, float *out,
                          int32_t *failed, PathBuf *pb) {
    if (x.c == 4) return path_item<4>(pa, x.p, n, s, L, x, in, out, failed, pb);
    if (x.c == 8) return path_item<8>(pa, x.p, n, s, L, x, in, out, failed, pb);
    if (x.c == 16) return path_item<16>(pa, x.p, n, s, L, x, in, out, failed, pb);
    return path_item<32>(pa, x.p, n, s, L, x, in, out, failed, pb);
}

__global__ __launch_bounds__(64) void k_path_dirs(PathArgs pa, SweepScratch sw) {
    __shared__ __align__(16) PathBuf pb;
    int n = 0, s = 0, L = 0;
    if (!sw.items) {   // no queue: a pair per workgroup
        ItemCode x{(int)blockIdx.x, 0, 1, 0, 1};
        if (path_interval(pa, x.p, n, s, L) != 0) return;
        path_shape(n, L, kInf, x.items, x.c);
        (void)path_dispatch(pa, x, n, s, L, nullptr, nullptr, nullptr, &pb);
        return;
    }
    const int n_items = *sw.n_items;
    if ((int)blockIdx.x >= sw.n_items[2]) return;
    for (int t = next_item(sw.queue); t < n_items; t = next_item(sw.queue)) {
        const ItemCode x = load_item(sw, t);
        bool ok = open_slots(sw, t, x);
        if (ok && path_interval(pa, x.p, n, s, L) == 0) {
            ok = path_dispatch(pa, x, n, s, L, slot_of(sw, t - 1), slot_of(sw, t), sw.failed, &pb);
            stores_done();   // every kEmpty is back
            if (x.i > 0) slot_done(sw, t - 1);
        }
    }
}

// Codes of 32 columns from column jb on: 64 bits at bit 2 jb of the row.
RA_DEV uint64_t path_codes(const char *row, int jb, int words) {
    const uint64_t *w = reinterpret_cast<const uint64_t *>(row);
    const int k = jb >> 5, sh = 2 * (jb & 31);
    const uint64_t lo = w[k], hi = w[k + 1 < words ? k + 1 : k];
    return sh ? lo >> sh | hi << (64 - sh) : lo;
}

// plan, failed: SweepScratch's of the direction pass, null if it had no queue.
__global__ __launch_bounds__(64) void k_path_trace(PathArgs pa, const int32_t *plan, const int32_t *failed) {
    const int lane = __lane_id();
    for (int64_t p = blockIdx.x; p < pa.n_pairs; p += gridDim.x) {
        int n = 0, s = 0, L = 0;
        int st = path_interval(pa, p, n, s, L);
        if (st == 0 && plan && path_lost(n, L, reinterpret_cast<const float *>(plan)[3], *failed != 0)) st = kGaveUp;
        st = __builtin_amdgcn_readfirstlane(st);
        s = __builtin_amdgcn_readfirstlane(s);
        const int64_t off = pa.path_off[p];
        const int rows = pa.q_len[p];
        if (rows <= 0 || off < 0 || off > pa.path_size || rows > pa.path_size - off) continue;
        int32_t *lo = pa.path_lo + off;
        int32_t *hi = pa.path_hi + off;
        if (st != 0) {
            for (int i = lane; i < rows; i += 64) lo[i] = hi[i] = st;
            continue;
        }
        const int64_t pitch = path_pitch(L);
        const int words = (int)(pitch / 8);
        const char *base = reinterpret_cast<const char *>(pa.dirs + pa.dir_off[p]);
        int i = __builtin_amdgcn_readfirstlane(n - 1), j = __builtin_amdgcn_readfirstlane(L - 1);
        int top = s + j;   // hi of the current row
        // Every step lowers i + j; the edges of the table allow only one move
        // (west along row 0, north along column 0), whatever the codes say.
        while (i >= 0) {
            const int i0 = i, jb = j > 31 ? j - 31 : 0;
            const int row = i0 - lane;
            const uint64_t codes = path_codes(base + (row < 0 ? 0 : row) * pitch, jb, words);
            const uint32_t c0 = (uint32_t)codes, c1 = (uint32_t)(codes >> 32);
            int vlo = 0, vhi = 0;
            int r = 0;   // lane of row i
            while (r < 64 && i >= 0 && j >= jb) {
                const uint32_t a0 = (uint32_t)__builtin_amdgcn_readlane((int)c0, r);
                const uint32_t a1 = (uint32_t)__builtin_amdgcn_readlane((int)c1, r);
                const int v = j - jb;
                int d = (int)((v < 16 ? a0 >> (2 * v) : a1 >> (2 * (v - 16))) & 3);
                if (i == 0) d = kPathW;
                else if (j == 0) d = kPathN;
                if (d == kPathW && j > 0) {
                    --j;
                    continue;
                }
                vlo = lane == r ? s + j : vlo;
                vhi = lane == r ? top : vhi;
                if (d == kPathNW) --j;
                --i;
                ++r;
                top = s + j;
            }
            if (lane < r) {
                lo[row] = vlo;
                hi[row] = vhi;
            }
        }
    }
}

int path_blocks_per_cu() {
    int nb = 0;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_path_dirs, 64, 0);
    return nb > 0 ? nb : 1;
}

hipError_t launch_path(const PathArgs &pa, int grid, const SweepScratch &sw, hipStream_t stream) {
    hipLaunchKernelGGL(k_path_dirs, dim3((unsigned)grid), dim3(64), 0, stream, pa, sw);
    const unsigned g = (unsigned)(pa.n_pairs < (1 << 20) ? pa.n_pairs : (1 << 20));
    hipLaunchKernelGGL(k_path_trace, dim3(g), dim3(64), 0, stream, pa, sw.items ? sw.n_items : nullptr,
                       sw.failed);
    return hipGetLastError();
}

}  // namespace ra
