// A recording HIP runtime and kernel launchers under the C ABI
// (csrc/rawalign_abi.cpp), so that its host side (scratch, routes, captures)
// runs without a GPU.  Device memory is addresses only.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <set>
#include <string>

#include "dtw_path.h"
#include "internal.h"

namespace {

struct State {
    std::map<uintptr_t, size_t> live;       // allocations
    std::set<uintptr_t> captured;           // buffers that captured launches use
    uintptr_t next = 1 << 20;
    size_t limit = ~(size_t)0, held = 0, largest = ~(size_t)0;
    int streams = 0;
    int last_sweep = 0;                     // its grid
    bool capturing = false;
    hipError_t last = hipSuccess;
    std::string log, bad;
} g;

void note(const std::string &s) { g.log += s + "\n"; }
void wrong(const std::string &s) { g.bad += s + "\n"; }
std::string str(long long v) { return std::to_string(v); }

// A launch uses `bytes` at p: allocated, and remembered while capturing.
void use(const char *what, const void *p, size_t bytes) {
    if (bytes == 0) return;
    auto it = g.live.upper_bound((uintptr_t)p);
    if (it == g.live.begin()) return wrong(std::string(what) + " is not allocated");
    --it;
    if ((uintptr_t)p + bytes > it->first + it->second)
        return wrong(std::string(what) + ": " + str(bytes) + " bytes of " + str(it->first + it->second - (uintptr_t)p));
    if (g.capturing) g.captured.insert(it->first);
}

void use_plan(const ra::PlanScratch &s, int64_t n_pairs) {
    use("hist", s.hist, sizeof(int32_t) * (ra::kNumRoutes * ra::kBuckets + 2 * ra::kNumRoutes));
    if (n_pairs > s.capacity) wrong("list capacity");
    use("list", s.list, sizeof(int32_t) * ra::kNumRoutes * s.capacity);
}

void use_sweep(const ra::SweepScratch &sw, int grid, bool own) {
    if (grid < ra::kCover) wrong("a chained launch of " + str(grid) + " workgroups");
    use("items", sw.items, sizeof(uint64_t) * sw.item_cap);
    use("ring", sw.ring, sizeof(float) * (size_t)sw.ring_slots * ra::kSlotFloats);
    if (sw.ring_slots < 2) wrong("ring slots");
    use("failure flag", sw.failed, sizeof(int32_t));
    auto ring = --g.live.upper_bound((uintptr_t)sw.ring), flag = --g.live.upper_bound((uintptr_t)sw.failed);
    if (ring != flag || (uintptr_t)sw.failed < (uintptr_t)(sw.ring + (size_t)sw.ring_slots * ra::kSlotFloats))
        wrong("the failure flag is not beside its ring");
    if (own) use("own columns", sw.own, sizeof(float) * (size_t)grid * ra::kOwnFloats);
    use("done", sw.done, sizeof(int32_t) * sw.ring_slots);
    use("queue", sw.queue, sizeof(int32_t) * ra::kQueues * ra::kQueueStride);
    use("partial", sw.partial, sizeof(double) * ra::kPlanGrid);
}

}  // namespace

// ---- the runtime --------------------------------------------------------------------

extern "C" {

hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    std::strcpy(p->name, "host");
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipGetLastError() {
    const hipError_t e = g.last;
    g.last = hipSuccess;
    return e;
}
hipError_t hipMalloc(void **p, size_t bytes) {
    if (g.capturing) {
        wrong("hipMalloc of " + str(bytes) + " in a capture");
        return g.last = hipErrorStreamCaptureUnsupported;
    }
    if (g.held + bytes > g.limit || bytes > g.largest) {
        note("refused " + str(bytes));
        return g.last = hipErrorOutOfMemory;
    }
    *p = (void *)g.next;
    g.live[g.next] = bytes;
    g.next += (bytes + 4095) / 4096 * 4096 + 4096;
    g.held += bytes;
    note("malloc " + str(bytes));
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (g.capturing) wrong("hipFree in a capture");
    auto it = g.live.find((uintptr_t)p);
    if (it == g.live.end()) {
        wrong("hipFree of an unknown address");
        return hipErrorInvalidValue;
    }
    if (g.captured.count(it->first)) wrong("hipFree of " + str(it->second) + " bytes that a captured graph uses");
    g.held -= it->second;
    g.live.erase(it);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int, size_t bytes, hipStream_t) {
    if (g.capturing) wrong("hipMemsetAsync in a capture");
    use("memset", p, bytes);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = g.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    if (g.capturing) wrong("hipStreamCreate in a capture");
    *s = (hipStream_t)(uintptr_t)(100 + g.streams++);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    if (g.capturing) wrong("hipEventCreate in a capture");
    *e = (hipEvent_t)(uintptr_t)1;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
// A sweep is the faster the fewer its waves, the anti-diagonal kernel slow.
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = g.last_sweep ? 1e-3f * g.last_sweep : 100.0f, hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }

// ---- for the tests ------------------------------------------------------------------

void mock_capture(int on) { g.capturing = on != 0; }
// Device memory in all (beyond what is held now), and the largest one allocation may be.
void mock_limit(long long more, long long largest) {
    g.limit = more < 0 ? ~(size_t)0 : g.held + (size_t)more;
    g.largest = largest < 0 ? ~(size_t)0 : (size_t)largest;
}
long long mock_held() { return (long long)g.held; }
// What happened and what was wrong since the last call.
const char *mock_log() {
    static std::string out;
    out.swap(g.log);
    g.log.clear();
    return out.c_str();
}
const char *mock_bad() {
    static std::string out;
    out.swap(g.bad);
    g.bad.clear();
    return out.c_str();
}
}

// ---- the launchers ------------------------------------------------------------------

namespace ra {

static hipError_t launched() { return hipGetLastError(); }   // as the launchers end

hipError_t launch_plan(const PairArrays &, int64_t n_pairs, const LaunchCfg &cfg, const PlanScratch &s,
                       const SweepScratch *sw, hipStream_t) {
    note(std::string("plan") + (cfg.chain ? " chain few=" + str(cfg.sweep_few) : ""));
    use_plan(s, n_pairs);
    if (cfg.chain) use_sweep(*sw, cfg.sweep_grid, false);
    return launched();
}
hipError_t launch_sweep(const PairArrays &a, int grid, const SweepScratch &sw, hipStream_t) {
    note("sweep grid=" + str(grid) + " ring=" + str(sw.ring_slots));
    g.last_sweep = grid;
    use_sweep(sw, grid, std::min<int64_t>(a.r_size, kMaxRegion) > kSweepStripe);
    return launched();
}
hipError_t launch_single_lo(const PairArrays &, int64_t, const LaunchCfg &cfg, const PlanScratch &, hipStream_t) {
    note("lo grid=" + str(cfg.lo_grid));
    return launched();
}
hipError_t launch_single_hi(const PairArrays &, int64_t, const LaunchCfg &cfg, const PlanScratch &, hipStream_t) {
    note("hi grid=" + str(cfg.hi_grid));
    return launched();
}
hipError_t launch_multi(const PairArrays &, int64_t, const LaunchCfg &cfg, const PlanScratch &s, hipStream_t) {
    note("multi grid=" + str(cfg.multi_grid));
    use("edge", s.edge, sizeof(float) * (size_t)cfg.multi_grid * kEdgeCap);
    return launched();
}
hipError_t launch_antidiag(const PairArrays &, int64_t, const LaunchCfg &cfg, const PlanScratch &s, hipStream_t) {
    note("antidiag grid=" + str(cfg.antidiag_grid));
    g.last_sweep = 0;
    use("rows", s.rowbuf, sizeof(float) * (size_t)cfg.antidiag_grid * kMaxRegion);
    return launched();
}
hipError_t launch_bnb_start(const BnbArgs &, int, hipStream_t) { return launched(); }
hipError_t launch_bnb_next(const BnbArgs &, int, int, hipStream_t) { return launched(); }
hipError_t launch_decide(const float *, int64_t, const int64_t *, const int32_t *, const int32_t *, int64_t, double, double,
                         int32_t *, double *, uint8_t *, bool, hipStream_t) {
    return launched();
}
hipError_t launch_tiny_plan(const PairArrays &, int64_t n_pairs, const TinyScratch &t, hipStream_t) {
    use("gaps", t.list, sizeof(TinyRec) * (size_t)n_pairs);
    return launched();
}
hipError_t launch_tiny(const PairArrays &, int64_t, const TinyScratch &, int, const hipStream_t *) { return launched(); }
hipError_t launch_span_prep(const int32_t *, int64_t, int32_t *, hipStream_t) { return launched(); }
hipError_t launch_span_finish(const int32_t *, const int32_t *, int64_t, int32_t *, hipStream_t) { return launched(); }
hipError_t launch_band_plan(const PairArrays &, const int32_t *, int64_t n_pairs, const PlanScratch &s, const SweepScratch *sw,
                            int grid, hipStream_t) {
    note(std::string("band plan") + (sw ? " chain" : ""));
    use_plan(s, n_pairs);
    if (sw) use_sweep(*sw, grid, true);
    return launched();
}
hipError_t launch_band(int cls, const PairArrays &, const int32_t *, int grid, const PlanScratch &s, const SweepScratch *sw,
                       hipStream_t) {
    if (cls == 3) note(std::string("band ") + (sw ? "chain" : "list") + " grid=" + str(grid));
    if (cls == 3 && sw) use_sweep(*sw, grid, true);
    if (cls == 3 && !sw) use("edge", s.edge, sizeof(float) * (size_t)grid * kEdgeCap);
    return launched();
}
hipError_t launch_path_plan(const PathArgs &, int grid, const PlanScratch &s, const SweepScratch &sw, hipStream_t) {
    use_plan(s, 0);
    use_sweep(sw, grid, false);
    return launched();
}
hipError_t launch_path(const PathArgs &, int grid, const SweepScratch &sw, hipStream_t) {
    note(std::string("path ") + (sw.items ? "chain" : "each") + " grid=" + str(grid));
    if (sw.items) use_sweep(sw, grid, false);
    return launched();
}
hipError_t launch_chain_sum(const float *, int64_t, const int64_t *, const int32_t *, int64_t, float *, hipStream_t) {
    return launched();
}
hipError_t noalloc_scratch(int, PlanScratch &) { return hipErrorInvalidValue; }

// As on the device.
int sweep_blocks_per_cu(bool) { return 20; }
int single_lo_blocks_per_cu(bool) { return 16; }
int single_hi_blocks_per_cu(bool) { return 8; }
int multi_blocks_per_cu(bool) { return 16; }
int antidiag_blocks_per_cu() { return 5; }
int path_blocks_per_cu() { return 8; }
int band_blocks_per_cu(int cls) { return cls == 0 ? 32 : 16; }

}  // namespace ra
