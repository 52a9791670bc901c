// dtw_chain.h -- edge columns between work items: the ring of slots that the
// stripe sweep and the path and band kernels hand their last columns through.
//
// A batch's items are in one list, those of a pair one after another, and
// item t's edge column is in slot t mod ring.  The values carry their own
// arrival: a slot is filled with kEmpty (a NaN that no cell can produce), the
// producer stores with agent scope, the consumer loads with agent scope until
// nothing in its block is kEmpty, and puts kEmpty back.  No fence, no flag, no
// order between different values is relied on.  A slot is written, and read,
// only after its previous item's consumer has marked it done (one counter per
// slot, cleared by the planner).
//
// Every wait is for an item with a lower number, and every queue has a resident
// wave (queue_of), so the lowest unfinished item is taken, never waits and the
// list drains.  A
// wait is nevertheless capped (kSpinTicks); past the cap every wave stops
// waiting, the cut pairs left are marked as failed and the ring is refilled by
// the next call's planner.
#pragma once

#include "dtw_device.h"

namespace ra {

constexpr uint32_t kEmpty = 0xffffffffu;
constexpr int kLoneItems = 8192;   // up to twice a wave per SIMD
constexpr uint64_t kSpinTicks = 500000000ull;   // 5 s of the constant 100 MHz clock

RA_DEV float load_agent(const float *p) {
    return __hip_atomic_load(const_cast<float *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
RA_DEV void store_agent(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
RA_DEV bool is_empty(float v) { return __builtin_bit_cast(uint32_t, v) == kEmpty; }
// What is stored to a slot is never kEmpty (a caller's own NaN could be).
RA_DEV float stored(float v) { return is_empty(v) ? __builtin_nanf("") : v; }

// One wait of a wave: pauses between polls, gives up past the time cap or
// once any wave of the launch has given up.
struct Patience {
    int32_t *failed;
    uint64_t deadline = 0;
    int polls = 0;
    RA_DEV bool pause() {
        if ((++polls & 63) == 0) {
            if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))
                return false;
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            if (deadline == 0) deadline = now + kSpinTicks;
            else if (now > deadline) {
                if (__lane_id() == 0) __hip_atomic_store(failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return false;
            }
        }
        if (polls < 16) __builtin_amdgcn_s_sleep(1);
        else __builtin_amdgcn_s_sleep(8);
        return true;
    }
};

// Waits for a load here and not at its next use: the counter of outstanding
// memory accesses falls in order, so after a store it would wait for that too
// (0.36 us at agent scope, for each 64-row block).
RA_DEV void arrived(float &v) { asm volatile("" : "+v"(v)); }

// Element ix of a slot for every lane that is `mine`, already loaded once into
// v: loads again until the producer has stored it, then puts kEmpty back.
// False when given up.
RA_DEV bool take(const float *slot, int32_t *failed, int ix, bool mine, float &v) {
    Patience wait{failed};
    while (__ballot(mine && is_empty(v)) != 0) {
        if (!wait.pause()) return false;
        if (mine) v = load_agent(slot + ix);
    }
    arrived(v);
    if (mine) store_agent(const_cast<float *>(slot) + ix, __builtin_bit_cast(float, kEmpty));
    return true;
}

// Item t's slot holds nothing of the items that used it before.
RA_DEV bool slot_free(const SweepScratch &sw, int t) {
    if (t < sw.ring_slots) return true;
    const int32_t *done = sw.done + t % sw.ring_slots;
    const int last = t - sw.ring_slots + 1;
    Patience wait{sw.failed};
    while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(const_cast<int32_t *>(done), __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT)) != last)
        if (!wait.pause()) return false;
    return true;
}

RA_DEV void slot_done(const SweepScratch &sw, int t) {
    if (__lane_id() == 0)
        __hip_atomic_store(sw.done + t % sw.ring_slots, t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workgroup's next item.  Every launch has kCover workgroups and so all
// queues; with the constant in place of `queues` the compiler gives k_sweep's
// loops other registers, which cost 2 to 4 % (1,024 long regions 15.4 ms for 14.8).
RA_DEV int next_item(int32_t *queue) {
    const int queues = (int)gridDim.x < kQueues ? (int)gridDim.x : kQueues;
    const int x = queue_of((int)blockIdx.x, queues);
    int it = 0;
    if (__lane_id() == 0) it = atomicAdd(queue + x * kQueueStride, 1);
    return __builtin_amdgcn_readfirstlane(it) * queues + x;
}

// Item t of the queue.
RA_DEV ItemCode load_item(const SweepScratch &sw, int t) {
    const uint64_t u = sw.items[t];
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return unpack_item(((uint64_t)hi << 32) | lo);
}

// Neither item t's slot nor the one it reads (item i of its pair, i > 0) holds
// anything of their earlier items: an early reader would take their values.  A
// pair's last item, which stores nothing, passes its slot on at once.  False
// when given up, except for a pair that is not cut: it uses no slot.
RA_DEV bool open_slots(const SweepScratch &sw, int t, const ItemCode &x) {
    bool ok = slot_free(sw, t);
    if (x.i > 0 && ok) ok = slot_free(sw, t - 1);
    if (x.i + 1 == x.items) slot_done(sw, t);
    return ok || x.items == 1;
}

RA_DEV float *slot_of(const SweepScratch &sw, int t) {   // t >= -1
    return sw.ring + (size_t)((t + sw.ring_slots) % sw.ring_slots) * kSlotFloats;
}

RA_DEV bool gave_up(const SweepScratch &sw) {
    return __hip_atomic_load(sw.failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// A wave's stores have reached memory.
RA_DEV void stores_done() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

}  // namespace ra
