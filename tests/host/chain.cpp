// The chained queue's slots (csrc/dtw_chain.h), played by one host thread.
#include "device_shim.h"

#include "dtw_chain.h"
#include "dtw_path.h"

extern "C" {

// Item t (item i of `items`) asks for its slots in a ring of which done[] has
// come this far; 1 if it goes on.  *failed: a wait has been given up.
int open_slots(int ring_slots, int *done, int *failed, int t, int i, int items) {
    ra::SweepScratch sw{};
    sw.ring_slots = ring_slots;
    sw.done = done;
    sw.failed = failed;
    shim_tick = ra::kSpinTicks;
    return ra::open_slots(sw, t, {0, 1, 1, i, items});
}

int path_lost(int n, int L, float lim, int failed) { return ra::path_lost(n, L, lim, failed != 0); }
}
