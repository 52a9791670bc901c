// The chained queue's rules (csrc/internal.h), for the host tests.
#include "internal.h"

extern "C" {
int queues() { return ra::kQueues; }
int cover() { return ra::kCover; }
int queue_of(int b) { return ra::queue_of(b, ra::kQueues); }
int live_workgroups(int n_items, int most) { return ra::live_workgroups(n_items, most); }
}
