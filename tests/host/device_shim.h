// Enough of the device's intrinsics to compile the chained queue's protocol
// (csrc/dtw_chain.h) for one host thread that plays a wave of one lane.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

static uint64_t shim_clock;
static uint64_t shim_tick = 1;   // clock units per look at it

template <class T>
inline T shim_load(T *p) { return *p; }
template <class T, class V>
inline void shim_store(T *p, V v) { *p = (T)v; }

#define __hip_atomic_load(p, order, scope) shim_load(p)
#define __hip_atomic_store(p, v, order, scope) shim_store(p, v)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_s_memrealtime() (shim_clock += shim_tick)
#define __builtin_amdgcn_s_sleep(x) ((void)0)
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_update_dpp(o, s, c, r, b, z) (s)
#define __builtin_amdgcn_make_buffer_rsrc(p, s, n, f) ((void *)(p))
#define __builtin_amdgcn_raw_buffer_load_b32(r, v, s, a) (0)
typedef void *__amdgpu_buffer_rsrc_t;
inline int __lane_id() { return 0; }
inline uint64_t __ballot(bool x) { return x; }
template <class T>
inline T __shfl(T v, int, int) { return v; }
template <class T>
inline T __shfl_xor(T v, int, int) { return v; }
static dim3 blockIdx, gridDim;
inline int atomicAdd(int32_t *p, int v) {
    const int x = *p;
    *p += v;
    return x;
}
