// dtw_rows.h -- the inner loop of the stripe sweep (dtw_sweep.hip): two query
// rows of a lane's columns at a time, in place.
#pragma once

#include "dtw_device.h"

namespace ra {

// a = |d| + m, one rounded addition, in a's own register.  The register is
// what the asm is for: A stays in place through both branches of the sweep's
// row test, where the compiler otherwise copies it (41 to 180 spilled
// registers at 32 columns).
RA_DEV void add_abs_into(float &a, float d, float m) { asm("v_add_f32 %0, |%1|, %2" : "+v"(a) : "v"(d), "v"(m)); }

// a = yes ? v : u, in a's own register.
RA_DEV void select_into(float &a, bool yes, float u, float v) {
    const uint64_t lanes = __ballot(yes);
    asm("v_cndmask_b32 %0, %1, %2, %3" : "+v"(a) : "v"(u), "v"(v), "s"(lanes));
}

// Rows x (upper) and y = x + 1 of the lane's C columns.  A holds the row
// above x on entry and row y on return; xl receives x's last column.  nw is
// the value north-west of x's first column, w0 and w1 the values west of the
// two rows.
//
// Column c of x is computed beside column c - 1 of y, so A[c-1] can take y
// as soon as x's column c has read the old value: the row needs no second
// buffer, and 2C registers instead of 3C leave room for five waves per SIMD
// at 32 columns per lane (four with double-buffered rows).  The scheduling
// barriers keep the columns in this order.  Left alone, the scheduler pulls
// the subtractions and one of the two chains ahead and needs copies and
// spills; in a loop of this step alone, 256 CUs: 18.4 TCUPS against 16.4 at
// 32 columns and five waves per SIMD, 17.7 against 16.4 at 16 columns and
// eight (13.5 for the double-buffered single-row step at four waves).
//
// ODD: lanes at the last row of an odd query (x = n - 1, `both` false) keep x
// instead of y, one select more per column.
template <int C, bool ODD>
RA_DEV void rows2(bool both, float q0, float q1, float nw, float w0, float w1, const float (&rv)[C], float (&A)[C],
                  float &xl) {
    float xpp = w0, y = w1, above = A[0];
    float xp = fabsf(q0 - rv[0]) + fminf(fminf(nw, above), w0);
    float dy = q1 - rv[0];
    float dx = C > 1 ? q0 - rv[C > 1 ? 1 : 0] : 0.0f;
    auto put = [&](int c, float m) {   // row y (or x) of column c
        if constexpr (ODD) {
            y = fabsf(dy) + m;
            select_into(A[c], both, xp, y);
        } else {
            add_abs_into(A[c], dy, m);
            y = A[c];
        }
    };
#pragma unroll
    for (int c = 1; c < C; ++c) {
        __builtin_amdgcn_sched_barrier(0);
        const float up = A[c];
        const float mx = fminf(fminf(above, up), xp);
        const float my = fminf(fminf(xpp, xp), y);
        const float x = fabsf(dx) + mx;
        if (c + 1 < C) dx = q0 - rv[c + 1 < C ? c + 1 : c];
        put(c - 1, my);
        dy = q1 - rv[c];
        above = up;
        xpp = xp;
        xp = x;
    }
    put(C - 1, fminf(fminf(xpp, xp), y));
    xl = xp;
}

}  // namespace ra
