"""Host-side pin of the planner's cut against the size of a ring slot: the
library's own rule (csrc/dtw_shape.h) and limits over every length a pair may
have."""
import ctypes

import numpy as np
import pytest

from .host import compile_host


@pytest.fixture(scope="module")
def S():
    so = compile_host("shape.cpp")
    so.sweep_shape.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.POINTER(ctypes.c_int)]
    so.limits = dict(zip(("edge", "slot", "stripe", "single", "items", "cols"), (so.limit(k) for k in range(6))))

    def shape(n, m, lim):
        out = (ctypes.c_int * 3)()
        so.sweep_shape(n, m, lim, out)
        return tuple(out)
    so.shape = shape
    return so


def _lengths(lim):
    edge = lim["edge"]
    return [1, 2, 400, 900, 5000, edge - 1, edge, edge + 1, lim["slot"] - 3, lim["slot"] - 2, lim["slot"], 20000, 32900, 40000,
            1 << 20, 4_000_000, 1 << 28]


def test_edge_columns_fit_their_slots(S):
    """Between items an edge column is the corner, n rows and two words of the
    running minimum.  Pairs the sweep takes (the planner sends queries above an
    edge column in regions above one stripe to the single-stripe kernel) are
    cut only if that fits a slot, alone, among equals and among larger ones;
    within an item of several stripes the rows fit the wave's own column."""
    lim = S.limits
    for n in _lengths(lim):
        for m in [1, 64, 448, 449, 896, 897, 1000, 2000, 2047, 2048, 2049, 4096, 4097, 20000, 65536]:
            if n > lim["edge"] and m > lim["stripe"]:
                continue   # the single-stripe kernel's, or refused
            for share in (1.0, 64.0, float(n) * m / (64 * 5120), float(n) * m / (64 * 33), float(n) * m / (64 * 2), 1e12):
                items, k, c = S.shape(n, m, max(share, 1.0))
                assert items >= 1 and k >= 1 and 1 <= c <= lim["cols"] and items <= lim["items"]
                assert (items - 1) * k * 64 * c < m <= items * k * 64 * c
                if items > 1:
                    assert n + 3 <= lim["slot"], f"column of {n + 3} floats in a slot of {lim['slot']} (m={m}, {items} items)"
                if k > 1:
                    assert n <= lim["edge"]


def test_cut_lengths_drawn(S):
    lim = S.limits
    rng = np.random.default_rng(7)
    cut = 0
    for _ in range(20000):
        n = int(np.exp(rng.uniform(0, np.log(1 << 24))))
        m = int(np.exp(rng.uniform(0, np.log(65536))))
        if m > lim["stripe"]:
            n = min(n, lim["edge"])
        items, _, _ = S.shape(n, m, float(max(1.0, n * m / 64 * rng.uniform(1e-4, 2))))
        cut += items > 1
        assert items == 1 or n + 3 <= lim["slot"], (n, m, items)
    assert cut > 1000
