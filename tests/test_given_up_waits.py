"""Host-side run of the chained queue's own slot code (csrc/dtw_chain.h) where a
wait is given up: pairs that are not cut use no slot and are aligned all the
same."""
import ctypes

import numpy as np
import pytest

from .host import compile_host

RING = 4


@pytest.fixture(scope="module")
def C():
    so = compile_host("chain.cpp")
    so.path_lost.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.c_int]
    return so


def _open(C, done, t, i, items, failed=0):
    d, f = np.array(done, np.int32), np.array([failed], np.int32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    ok = C.open_slots(RING, ptr(d), ptr(f), t, i, items)
    return bool(ok), d.tolist(), bool(f[0])


def test_slots_that_are_free(C):
    done = [5, 6, 7, 4]   # items 4, 5, 6 and 3 consumed
    assert _open(C, done, 8, 0, 3) == (True, done, False)
    assert _open(C, done, 9, 1, 3) == (True, done, False)
    assert _open(C, [0] * RING, 1, 1, 3) == (True, [0] * RING, False)   # the ring's first round
    # a pair's last item, cut or not, passes its slot on at once
    assert _open(C, done, 8, 0, 1) == (True, [9, 6, 7, 4], False)
    assert _open(C, [0] * RING, 2, 2, 3) == (True, [0, 0, 3, 0], False)


def test_a_wait_that_is_given_up(C):
    """Slot of item 8 still holds item 4's column, and nobody takes it."""
    stuck = [1, 6, 7, 4]
    ok, _, failed = _open(C, stuck, 8, 0, 3)
    assert not ok and failed
    ok, _, failed = _open(C, stuck, 8, 0, 1)
    assert ok and failed, "an uncut pair does not depend on the slot"
    # the same once another wave has given up
    assert not _open(C, stuck, 8, 1, 3, failed=1)[0]
    assert _open(C, stuck, 8, 0, 1, failed=1)[0]


def test_paths_of_uncut_pairs_are_kept(C):
    for n, L in ((100, 300), (5000, 4000), (16384, 65536)):
        cost = n * L / 64
        assert not C.path_lost(n, L, cost * 2, 1)     # one item
        assert not C.path_lost(n, L, cost / 4, 0)     # nothing given up
        assert C.path_lost(n, L, cost / 4, 1)
    assert not C.path_lost(16385, 4000, 1.0, 1)       # never cut
