"""Host-side pin of the sweep's scratch: no more items, slots and columns than a
call's pairs can need (csrc/dtw_shape.h, csrc/internal.h), on the recording HIP
runtime."""
import ctypes

import numpy as np
import pytest

from .host import compile_host
from .host.abi import Abi

MB = 1 << 20


@pytest.fixture(scope="module")
def S():
    so = compile_host("shape.cpp")
    so.sweep_shape.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.POINTER(ctypes.c_int)]
    so.most_items.argtypes = [ctypes.c_longlong, ctypes.c_longlong]
    so.most_items.restype = ctypes.c_longlong
    return so


def test_most_items(S):
    rng = np.random.default_rng(1)
    out = (ctypes.c_int * 3)()
    for _ in range(30000):
        N, M = (int(np.exp(rng.uniform(0, np.log(x)))) for x in (1 << 20, 200000))
        n, m = (int(min(v, max(1, v * rng.random() ** 0.2))) for v in (min(N, 16384), min(M, 65536)))
        S.sweep_shape(n, m, float(max(1.0, n * m / 64 * 10 ** rng.uniform(-4, 0.5))), out)
        assert 1 <= out[0] <= S.most_items(N, M), (n, m, N, M, out[0])


@pytest.fixture(scope="module")
def abi():
    return Abi()


@pytest.fixture
def _bytes(abi):
    def held(call, *a, **k):
        abi.stream += 1   # a stream without scratch
        before = abi.held()
        assert getattr(abi, call)(*a, **k) == 0 and abi.bad() == []
        return abi.held() - before
    return held


def test_small_calls_take_little(_bytes):
    """A read's candidates in a large reference, a lone pair, a few chunks: two
    columns of 64 KB, one in the ring and one of a wave's own, for each item that
    its pairs can have (34 a pair with 1,500 events; 64 waves at least); the
    planner's words and slot counters beside."""
    column = 2 * 65792
    for call in ("batch", "extend", "span"):
        for n, q in ((1, 1500), (10, 1500), (30, 400)):
            assert _bytes(call, n, q, 10 ** 8) <= max(64, n * 35) * column + MB
        assert _bytes(call, 10, 1500, 2000) <= 10 * 8 * column + MB
    for call in ("path", "band"):
        assert _bytes(call, 1, 1500, 5000) <= 64 * column + MB


def test_large_calls_take_no_more_than_documented(_bytes):
    """Edge columns 0.9 GB at most, and 8 bytes per item: 34 a pair on a
    reference above the longest region."""
    for n, q, r in ((100000, 10 ** 8, 10 ** 8), (10 ** 6, 10 ** 6, 10 ** 8), (10 ** 6, 10 ** 6, 2000)):
        assert _bytes("batch", n, q, r) <= 900 * MB + n * (34 * 8 + 2 * 16) + 2 * MB


def test_waves_of_large_batches(S):
    """Where 16 waves per CU were measured to be faster than 20, they are taken;
    where they were slower by 2 % or more, not (pairs, million cells a pair)."""
    S.few_waves.argtypes = [ctypes.c_longlong, ctypes.c_double, ctypes.c_int]
    few = lambda pairs, m: bool(S.few_waves(pairs, pairs * m * 1e6, 4096))
    for pairs, m in ((49152, 1.7), (49152, 3.4), (65536, 1.7), (65536, 3.4), (65536, 6.8), (98304, 3.4), (100000, 9.2)):
        assert few(pairs, m), (pairs, m)
    for pairs, m in ((8192, 3.4), (8192, 6.8), (16384, 1.7), (16384, 3.4), (16384, 6.8), (24576, 3.4), (32768, 3.4), (32768, 6.8),
                     (65536, 0.4), (98304, 0.4), (98304, 0.2), (49152, 0.2)):
        assert not few(pairs, m), (pairs, m)
    assert not S.few_waves(10 ** 6, 1e13, 0)
