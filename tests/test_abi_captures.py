"""Host-side run of the C ABI on a recording HIP runtime: calls inside a stream
capture allocate nothing, whatever smaller or other calls warmed the stream up
(one of at least as many pairs among them), and use only memory that is there."""
import numpy as np
import pytest

from .host.abi import Abi


@pytest.fixture(scope="module")
def abi():
    return Abi()


@pytest.fixture
def A(abi):
    abi.stream += 1   # nothing of the tests before
    abi.log(), abi.bad()
    return abi


def _captured(A, call, *a, **k):
    A.log()
    A.capture(True)
    rc = call(*a, **k)
    A.capture(False)
    return rc, A.bad(), A.log()


def test_warm_up_on_a_shorter_reference(A):
    """The warm-up's items would do for the capture, its edge columns not."""
    assert A.batch(1000, 10 ** 6, 2000) == 0
    assert _captured(A, A.batch, 500, 10 ** 6, 6000)[:2] == (0, []), A.error


def test_warm_up_of_the_same_call_takes_the_sweep(A):
    for n, q, r in ((1, 400, 900), (40, 5000, 70000), (700, 10 ** 6, 2000), (9000, 10 ** 6, 10 ** 6)):
        A.stream += 1
        assert A.batch(n, q, r) == 0 and A.bad() == []
        rc, bad, log = _captured(A, A.batch, n, q, r)
        assert rc == 0 and bad == [] and any(x.startswith("sweep") for x in log)


@pytest.mark.parametrize("streams", [1, 3])
@pytest.mark.parametrize("kind", ["batch", "extend", "span"])
def test_any_smaller_warm_up(A, kind, streams):
    rng = np.random.default_rng(streams)
    call = getattr(A, kind)
    o = A.opts(streams=streams)
    for _ in range(60):
        A.stream += 1
        n = int(np.exp(rng.uniform(0, np.log(20000))))
        for _ in range(int(rng.integers(1, 4))):
            assert call(n + int(rng.integers(0, 50)), 10 ** 6, int(np.exp(rng.uniform(np.log(100), np.log(10 ** 6)))), opts=o) == 0
        r = int(np.exp(rng.uniform(np.log(100), np.log(10 ** 6))))
        rc, bad, _ = _captured(A, call, n, 10 ** 6, r, opts=o)
        assert rc == 0 and bad == [], (n, r, A.error, bad)


def test_band_and_path_after_other_calls(A):
    rng = np.random.default_rng(3)
    for _ in range(80):
        A.stream += 1
        n = int(np.exp(rng.uniform(0, np.log(5000))))
        size = lambda: int(np.exp(rng.uniform(np.log(100), np.log(10 ** 6))))
        for _ in range(2):
            assert A.band(n, 10 ** 6, size()) == 0 and A.path(n, 10 ** 6, size()) == 0 and A.batch(n, 10 ** 6, size()) == 0
        assert A.bad() == []
        for call in (A.band, A.path):
            r = size()
            rc, bad, _ = _captured(A, call, n, 10 ** 6, r)
            assert rc == 0 and bad == [], (call.__name__, n, r, A.error, bad)
