"""Host-side run of the C ABI on a recording HIP runtime: what a captured graph
uses stays allocated whatever later calls on its stream need, and what is kept
for it is bounded."""
import numpy as np
import pytest

from .host.abi import Abi


@pytest.fixture(scope="module")
def abi():
    return Abi()


@pytest.fixture
def A(abi):
    abi.stream += 1
    abi.log(), abi.bad()
    return abi


def _capture(A, call, *a, **k):
    assert call(*a, **k) == 0
    A.capture(True)
    rc = call(*a, **k)
    A.capture(False)
    assert rc == 0 and A.bad() == [], A.error


def _size(rng):
    return int(np.exp(rng.uniform(np.log(100), np.log(10 ** 6))))


@pytest.mark.parametrize("kind", ["batch", "extend", "span", "path", "band", "gaps"])
def test_graphs_keep_their_memory(A, kind):
    """Later calls of no more pairs, but on longer references, of other entry
    points or with other options; then of more pairs too."""
    rng = np.random.default_rng(len(kind))
    for trial in range(12):
        A.stream += 1
        n = int(np.exp(rng.uniform(0, np.log(3000))))
        _capture(A, getattr(A, kind), n, 10 ** 6, _size(rng))
        for k in range(12):
            call = getattr(A, rng.choice(["batch", "extend", "span", "path", "band", "gaps"]))
            assert call(n if k < 6 else 3 * n, 10 ** 6, _size(rng)) == 0
            assert A.bad() == [], (trial, k, call.__name__)
        assert A.batch(n, 10 ** 6, 10 ** 6, opts=A.opts(long_kernel=1)) == 0 and A.bad() == []


def test_early_termination_graph(A):
    _capture(A, A.bnb, 50, 10 ** 6, 5000, 10, 900)
    for n, r, reads in ((50, 10 ** 6, 10), (20, 70000, 40), (400, 10 ** 6, 100)):
        assert A.bnb(n, 10 ** 6, r, reads, 900) == 0 and A.bad() == []


def test_what_is_kept_is_bounded(A):
    """Growing call by call keeps at most as much again as the last one needs."""
    def grow():
        before = A.held()
        for n in range(1, 120, 3):
            assert A.batch(n, 10 ** 6, 10 ** 6) == 0 and A.batch(n, 10 ** 6, 10 ** 6, opts=A.opts(long_kernel=1)) == 0
        return A.held() - before

    free = grow()
    A.stream += 1
    _capture(A, A.batch, 1, 1000, 1000)
    assert grow() <= 4 * free and A.bad() == []


def test_the_failure_flag_belongs_to_its_ring(A):
    """A wait given up in a replay leaves the graph's ring to be refilled by the
    graph's next planner, whatever eager calls on a newer ring do in between: the
    launches check that the flag lies behind the ring they use."""
    _capture(A, A.batch, 3, 1000, 1000)
    for n in (40, 400, 4000):
        assert A.batch(n, 10 ** 6, 10 ** 6) == 0 and A.path(n, 10 ** 6, 10 ** 6) == 0 and A.band(n, 10 ** 6, 10 ** 6) == 0
    assert A.bad() == []
