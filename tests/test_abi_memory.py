"""Host-side run of the C ABI on a recording HIP runtime with little device
memory: calls whose stripe sweep cannot have its scratch take the routes that
need none of it, as long as those have theirs."""
import pytest

from .host.abi import Abi

MB = 1 << 20
BIG = 10 ** 6   # events, levels


@pytest.fixture(scope="module")
def abi():
    return Abi()


@pytest.fixture
def A(abi):
    abi.stream += 1
    abi.log(), abi.bad()
    yield abi
    abi.limit()


def _routes(A):
    assert A.bad() == []
    return [x.split()[0] for x in A.log() if not x.startswith(("malloc", "refused"))]


# What the routes without the sweep hold: per pair 16 bytes of lists (1,024
# pairs at least) and, up to 4,096 waves, an edge column of 64 KB.
@pytest.mark.parametrize("n", [1, 10, 300, 5000])
@pytest.mark.parametrize("kind", ["batch", "extend", "span"])
def test_batches(A, n, kind):
    A.limit(more=min(n, 4096) * 65536 + 64 * max(n, 1024) + MB)
    assert getattr(A, kind)(n, BIG, BIG) == 0, A.error
    assert "sweep" not in (r := _routes(A)) and "multi" in r and "lo" in r and "hi" in r
    A.limit()
    assert getattr(A, kind)(n, BIG, BIG) == 0 and "sweep" in _routes(A)
    A.limit(more=0)   # what is there does
    assert getattr(A, kind)(n, BIG, BIG) == 0 and "sweep" in _routes(A)


@pytest.mark.parametrize("largest", [2 * MB, 40 * MB])
def test_one_buffer_is_too_large(A, largest):
    """Items, ring or columns alone."""
    A.limit(largest=largest)
    for n, r in ((20, BIG), (20, 2000), (30, 70000)):
        assert A.batch(n, BIG, r) == 0 and A.band(n, BIG, r) == 0 and A.path(n, BIG, r) == 0, A.error
        assert A.bnb(n, BIG, r, n // 5, 900) == 0, A.error
    assert A.bad() == []


@pytest.mark.parametrize("n", [1, 10, 500])
def test_paths_and_bands(A, n):
    A.limit(more=n * 65536 + 64 * max(n, 1024) + MB)
    assert A.path(n, BIG, BIG) == 0, A.error
    assert "path each" in [" ".join(x.split()[:2]) for x in A.log()]
    A.limit(more=n * 65536 + MB)
    assert A.band(n, BIG, BIG) == 0, A.error
    assert "band list" in [" ".join(x.split()[:2]) for x in A.log()] and A.bad() == []


def test_too_little_for_any_route(A):
    A.limit(more=0)
    assert A.batch(10, BIG, BIG) == -3 and "allocation" in A.error
