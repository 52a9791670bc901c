"""Host-side run of the C ABI on a recording HIP runtime: early termination's
scratch doubles as its batches grow, and batches of more pairs and of more reads
in turn do not make it move each time."""
import pytest

from .host.abi import Abi


@pytest.fixture(scope="module")
def A():
    return Abi()


def _moves(A, sizes):
    assert A.batch(4000, 10 ** 6, 2000) == 0 and A.extend(4000, 10 ** 6, 2000) == 0   # the sweep's own scratch
    A.log()
    count = 0
    for n, reads in sizes:
        assert A.bnb(n, 10 ** 6, 2000, reads, 900) == 0 and A.bad() == []
        count += sum(x.startswith("malloc") for x in A.log())
    return count


def test_growing_batches(A):
    """From 100 to 3,000 pairs, five doublings, and as many of the reads, which
    may fall on other calls; and the first."""
    A.stream += 1
    assert _moves(A, [(n, n // 4 + 1) for n in range(100, 3000, 20)]) <= 11


def test_more_pairs_and_more_reads_in_turn(A):
    A.stream += 1
    assert _moves(A, [(2000, 10), (100, 1500)] * 20) <= 4
