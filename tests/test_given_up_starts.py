"""Host-side pin of what a reverse pass that gave up (end -5) makes of a pair's
start and path: -5, no column of the region."""
import pytest

from .host import compile_host

GAVE_UP = -5


@pytest.fixture(scope="module")
def S():
    return compile_host("span.cpp")


def test_start(S):
    for end in (0, 1, 7, 4000, 65535):
        for rev in (0, end // 2, end):
            assert S.span_start(end, rev) == end - rev
        assert S.span_start(end, GAVE_UP) == GAVE_UP
    for end in (-1, -2, GAVE_UP):   # the forward pass's own sentinel
        for rev in (-1, -2, 0):
            assert S.span_start(end, rev) == end


def test_path(S):
    assert S.interval(100, 400, 10, 300) == 0
    assert S.interval(100, 400, GAVE_UP, 300) == GAVE_UP
    assert S.interval(100, 400, GAVE_UP, GAVE_UP) == GAVE_UP
    for start, end in ((-1, 300), (-2, 300), (301, 300), (10, 400)):
        assert S.interval(100, 400, start, end) == -2
    assert S.interval(100, 400, -1, -1) == -1 and S.interval(100, 400, -2, -2) == -2
