"""Host-side run of what early termination does with its pairs between rounds
(csrc/dtw_bnb.h): a part whose sweep gave up (NaN, -5) ends its pair, whose
resident row is not the pair's any more; the others go on as without it."""
import ctypes

import numpy as np
import pytest

from .host import compile_host


@pytest.fixture(scope="module")
def B():
    return compile_host("bnb.cpp")


def _rounds(B, n, cost, fails, n_events, b_match=0.4, block=64, rounds=6):
    P, N = cost.shape
    out, end = np.zeros(P, np.float32), np.full(P, -9, np.int32)
    swept, took = np.zeros(P, np.int32), np.zeros(P, np.int32)
    n, cost, fails = np.asarray(n, np.int32), np.ascontiguousarray(cost, np.float32), np.asarray(fails, np.int32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    B.rounds(P, N, ptr(n), ptr(cost), ptr(fails), n_events, ctypes.c_double(b_match), block, rounds, ptr(out), ptr(end), ptr(swept),
             ptr(took))
    return out, end, swept, took


N, PAIRS = 1000, 6


def _costs(rng):
    """Costs that never fall along the rows; those that rise early look as if
    they would be dropped soon, and take the most rounds."""
    row = np.arange(1, N + 1) / N
    noise = np.cumsum(rng.random((PAIRS, N)), axis=1)
    return noise / 1000 + 90 * row ** rng.uniform(0.2, 1.5, (PAIRS, 1)) * rng.uniform(0.9, 1.1, (PAIRS, 1))


@pytest.mark.parametrize("lost", range(4))
def test_a_given_up_part_ends_its_pair(B, lost):
    rng = np.random.default_rng(lost)
    seen = 0
    for trial in range(40):
        cost = _costs(rng)
        n = rng.choice([N, N - 1, N - 37], PAIRS)
        last = cost[np.arange(PAIRS), n - 1].astype(np.float32)
        for p in range(PAIRS):
            fails = np.full(PAIRS, -1)
            fails[p] = lost
            out, end, swept, took = _rounds(B, n, cost, fails, N)
            if took[p] >> lost & 1:
                seen += 1
                assert end[p] == -5 and np.isnan(out[p]), (trial, p)
                assert not took[p] >> (lost + 1), "went on from a row that was not finished"
            whole = end == np.arange(PAIRS)
            assert np.array_equal(out[whole], last[whole]) and np.array_equal(swept[whole], n[whole])
            assert np.isin(end[~whole], (-3, -5)).all()
            # the read's best among the pairs that were aligned is one of them
            left = np.where(end == -5, np.inf, last)
            assert whole[np.argmin(left)], (trial, p)
    assert seen > 20


def test_a_given_up_first_candidate_prunes_nothing(B):
    """Its read has no best Score from it: the others are aligned whole or
    dropped for another's."""
    rng = np.random.default_rng(9)
    cost = _costs(rng)
    cost[0] *= 1e-3          # the winner, if it had been aligned
    n = np.full(PAIRS, N)
    ref, rend, _, _ = _rounds(B, n, cost, np.full(PAIRS, -1), N)
    assert (rend[1:] == -3).any()
    out, end, swept, _ = _rounds(B, n, cost, [0] + [-1] * (PAIRS - 1), N)
    assert end[0] == -5 and np.isnan(out[0]) and swept[0] == N
    best = 1 + int(np.argmin(cost[1:, -1]))
    assert end[best] == best and out[best] == np.float32(cost[best, -1])
