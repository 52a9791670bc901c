"""Serving: a job whose sweep was given up (NaN, -5) leaves its resident row half
written, so its read ends as failed, its rows are freed and nothing is aligned
on from them; the other reads go on."""
import numpy as np
import pytest

from oracle import oracle
from paper_2310_05037_amd import serve

from .serving_oracle import OracleBackend
from .test_serving_host import VClock, drive, small_workload


class GivingUp(OracleBackend):
    """The `lost`-th chunk of the read at region offset `at` is given up."""

    def __init__(self, r, arena, at, lost):
        super().__init__(r, arena)
        self.at, self.lost, self.seen, self.after = at, lost, 0, 0

    def run(self, b, b_match, threshold):
        score, end, best, bs, mapped = super().run(b, b_match, threshold)
        jobs = np.flatnonzero(b.r_off == self.at)
        if len(jobs):
            self.seen += 1
            self.after += self.seen > self.lost
        if len(jobs) and self.seen == self.lost:
            j = jobs[0]
            score[j], end[j] = np.nan, -5
            ro, rl, wo = int(b.r_off[j]), int(b.r_len[j]), int(b.row_off[j])
            self.rows[wo + rl // 2:wo + rl] = 0.0
            best, bs, mapped = oracle.decide(score, b.cand_off, b.cand_cnt, b.n_events, b_match, threshold)
        return score, end, best, bs, mapped


@pytest.mark.parametrize("lost", [1, 2])
def test_read_of_a_given_up_job_fails(lost):
    w = small_workload()
    arena = sum(int(rd.r_len.sum()) for rd in w.reads)

    def run(backend):
        clock = VClock()
        eng = serve.Engine(backend, arena, w.chunk, w.period, clock=clock)
        for i, rd in enumerate(w.reads):
            eng.submit(i, rd.arrival, rd.events, rd.r_off, rd.r_len)
        drive(eng, clock)
        assert eng.all_done() and eng.arena.used == 0
        return eng

    ref = run(OracleBackend(w.r, arena))
    offs = [o for rd in w.reads for o in rd.r_off]
    victim = next(k for k, rd in enumerate(w.reads) if len(ref.reads[k].results) > lost and offs.count(rd.r_off[0]) == 1)
    backend = GivingUp(w.r, arena, int(w.reads[victim].r_off[0]), lost)
    eng = run(backend)
    assert backend.seen == lost and backend.after == 0
    assert eng.reads[victim].status == "failed" and eng.failed_ticks == 0
    assert len(eng.reads[victim].results) == lost - 1
    for k, st in enumerate(eng.reads):
        if k != victim:
            assert st.status == ref.reads[k].status and len(st.results) == len(ref.reads[k].results)
            for x, y in zip(st.results, ref.reads[k].results):
                assert x[0] == y[0] and x[2] == y[2] and np.array_equal(x[3], y[3]) and np.array_equal(x[4], y[4])
