"""Batches captured into a HIP graph after warm-up calls of other sizes on the
same stream, replayed three times with eager work between: the routes that need
no scratch of the sweep, and the sweep itself, bit for bit the eager results;
and three captured batches replayed on three streams at once."""
import numpy as np
import pytest

from paper_2310_05037_amd import workloads as W

from . import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    from paper_2310_05037_amd import lib
    assert torch.cuda.is_available()
    lib.load()
    return lib


def _capture(L, db, st, **kw):
    import torch
    opts = L.make_opts(**kw)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(st):
        with torch.cuda.graph(g, stream=st):
            db.run(opts=opts, stream=st)
    return g


@pytest.mark.parametrize("streams", [1, 3])
def test_capture_after_a_shorter_reference(L, streams):
    import torch
    rng = np.random.default_rng(streams)
    a = W.random_pairs(rng, 300, (50, 400), (100, 1500))
    a.r, a.r_off = a.r[:1500], np.zeros_like(a.r_off)   # every region in 1,500 levels
    small = L.DeviceBatch(a)
    b = W.random_pairs(rng, 200, (50, 700), (1000, 9000))
    db = L.DeviceBatch(b)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        small.run(opts=L.make_opts(streams=streams), stream=st)
    st.synchronize()
    print(f"  gpu: capture after a shorter reference streams={streams}", flush=True)
    g = _capture(L, db, st, streams=streams)
    for _ in range(3):
        db.score.fill_(-9.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        parity.check(b, *db.results())


def test_three_captured_sweeps_at_once(L):
    import torch
    rng = np.random.default_rng(8)
    work = []
    for k in range(3):
        b = W.random_pairs(rng, 30 + 10 * k, (300, 2500), (2000, 30000))
        db, st = L.DeviceBatch(b), torch.cuda.Stream()
        with torch.cuda.stream(st):
            db.run(opts=L.make_opts(), stream=st)
        st.synchronize()
        work.append((b, db, st, _capture(L, db, st), parity.oracle_batch(b)))
    print("  gpu: three captured sweeps at once", flush=True)
    for _ in range(5):
        for _, db, st, g, _ in work:
            db.score.fill_(-9.0)
        torch.cuda.synchronize()
        for _, db, st, g, _ in work:
            with torch.cuda.stream(st):
                g.replay()
                db.run(opts=L.make_opts(), stream=st)
        torch.cuda.synchronize()
        for b, db, _, _, ref in work:
            parity.check(b, *db.results(), ref=ref)


def test_graph_after_calls_that_outgrow_its_scratch(L):
    """Replays after uncaptured calls of the same stream on a longer reference
    and of other entry points, which need larger scratch."""
    import torch
    rng = np.random.default_rng(12)
    b = W.random_pairs(rng, 40, (300, 900), (900, 1800))
    b.r, b.r_off = b.r[:1800], np.zeros_like(b.r_off)
    db = L.DeviceBatch(b)
    big = W.random_pairs(rng, 40, (300, 900), (2000, 20000))
    dbig = L.DeviceBatch(big)
    band = torch.full((40,), 300, dtype=torch.int32, device="cuda")
    start = torch.empty(40, dtype=torch.int32, device="cuda")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        db.run(opts=L.make_opts(), stream=st)
    st.synchronize()
    g = _capture(L, db, st)
    ref = parity.oracle_batch(b)
    a = (dbig.q, dbig.q_off, dbig.q_len, dbig.r, dbig.r_off, dbig.r_len)
    later = [lambda: dbig.run(opts=L.make_opts(), stream=st),
             lambda: L.rawalign_dtw_band(*a, band, dbig.score, dbig.end, stream=st),
             lambda: L.rawalign_dtw_span(*a, dbig.score, dbig.end, start, stream=st)]
    print("  gpu: graph after calls that outgrow its scratch", flush=True)
    for call in later:
        with torch.cuda.stream(st):
            call()
            db.score.fill_(-9.0)
            g.replay()
        torch.cuda.synchronize()
        parity.check(b, *db.results(), ref=ref)
