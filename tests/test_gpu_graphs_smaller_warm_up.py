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
