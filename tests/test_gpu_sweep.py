"""GPU parity of the stripe sweep at its edges, bit for bit against the float
oracle (a shortest-path recurrence has one value whatever the order, so there
is no tolerance): queries around a two-row step, a block and the skew, regions
around a lane, a stripe and an item, few pairs (cut into many items) and more
items than the ring holds, streamed in chunks and whole."""
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


EDGES = {   # pairs, queries, regions
    "lone": (1, [3001], [2500]),
    "steps": (400, [1, 2, 3, 31, 32, 33, 63, 64, 65, 126, 127, 128, 129, 257], [1, 2, 63, 64, 65, 127, 128, 129, 511, 2047, 2048, 2049]),
    "items": (24, [899, 900, 1537], [2047, 2048, 2049, 4095, 4097, 7000]),
    "widest": (4, [700], [65535, 65536]),
    "ring": (9000, [40, 97], [300, 2600]),
}


@pytest.mark.parametrize("case", sorted(EDGES))
@pytest.mark.parametrize("chunks", [0, 3])
def test_sweep_edges(L, case, chunks):
    import torch
    pairs, ns, ms = EDGES[case]
    rng = np.random.default_rng(len(case))
    b = W.random_pairs(rng, pairs, (max(ns), max(ns)), (max(ms), max(ms)))
    b.q_len[:] = rng.choice(ns, pairs)
    b.r_len[:] = rng.choice(ms, pairs)
    print(f"  gpu: sweep {case} chunks={chunks} pairs={pairs} n={ns} m={ms}", flush=True)
    db = L.DeviceBatch(b)
    if chunks:
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        row_off = np.concatenate([[0], np.cumsum(b.r_len.astype(np.int64))[:-1]])
        rows = torch.zeros(int(b.r_len.sum()), dtype=torch.float32, device="cuda")
        cut = [b.q_len.astype(np.int64) * k // chunks for k in range(chunks + 1)]
        for k in range(chunks):
            L.rawalign_dtw_extend(db.q, dev(b.q_off + cut[k]), dev((cut[k + 1] - cut[k]).astype(np.int32)), db.r,
                                  db.r_off, db.r_len, rows, dev(row_off),
                                  torch.full((pairs,), int(k == 0), dtype=torch.uint8, device="cuda"), db.score, db.end)
    else:
        db.run()
    print(parity.check(b, *db.results()))
