"""Host-side pin of the stripe sweep's schedule (csrc/dtw_sweep.hip): which
lane computes which rows at which step, what travels through the 64-row
blocks and the edge columns, and the odd query's last row, against the plain
table in float32.  Every index into a slot is checked against its size."""
import numpy as np
import pytest

F = np.float32
INF = F(np.inf)
EMPTY = None   # the mark of an edge element nobody has stored


def table(q, r, row, corner):
    """D with row -1 = row, D(-1,-1) = corner, column -1 +inf, cell by cell."""
    n, m = len(q), len(r)
    D = np.empty((n, m), F)
    up, nw0 = row.astype(F), corner
    for i in range(n):
        left, diag = INF, nw0
        for j in range(m):
            left = F(abs(F(q[i] - r[j])) + min(diag, up[j], left))
            D[i, j] = left
            diag = up[j]
        up, nw0 = D[i], INF
    return D


class Slot:
    """Edge column: elements appear once, are taken once."""

    def __init__(self, size):
        self.v = [EMPTY] * size

    def put(self, ix, x):
        assert 0 <= ix < len(self.v) and self.v[ix] is EMPTY, ix
        self.v[ix] = x

    def take(self, ix):
        assert self.v[ix] is not EMPTY, f"element {ix} read before it was stored"
        x, self.v[ix] = self.v[ix], EMPTY
        return x


def rows2(x, n, q0, q1, nw, w0, w1, rv, A, xl):
    """One lane's step, in place, in the kernel's column order."""
    C = len(rv)
    both = x < n - 1
    above, xpp, y = A[0], w0, w1
    xp = F(abs(F(q0 - rv[0])) + min(nw, above, w0))
    for c in range(1, C + 1):
        if c < C:
            up = A[c]
            mx = min(above, up, xp)
        y = F(abs(F(q1 - rv[c - 1])) + min(xpp, xp, y))
        A[c - 1] = y if both else xp
        if c < C:
            xpp, xp, above = xp, F(abs(F(q0 - rv[c])) + mx), up
    return xp


def sweep_stripe(q, r, row, corner, s, S, C, slot_in, slot_out):
    n, m = len(q), len(r)
    lanes = range(64)
    col0 = [(s * 64 + k) * C for k in lanes]
    rv = [[r[j] if j < m else F(0) for j in range(c0, c0 + C)] for c0 in col0]
    A = [[row[j] if j < m else F(0) for j in range(c0, c0 + C)] for c0 in col0]
    ein, eout = s > 0, s + 1 < S
    if eout:
        slot_out.put(0, A[63][C - 1])
    left = slot_in.take(0) if ein else corner
    P = [[F(0), INF, F(0), left] for _ in lanes]
    xl = [F(0)] * 64
    steps = (n + 1) // 2 + 63 if n else 0
    out = [None] * 64
    for t0 in range(0, steps, 32):
        row0 = 2 * t0
        feed = [(F(0), INF)] * 64
        for k in lanes:
            i = row0 + k
            if i < n:
                feed[k] = (q[i], slot_in.take(1 + i) if ein else INF)
        for u in range(32):
            b = feed[2 * u] + feed[2 * u + 1]
            q0 = [b[0]] + [P[k - 1][0] for k in range(1, 64)]
            w0 = [b[1]] + [xl[k - 1] for k in range(1, 64)]
            q1 = [b[2]] + [P[k - 1][2] for k in range(1, 64)]
            w1 = [b[3]] + [A[k - 1][C - 1] for k in range(1, 64)]
            nw = [P[k][3] for k in lanes]
            for k in lanes:
                x = 2 * (t0 + u - k)
                if 0 <= x < n:
                    xl[k] = rows2(x, n, q0[k], q1[k], nw[k], w0[k], w1[k], rv[k], A[k], xl[k])
            P = [[q0[k], w0[k], q1[k], w1[k]] for k in lanes]
            out[2 * u], out[2 * u + 1] = xl[63], A[63][C - 1]
        for k in lanes:
            i = row0 - 126 + k
            if eout and 0 <= i < n:
                slot_out.put(1 + i, out[k])
    return np.array([A[k][c] for k in lanes for c in range(C)], F)


def sweep(q, r, row, corner, C):
    """All stripes of a pair, one after another; the last row."""
    m = len(r)
    S = -(-m // (64 * C))
    slots = [Slot(1 + len(q) + 2) for _ in range(S)]
    cols = []
    for s in range(S):
        cols.append(sweep_stripe(q, r, row, corner, s, S, C, slots[s - 1] if s else None, slots[s]))
    assert all(v is EMPTY for sl in slots for v in sl.v), "an edge element was never taken"
    return np.concatenate(cols)[:m]


@pytest.mark.parametrize("n,m,C", [(1, 1, 1), (1, 130, 1), (2, 65, 1), (3, 70, 1), (5, 200, 2), (63, 64, 1), (64, 190, 1),
                                   (65, 129, 2), (126, 128, 1), (127, 130, 1), (128, 300, 3), (129, 100, 1), (191, 66, 1)])
@pytest.mark.parametrize("mode", ["free", "corner", "resident"])
def test_schedule_equals_table(n, m, C, mode):
    rng = np.random.default_rng(1000 * n + m + C)
    q, r = rng.standard_normal(n).astype(F), rng.standard_normal(m).astype(F)
    if mode == "free":
        row, corner, first = np.zeros(m, F), INF, F(0)   # +inf or 0 left of a zero row give the same
    elif mode == "corner":
        row, corner, first = np.full(m, INF, F), F(0), F(0)
    else:
        row, corner, first = np.abs(rng.standard_normal(m)).astype(F) * 9, INF, INF
    got = sweep(q, r, row, corner, C)
    want = table(q, r, row, first)[-1]
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


def _shape(n, m, lim):
    """sweep_shape in csrc/dtw_device.h: items, stripes per item, columns per lane."""
    stripes, items = max(1, -(-m // 2048)), 1
    if lim > 0:
        want = np.ceil(F(n) * F(m) / (F(64) * F(lim)))
        most = np.ceil(F(m) / (F(64) * max(F(7), np.sqrt(F(26) * F(m) / F(n)))))
        if want > 1:
            items = max(int(min(want, most)), stripes)
    k = 1 if items > 1 else stripes
    c = max(1, -(-m // (64 * items * k)))
    return (-(-m // (64 * c)) if items > 1 else 1), k, c


def test_items_cover_the_region():
    """Every item starts inside the region, the items reach its end, the lane
    widths and counts are representable, and a batch's items fit the list."""
    rng = np.random.default_rng(5)
    for _ in range(300):
        P = int(rng.integers(1, 200))
        n = np.exp(rng.uniform(0, np.log(16384), P)).astype(int) + 1
        m = np.exp(rng.uniform(0, np.log(65536), P)).astype(int).clip(1, 65536)
        slots = int(rng.choice([256, 1024, 5120]))
        lim = max(1.0, float((n.astype(float) * m).sum()) / (64.0 * slots))
        total = 0
        for a, b in zip(n.tolist(), m.tolist()):
            items, k, c = _shape(a, b, lim)
            assert 1 <= c <= 32 and 1 <= k <= 32 and items <= 256
            assert (items - 1) * k * 64 * c < b <= items * k * 64 * c
            total += items
        assert total <= P * -(-int(m.max()) // 2048) + P + 3 * slots


# ---- the ring of edge columns: who may write and read a slot when ------------------

def _wave(ring, state, check_reader):
    """One resident wave of the chained sweep; yields wherever another wave
    may run.  Slot elements carry (item, index) tags."""
    items, slots, done = state["items"], state["slots"], state["done"]

    def free(t):
        while t >= ring and done[t % ring] != t - ring + 1:
            yield
    while state["next"] < len(items):
        t = state["next"]
        state["next"] += 1
        s, S, n = items[t]
        yield from free(t)
        if s and check_reader:
            yield from free(t - 1)
        if s + 1 == S:
            done[t % ring] = t + 1
        out, inp = slots[t % ring], slots[(t - 1) % ring]
        blocks = -(-n // 4)
        if s + 1 < S:
            yield
            assert out[0] is EMPTY
            out[0] = (t, 0)
        for b in range(blocks + 2):   # rows leave two blocks after they come in
            lo, hi = 4 * b, min(4 * b + 4, n)
            if s and lo < n:
                ix = ([0] if b == 0 else []) + list(range(1 + lo, 1 + hi))
                while any(inp[i] is EMPTY for i in ix):
                    yield
                for i in ix:
                    assert inp[i] == (t - 1, i), "a column of another item"
                yield
                for i in ix:
                    inp[i] = EMPTY
            yield
            if s + 1 < S:
                for i in range(max(0, lo - 8), min(lo - 4, n)):
                    assert out[1 + i] is EMPTY, "a column not yet consumed"
                    out[1 + i] = (t, 1 + i)
        if s:
            yield
            done[(t - 1) % ring] = t
        state["finished"] += 1


def _run_ring(seed, ring, waves, check_reader=True):
    rng = np.random.default_rng(seed)
    items = []
    while len(items) < 60:
        S, n = int(rng.integers(1, 7)), int(rng.integers(1, 30))
        items += [(s, S, n) for s in range(S)]
    state = {"items": items, "slots": [[EMPTY] * 40 for _ in range(ring)], "done": [0] * ring, "next": 0, "finished": 0}
    live = [_wave(ring, state, check_reader) for _ in range(waves)]
    budget = 400_000
    while live and budget:
        budget -= 1
        k = int(rng.integers(len(live))) if rng.random() < 0.8 else 0
        try:
            next(live[k])
        except StopIteration:
            live.pop(k)
    assert not live, "the queue did not drain"
    assert state["finished"] == len(items)
    assert all(v is EMPTY for sl in state["slots"] for v in sl)


@pytest.mark.parametrize("ring,waves", [(2, 1), (2, 5), (3, 8), (5, 4), (16, 9)])
def test_ring_protocol(ring, waves):
    for seed in range(12):
        _run_ring(seed, ring, waves)


def test_ring_protocol_needs_the_readers_check():
    """Without it a reader that is early takes the slot's previous column."""
    bad = 0
    for seed in range(12):
        try:
            _run_ring(seed, 3, 8, check_reader=False)
        except AssertionError:
            bad += 1
    assert bad
