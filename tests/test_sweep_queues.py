"""Host-side model of the chained queue's eight heads (csrc/internal.h,
csrc/dtw_chain.h) where a launch does not get the whole chip: workgroups go
round the eight dies in turn, each die starts its own in order as slots come
free, and launches on other streams hold slots as well.  A wave waits until the
item before its own has been taken; every launch must drain."""
import numpy as np
import pytest

from .host import compile_host

DIES = 8


@pytest.fixture(scope="module")
def Q():
    return compile_host("queues.cpp")


@pytest.mark.parametrize("dies", [1, 2, 4, 8])
def test_every_queue_is_covered(Q, dies):
    """Whichever die gives a launch slots: its first workgroups there, in
    order, take from every queue (eight on one of eight dies, at most 64
    wherever the chip is fewer)."""
    for grid in [64, 65, 100, 330, 1470, 4096, 5120]:
        for n_items in (1, 2, 7, 8, 9, 63, 64, 65, 200, 4 * grid):
            live = min(grid, Q.live_workgroups(n_items, 0x7fffffff))
            assert min(n_items, grid) <= live
            for d in range(dies):
                mine = list(range(d, live, dies))[:64 // dies]
                assert {Q.queue_of(b) for b in mine} == set(range(Q.queues())), (grid, n_items, d)
    for most in (1, 64, 4096):
        assert Q.cover() <= Q.live_workgroups(10 ** 6, most) <= max(most, Q.cover())


class Launch:
    def __init__(self, Q, grid, items):
        self.Q, self.grid, self.items = Q, grid, items   # items: True where the item reads the one before
        self.heads = [0] * 8
        self.taken = [False] * len(items)
        self.done = [False] * len(items)
        self.waiting = {d: [b for b in range(grid) if b % DIES == d] for d in range(DIES)}
        self.waves = []

    def start(self, die):
        b = self.waiting[die].pop(0)
        if b < self.Q.live_workgroups(len(self.items), 0x7fffffff):
            self.waves.append([die, b, None])
            return True
        return False

    def step(self, free):
        """One step of every wave; free[die] grows where one exits."""
        moved = False
        q = self.Q.queues()
        for w in list(self.waves):
            die, b, t = w
            if t is None:
                x = self.Q.queue_of(b)
                t, self.heads[x] = self.heads[x] * q + x, self.heads[x] + 1
                moved = True
                if t >= len(self.items):
                    self.waves.remove(w)
                    free[die] += 1
                    continue
                self.taken[t], w[2] = True, t
            elif not self.items[t] or self.done[t - 1]:
                self.done[t], w[2] = True, None
                moved = True
        return moved

    def finished(self):
        return all(self.done)


def _drain(launches, slots, first):
    """first[d]: the launch whose workgroups die d starts first (the others
    follow when it has none left)."""
    free = [slots] * DIES
    for _ in range(100000):
        moved = False
        for d in range(DIES):
            order = [launches[first[d]]] + [x for x in launches if x is not launches[first[d]]]
            for x in order:
                while free[d] and x.waiting[d]:
                    moved = True
                    if x.start(d):
                        free[d] -= 1
        for x in launches:
            moved = x.step(free) or moved
        if all(x.finished() for x in launches):
            return True
        if not moved:
            return False
    raise AssertionError("no end")


@pytest.mark.parametrize("streams", [1, 2, 3])
def test_launches_that_share_the_chip_drain(Q, streams):
    rng = np.random.default_rng(streams)
    for trial in range(60):
        slots = int(rng.integers(8, 24))
        launches = []
        for _ in range(streams):
            grid = int(rng.choice([slots * DIES, slots * DIES // 2, 90]))
            items = []
            while len(items) < 3 * grid:
                items += [k > 0 for k in range(int(rng.integers(1, 40)))]
            launches.append(Launch(Q, grid, items))
        first = [int(rng.integers(streams)) for _ in range(DIES)]
        assert _drain(launches, slots, first), (trial, first)


def test_one_die_for_each_launch(Q):
    """The die fill that starves a queue whose workgroups are all on one die."""
    items = [k % 24 > 0 for k in range(600)]
    launches = [Launch(Q, 16 * DIES, list(items)) for _ in range(2)]
    assert _drain(launches, 16, [0, 0, 0, 0, 1, 1, 1, 1])
