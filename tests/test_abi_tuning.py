"""Host-side run of the tuner and its caches on a recording HIP runtime: a tuned
setting that names the stripe sweep leaves its waves to the planner, which
chooses them by the batch, and so does a cache of an earlier library version,
whose grids were those of kernels that the sweep took the place of."""
import json

import pytest

from .host.abi import Abi


@pytest.fixture
def A():
    return Abi()


def _waves(A):
    """(waves that a large batch of long pairs may take, workgroups launched)."""
    A.log()
    assert A.batch(100000, 10 ** 8, 10 ** 8) == 0
    log = A.log()
    few = next(x for x in log if x.startswith("plan chain")).split("few=")[1]
    grid = next(x for x in log if x.startswith("sweep")).split()[1].split("=")[1]
    return int(few), int(grid)


DEFAULT = (16 * 256, 20 * 256)


def test_tuner_leaves_the_waves_to_the_planner(A, tmp_path):
    assert _waves(A) == DEFAULT
    cache = str(tmp_path / "tune.json")
    best = A.autotune(1000, 10 ** 7, 10 ** 7, cache)
    assert best["long_kernel"] == 0
    assert _waves(A) == DEFAULT, best
    B = Abi()
    rc, loaded = B.load_tuning(cache)
    assert rc == 0 and loaded == best and _waves(B) == DEFAULT


@pytest.mark.parametrize("long_kernel,waves", [(0, (16, 8, 16)), (2, (12, 4, 8)), (0, (16, 16, 16)), (0, (0, 0, 0))])
def test_caches_of_the_version_before(A, tmp_path, long_kernel, waves):
    path = str(tmp_path / "old.json")
    json.dump({"device": "host", "arch": "gfx950", "version": "rawalign-mi355x 0.6.0", "mode": 1, "long_kernel": long_kernel,
               "lo_waves_per_cu": waves[0], "hi_waves_per_cu": waves[1], "long_waves_per_cu": waves[2], "streams": 3,
               "single_max": 2048, "pipe_waves": 4, "ms": 50.0}, open(path, "w"))
    rc, o = A.load_tuning(path)
    assert rc == 0 and o["long_kernel"] == long_kernel and o["streams"] == 3 and _waves(A) == DEFAULT


def test_anti_diagonal_caches_keep_their_grids(A, tmp_path):
    path = str(tmp_path / "old.json")
    json.dump({"device": "host", "arch": "gfx950", "version": "rawalign-mi355x 0.6.0", "mode": 1, "long_kernel": 1, "lo_waves_per_cu": 12,
               "hi_waves_per_cu": 4, "long_waves_per_cu": 3, "streams": 1, "single_max": 2048, "pipe_waves": 0, "ms": 50.0},
              open(path, "w"))
    assert A.load_tuning(path)[0] == 0
    A.log()
    assert A.batch(100000, 10 ** 8, 10 ** 8) == 0
    log = A.log()
    assert "antidiag grid=768" in log and "lo grid=3072" in log and "hi grid=1024" in log


def test_explicit_grids_are_the_caller_s(A):
    A.log()
    assert A.batch(100000, 10 ** 8, 10 ** 8, opts=A.opts(lo_waves_per_cu=4, hi_waves_per_cu=4, long_waves_per_cu=8)) == 0
    assert any(x.startswith("sweep grid=2048") for x in A.log())


@pytest.mark.parametrize("field,value", [("version", "rawalign-mi355x 0.5.0"), ("arch", "gfx942"), ("device", "other")])
def test_other_caches_are_refused(A, tmp_path, field, value):
    cache = str(tmp_path / "tune.json")
    A.autotune(100, 10 ** 6, 10 ** 6, cache)
    doc = json.load(open(cache))
    assert A.load_tuning(cache)[0] == 0
    json.dump(dict(doc, **{field: value}), open(cache, "w"))
    assert A.load_tuning(cache)[0] == -1
