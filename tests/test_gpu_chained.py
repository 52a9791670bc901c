"""GPU parity, bit for bit against the float oracle, of the path and band
kernels where a few pairs are cut into stripes that several waves sweep at
once: intervals and bands around a lane, a stripe and a block of 32 rows."""
import numpy as np
import pytest

from . import test_gpu_path as path
from .test_gpu_path import L  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spans", [[255], [256], [257, 1024], [1023, 1025, 2049], [5000], [1, 31, 32, 33, 700, 4096]])
def test_path_cut_into_stripes(L, spans):  # noqa: F811
    rng = np.random.default_rng(len(spans) + spans[0])
    b = path._embedded(rng, spans, f"path_cut_{spans[0]}", dwell_p=0.5)
    path._check(b, path._gpu_path(L, b), range(b.n_pairs))
