"""GPU parity, bit for bit against the float oracle, of the path and band
kernels where a few pairs are cut into stripes that several waves sweep at
once: intervals and bands around a lane, a stripe and a block of 32 rows."""
import numpy as np
import pytest

from . import test_gpu_band as band
from . import test_gpu_path as path
from .test_gpu_path import L  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spans", [[255], [256], [257, 1024], [1023, 1025, 2049], [5000], [1, 31, 32, 33, 700, 4096]])
def test_path_cut_into_stripes(L, spans):  # noqa: F811
    rng = np.random.default_rng(len(spans) + spans[0])
    b = path._embedded(rng, spans, f"path_cut_{spans[0]}", dwell_p=0.5)
    path._check(b, path._gpu_path(L, b), range(b.n_pairs))


@pytest.mark.parametrize("n,m,w", [(3000, 1025, 130), (3000, 1024, 0), (3000, 1023, 700), (900, 5000, 400),
                                   (96, 257, 40), (97, 2049, 2048), (7000, 4097, 127), (2000, 6000, 1), (12, 9000, 300)])
@pytest.mark.parametrize("pairs", [1, 40])
def test_band_cut_into_stripes(L, n, m, w, pairs):  # noqa: F811
    rng = np.random.default_rng(n + m + w)
    ns = np.maximum(n - 7 * np.arange(pairs), 1)
    ms = np.maximum(m - 3 * np.arange(pairs), 1)
    b = band._pairs(rng, ns, ms, f"band_cut_{n}_{m}_{w}")
    width = np.maximum(w - np.arange(pairs) % 3, 0).astype(np.int32)
    band._check(b, width, *band._gpu_band(L, b, width))
