"""GPU parity of the pairs written from given thresholds on both sides of the longest layer whose earlier tiles the split adds up
by itself (4096 tiles; beyond, a launch of its own folds the counts): full, ragged and tied tiles before every workgroup's."""
import numpy as np
import pytest

from test_gpu_compact import TILE, _select_and_compact

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n", [4096 * TILE, 4096 * TILE + 1, 300 * TILE + 5])
def test_both_sides(gpu_lib, n):
    rng = np.random.default_rng(n)
    w = np.ones(n, np.float32)
    r = rng.standard_normal(n, dtype=np.float32)
    r[5 * TILE:9 * TILE + 3] = 7.0                           # tie with nothing else, above most
    for k in (n // 64, 2 * TILE + 1):                        # the second cuts through the ties
        _select_and_compact(gpu_lib, w, r, k, "n=%d k=%d" % (n, k))
