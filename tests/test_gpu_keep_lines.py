"""Tables on both sides of the lines up to which look 1 leaves weights and residuals in the memory-side cache: 40 and 64 MiB a buffer
where it accumulates, 160 MiB where it only reads."""
import numpy as np
import pytest

from test_gpu_selection_paths import _check

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("mib", [40, 64])
@pytest.mark.parametrize("more", [0, 1])
def test_compress_layer(gpu_lib, mib, more):
    import torch
    n = (mib << 18) + more
    rng = np.random.default_rng(mib)
    w = rng.standard_normal(n, dtype=np.float32)
    g = rng.standard_normal(n, dtype=np.float32)
    r = rng.standard_normal(n, dtype=np.float32)
    _check(gpu_lib, torch, w, g, r, n // 100, "%d MiB and %d" % (mib, more))
