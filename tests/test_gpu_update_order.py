"""GPU parity of the sparse update at pair counts around its workgroups (256 pairs) and its groups of eight of them, which it
takes from the last to the first: every pair exactly once, whatever is left over at the end; and without residuals."""
import numpy as np
import pytest

import oracle
from harness import bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [0, 3])
@pytest.mark.parametrize("k", [1, 255, 256, 257, 7 * 256, 7 * 256 + 1, 8 * 256 - 1, 8 * 256, 8 * 256 + 1, 15 * 256 + 9, 16 * 256,
                               16 * 256 + 1, 1000003])
def test_every_pair_once(gpu_lib, k, W):
    import torch
    rng = np.random.default_rng(k + W)
    n, dev = 2 * k + 3, "cuda:0"
    idx = (2 * np.arange(k) + rng.integers(0, 2, k)).astype(np.uint32)
    w, s = rng.standard_normal(n, dtype=np.float32), rng.standard_normal(k, dtype=np.float32)
    r = [rng.standard_normal(n, dtype=np.float32) for _ in range(W)]
    wd, sd, idxd = (torch.from_numpy(x).to(dev) for x in (w, s, idx.view(np.int32)))
    rd = [torch.from_numpy(x).to(dev) for x in r]
    scale = float(np.float32(-0.01))
    gpu_lib.apply_sparse_update(wd, idxd, sd, k, scale, rd)
    torch.cuda.synchronize()
    oracle.apply_sparse_update(w, idx, s, scale, r)
    assert np.array_equal(bits(wd.cpu().numpy()), bits(w))
    for p in range(W):
        assert np.array_equal(bits(rd[p].cpu().numpy()), bits(r[p])), "residual %d" % p
