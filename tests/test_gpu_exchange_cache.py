"""GPU parity of the two exchange calls on both sides of the line at which they switch to non-temporal accesses (pairs x
workers x 128 bytes = 256 MiB), and at the smallest calls: sums, weights and cleared residuals against numpy, bit for bit."""
import numpy as np
import pytest

from harness import bits

pytestmark = pytest.mark.gpu
LINE = (256 << 20) // 128


@pytest.mark.parametrize("k,W", [(1, 1), (257, 3), (LINE // 8, 8), (LINE // 8 + 1, 8), (LINE // 32 + 1, 32)])
def test_exchange_on_both_sides_of_the_cache_line(gpu_lib, k, W):
    import torch
    rng = np.random.default_rng(k + W)
    n = 3 * k + 5
    idx = (3 * np.arange(k) + rng.integers(0, 3, k)).astype(np.uint32)
    w = rng.standard_normal(n, dtype=np.float32)
    r = [rng.standard_normal(n, dtype=np.float32) for _ in range(W)]
    dev = "cuda:0"
    wd, idxd = torch.from_numpy(w).to(dev), torch.from_numpy(idx.view(np.int32)).to(dev)
    rd = [torch.from_numpy(x).to(dev) for x in r]
    sumd = torch.empty(k, device=dev)
    scale = float(np.float32(-0.01 / W))
    gpu_lib.gather_sum_at_indices(rd, idxd, k, sumd)
    gpu_lib.apply_sparse_update(wd, idxd, sumd, k, scale, rd)
    torch.cuda.synchronize()
    total = r[0][idx]
    for p in range(1, W):
        total = total + r[p][idx]
    w[idx] = w[idx] + np.float32(scale) * total
    assert np.array_equal(bits(sumd.cpu().numpy()), bits(total))
    assert np.array_equal(bits(wd.cpu().numpy()), bits(w))
    for p in range(W):
        r[p][idx] = 0.0
        assert np.array_equal(bits(rd[p].cpu().numpy()), bits(r[p])), "residual %d" % p
