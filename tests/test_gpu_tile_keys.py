"""Keys of a tile where their short forms could go wrong: one zero score among a wavefront's thousand, tiles of zeros, infinite and
NaN scores under moved keys (from 513 tiles on a sampled mark moves them), ends of layers inside each of a tile's chunks, and a
caller's record that lies above every key."""
import numpy as np
import pytest

from test_gpu_selection_paths import TILE, _check

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("tiles", [9, 600])
@pytest.mark.parametrize("end", [0, 1, 1023, 1025, 2050, 3075])
def test_zeros_infinities_nan(gpu_lib, tiles, end):
    import torch
    n = tiles * TILE + end
    rng = np.random.default_rng(n)
    w = rng.normal(0.0, 0.1, n).astype(np.float32)
    r = (rng.uniform(-1.0, 1.0, n) * np.abs(w)).astype(np.float32)
    z = np.zeros(n, np.float32)
    one_each = r.copy()
    one_each[rng.integers(0, 1024, n // 1024) + 1024 * np.arange(n // 1024)] = 0.0
    _check(gpu_lib, torch, w, z, one_each, n // 64, "a zero here and there n=%d" % n)
    blocks = r.copy()
    blocks[(np.arange(n) // TILE) % 3 == 1] = 0.0
    _check(gpu_lib, torch, w, z, blocks, n // 64, "tiles of zeros n=%d" % n)
    at = rng.choice(n, n // 32, replace=False)
    wi, ri = w.copy(), r.copy()
    ri[at[::3]] = np.inf                                     # infinite score
    wi[at[1::3]] = 0.0                                       # with eps = 0 infinite, too
    wi[at[2::3]], ri[at[2::3]] = 0.0, 0.0                    # 0 / 0
    for k in (n // 128, n // 40, n // 20):
        _check(gpu_lib, torch, wi, z, ri, k, "infinite and NaN n=%d k=%d" % (n, k), eps=0.0)


@pytest.mark.parametrize("n", [5, TILE + 1, 9 * TILE + 1025])
@pytest.mark.parametrize("key", [0x7FFFFFFE, 0x7FFFFFFF, 0x80000000, 0xFFFFFFFF])
def test_record_above_every_key(gpu_lib, n, key):
    """Nothing is above it or ties with it: no pair is written, whatever the record says of their number."""
    import torch
    r, w = torch.rand(n, device="cuda"), torch.ones(n, device="cuda")
    k = max(1, n // 3)
    thr = torch.from_numpy(np.array([key, 0, k], np.uint32).view(np.int32)).cuda()
    idx, val = torch.full((k,), -7, dtype=torch.int32, device="cuda"), torch.full((k,), -7.0, device="cuda")
    ws = torch.empty(gpu_lib.workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    gpu_lib.compact_pairs(w, r, 1e-8, thr, k, idx, val, ws)
    torch.cuda.synchronize()
    assert bool((idx == -7).all()) and bool((val == -7.0).all())
