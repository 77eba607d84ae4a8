"""GPU parity of compact_pairs, which copies what is at or above the record's threshold into per-tile slots in one pass:
sizes around the tile and super-tile edges, ties cut by the record's quota, tiles whose kept elements overflow their slot
(they are read again by the ordered split), every element kept, infinite and zero thresholds."""
import numpy as np
import pytest

import oracle
from harness import bits

pytestmark = pytest.mark.gpu
TILE = 4096
EPS = 1e-8


def _select_and_compact(iwp, w, r, k, tag):
    import torch
    n = r.size
    wd, rd = torch.from_numpy(w).cuda(), torch.from_numpy(r).cuda()
    thr = torch.zeros(3, dtype=torch.int32, device="cuda")
    idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
    val = torch.full((k,), float("nan"), device="cuda")
    ws = torch.empty(iwp.workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    iwp.select_threshold(wd, rd, k, EPS, thr, ws)
    iwp.compact_pairs(wd, rd, EPS, thr, k, idx, val, ws)
    torch.cuda.synchronize()
    r_ref = r.copy()
    idx_ref, val_ref, _ = oracle.compress_layer(w, np.zeros_like(r), r_ref, k, EPS)
    assert np.array_equal(idx.cpu().numpy().view(np.uint32), idx_ref), tag
    assert np.array_equal(bits(val.cpu().numpy()), bits(val_ref)), tag
    assert np.array_equal(bits(rd.cpu().numpy()), bits(r)), tag + ": the residual is only read"


@pytest.mark.parametrize("n", [1, 3, 4095, 4096, 4097, 8 * TILE - 1, 8 * TILE + 1, 70_003])
@pytest.mark.parametrize("keep", [0.001, 0.05, 1.0])
def test_sizes(gpu_lib, n, keep):
    rng = np.random.default_rng(n)
    w = (rng.standard_normal(n) * 0.05).astype(np.float32)
    r = (rng.standard_t(3, n) * 1e-3).astype(np.float32)
    _select_and_compact(gpu_lib, w, r, max(1, int(n * keep)), "n=%d keep=%g" % (n, keep))


def test_ties_overflowing_slots_and_extremes(gpu_lib):
    rng = np.random.default_rng(5)
    n = 20 * TILE + 9
    w = np.ones(n, np.float32)
    r = rng.uniform(0.1, 0.2, n).astype(np.float32)
    r[2 * TILE:5 * TILE + 7] = 3.0                           # all of three tiles tie at the top
    r[9 * TILE:10 * TILE] = rng.uniform(1.0, 2.0, TILE).astype(np.float32)
    for k in (1, n // 64, TILE, 3 * TILE + 7, 3 * TILE + 8, 4 * TILE + 7, 5 * TILE):
        _select_and_compact(gpu_lib, w, r, k, "k=%d" % k)
    r[:] = 0.0
    _select_and_compact(gpu_lib, w, r, 2 * TILE + 1, "all zero")
    r[::5] = np.float32(3.0e38)
    w[::5] = 0.0                                             # 3e38 / 1e-8: infinite scores
    _select_and_compact(gpu_lib, w, r, n // 10, "infinite threshold")
