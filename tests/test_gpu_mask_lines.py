"""Masks of one to three nodes on both sides of the line between 512 and 256 threads a tile (2560 tiles), with layers that end around a
chunk of either (2048 and 1024 elements), plain and with random selection."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import ThresholdSet, bits

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]
TILE, W = 4096, 3


@pytest.mark.parametrize("n_lead", [1, 2, 3])
@pytest.mark.parametrize("tiles", [12, 2560, 2561])
def test_masks(gpu_lib, tiles, n_lead):
    sizes = [1023, 1025, 2047, 2048, 2049, TILE + 2047, TILE + 2049]
    sizes.append((tiles - 9) * TILE - 1)
    ps = wl.custom_set([(n, 0) for n in sizes], W=W, seed=tiles, align=1, start=n_lead)
    assert sum((n + TILE - 1) // TILE for n in sizes) == tiles
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    r0 = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    leaders = np.array([[(j + q) % W for q in range(n_lead)] for j in range(len(sizes))], np.uint32)
    thr = np.full(len(sizes), np.quantile(np.abs(sets[0][:100000]) / (np.abs(w[:100000]) + np.float32(1e-8)), 0.95), np.float32)
    scale = float(np.float32(-0.01))
    for random in ([None, (77, 3)] if tiles < 100 else [None]):
        w_ref, r_ref = w.copy(), [x.copy() for x in r0]
        ts = ThresholdSet(gpu_lib, ps, w, sets, r0, n_lead, ps.flat)
        ts.step(list(range(W)), leaders, thr, scale, random=random)
        mask, cnt, idx, sm = oracle.step_threshold(w_ref, sets, r_ref, ps.rows(), leaders, thr, 1e-8, scale, ps.flat, random=random)
        got, total = ts.download(), int(cnt.sum())
        assert np.array_equal(got["idx"][:total], idx) and np.array_equal(bits(got["sum"][:total]), bits(sm))
        assert np.array_equal(bits(got["w"]), bits(w_ref))
        for p in range(W):
            assert np.array_equal(bits(got["r"][p]), bits(r_ref[p]))
