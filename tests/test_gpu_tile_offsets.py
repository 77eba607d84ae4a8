"""Where the tiles' pairs start, found by every workgroup of the one launch (up to 256 tiles) or of the workers' pass (up to 1024), or by a
launch of its own: the counts that the caller sees with empty layers among the others and more layers than threads, and a total that just fits the caller's
room, or exceeds it by one."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import ThresholdSet, bits

pytestmark = pytest.mark.gpu
W, TILE = 2, 4096


@pytest.mark.parametrize("room", ["all", "fits", "one too few"])
@pytest.mark.parametrize("tiles,empty", [(1, 0), (9, 700), (255, 3), (256, 0), (257, 700), (1024, 3), (1025, 0)])
def test_counts(gpu_lib, tiles, empty, room):
    rng = np.random.default_rng(tiles)
    sizes = [1, 5 * TILE - 1, TILE] if tiles >= 9 else [TILE - 3]
    left = tiles - sum((n + TILE - 1) // TILE for n in sizes)
    sizes += [left * TILE - 2] if left else []
    for _ in range(empty):
        sizes.insert(int(rng.integers(0, len(sizes) + 1)), 0)
    ps = wl.custom_set([(n, 0) for n in sizes], W=W, seed=tiles, align=1, start=1)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    r0 = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    leaders = np.array([[j % W] for j in range(len(sizes))], np.uint32)
    thr = np.full(len(sizes), np.quantile(np.abs(sets[0]) / (np.abs(w) + np.float32(1e-8)), 0.9), np.float32)
    scale = float(np.float32(-0.01))
    w_ref, r_ref = w.copy(), [x.copy() for x in r0]
    mask, cnt, idx, sm = oracle.step_threshold(w_ref, sets, r_ref, ps.rows(), leaders, thr, 1e-8, scale, ps.flat)
    total = int(cnt.sum())
    ts = ThresholdSet(gpu_lib, ps, w, sets, r0, 1, {"all": ps.flat, "fits": total, "one too few": total - 1}[room])
    ts.step(list(range(W)), leaders, thr, scale)
    got = ts.download()
    count = ts.count.cpu().numpy()
    assert np.array_equal(count[:len(sizes)], cnt) and count[-2] == total and count[-1] == (room == "one too few")
    if room == "one too few":                                  # accumulated, nothing exchanged
        assert np.array_equal(bits(got["w"]), bits(w))
        for p in range(W):
            assert np.array_equal(bits(got["r"][p]), bits(r0[p] + sets[p]))
        return
    assert np.array_equal(got["idx"][:total], idx) and np.array_equal(bits(got["sum"][:total]), bits(sm))
    assert np.array_equal(bits(got["w"]), bits(w_ref))
    for p in range(W):
        assert np.array_equal(bits(got["r"][p]), bits(r_ref[p]))
