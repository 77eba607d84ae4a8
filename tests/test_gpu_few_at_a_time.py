"""Launches that hold fewer workgroups per compute unit than would fit: tables on both sides of the rules (accumulating workers,
filled tiles, share that is sent, workgroups in all) give the oracle's step bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, ThresholdSet, assert_step_equal, bits

pytestmark = pytest.mark.gpu
TILE = 4096


@pytest.mark.parametrize("W,sizes,share", [(3, [40 * TILE + 5, 9 * TILE], 40), (2, [40 * TILE + 5, 9 * TILE], 40),
                                           (3, [40 * TILE, 9 * TILE], 16), (3, [40 * TILE, 9 * TILE], 15),
                                           (5, [2 * TILE] * 90, 33), (5, [2 * TILE] * 45 + [TILE - 1] * 45, 33)])
def test_steps(gpu_lib, W, sizes, share):
    ps = wl.custom_set([(n, n // share) for n in sizes], W=W, seed=share, align=1, start=3)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    gs = GpuSet(gpu_lib, ps, w, sets, fused=True, hint="none")
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    for t in range(2):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % W for p in range(W)]
        ref = oracle.step(w, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w, r_ref, *ref, ps.layers, tag="W=%d step %d" % (W, t))


@pytest.mark.parametrize("W,sizes,share", [(3, [300 * TILE + 5, 9 * TILE], 40), (2, [300 * TILE + 5, 9 * TILE], 40),
                                           (3, [300 * TILE, 9 * TILE], 16), (3, [300 * TILE, 9 * TILE], 15),
                                           (3, [300 * TILE, 9 * TILE], 32), (3, [300 * TILE, 9 * TILE], 31),
                                           (5, [2 * TILE] * 130 + [9 * TILE], 33), (5, [TILE - 1] * 300 + [9 * TILE], 33)])
def test_steps_of_more_tiles_than_one_launch_takes(gpu_lib, W, sizes, share):
    """From 257 tiles on the followers and the update have launches of their own, which the rules are about."""
    ps = wl.custom_set([(n, n // share) for n in sizes], W=W, seed=share, align=1, start=3)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    gs = GpuSet(gpu_lib, ps, w, sets, fused=True, hint="none")
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    for t, kernel in enumerate(("k_follow_gather", "k_reduce_update")):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % W for p in range(W)]
        ref = oracle.step(w, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gpu_lib.timing_enable(kernel)
        gs.step(ids, lead)
        assert gpu_lib.timing_collect()[1] == 1
        assert_step_equal(gs.download(), w, r_ref, *ref, ps.layers, tag="W=%d step %d" % (W, t))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("tiles", [1275, 1280, 1281])             # 16 workers: 20480 workgroups at the line
def test_threshold_step(gpu_lib, tiles):
    W, layers = 16, 5
    sizes = [tiles // layers * TILE - 3] * (layers - 1)
    sizes.append((tiles - (layers - 1) * (tiles // layers)) * TILE - 1)
    ps = wl.custom_set([(n, 0) for n in sizes], W=W, seed=tiles, align=1, start=3)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    ts = ThresholdSet(gpu_lib, ps, w, sets, r_ref, 1, ps.flat)
    leaders = np.array([[j % W] for j in range(layers)], np.uint32)
    thr = np.array([np.quantile(np.abs(sets[j][L.offset:L.offset + L.n]) / (np.abs(w[L.offset:L.offset + L.n]) + 1e-8), 0.98)
                    for j, L in enumerate(ps.layers)], np.float32)
    ts.step(list(range(W)), leaders, thr, -0.01)
    mask, cnt, idx, sm = oracle.step_threshold(w, sets, r_ref, ps.rows(), leaders, thr, 1e-8, float(np.float32(-0.01)), ps.flat)
    got, total = ts.download(), int(cnt.sum())
    assert np.array_equal(got["idx"][:total], idx) and np.array_equal(bits(got["sum"][:total]), bits(sm))
    assert np.array_equal(bits(got["w"]), bits(w))
    for p in range(W):
        assert np.array_equal(bits(got["r"][p]), bits(r_ref[p]))
