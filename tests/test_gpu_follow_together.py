"""Small tables: which steps take one launch for all workers, exchange and update.  GPU parity on both sides of the rule (6 to 9
workers with a gradient, a chunk of elements a layer, 140 chunks or 14 a worker besides two a layer, 256 tiles) on the top-k and the threshold route, and the launches that
each side makes: more workers on few elements go through the workers' own launch (32 workers on 30 k elements 29 us a step, 40
in one launch); quads that a layer's ends cut."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, ThresholdSet, assert_step_equal, bits

pytestmark = pytest.mark.gpu
TILE = 4096
W = 11
ENOUGH = {9: (140 + 2 * 2) * 1024, 11: (14 * 11 + 2 * 2) * 1024}    # elements, in two layers
CASES = [(8, 5 * TILE, True), (9, 5 * TILE, False), (9, ENOUGH[9] - 1, False), (9, ENOUGH[9], True), (11, ENOUGH[11] - 1, False),
         (11, ENOUGH[11], True), (11, 256 * TILE - 4091, True), (11, 256 * TILE - 4090, False)]


def _sizes(elements):
    return [elements - 2 * TILE - 5, 2 * TILE + 5]                 # the second takes three tiles


def _gradients(streaming):
    return [p if p < streaming else None for p in range(W)]


def _launches(iwp, kernel, call):
    iwp.timing_enable(kernel)
    call()
    return iwp.timing_collect()[1]


@pytest.mark.parametrize("streaming,elements,together", CASES)
def test_top_k(gpu_lib, streaming, elements, together):
    ps = wl.custom_set([(n, n // 50) for n in _sizes(elements)], W=W, seed=streaming, align=1, start=3)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    r_ref = [(x * np.float32(0.5)).astype(np.float32) for x in sets]
    gs = GpuSet(gpu_lib, ps, w.copy(), sets, r_np=[x.copy() for x in r_ref], fused=True, hint="none")
    g_ids = _gradients(streaming)
    for t, kernel in enumerate(("k_follow_sum", "k_follow_gather")):
        lead = np.array([3 + t, 10 - t], np.uint32)                # one without a gradient among them
        ref = oracle.step(w, sets, r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale),
                          accumulate_mask=[i is not None for i in g_ids])
        assert _launches(gpu_lib, kernel, lambda: gs.step(g_ids, lead)) == (1 if together == (t == 0) else 0)
        assert_step_equal(gs.download(), w, r_ref, *ref, ps.layers, tag="step %d" % t)


@pytest.mark.parametrize("streaming,elements,together", CASES)
def test_thresholds(gpu_lib, streaming, elements, together):
    ps = wl.custom_set([(n, 0) for n in _sizes(elements)], W=W, seed=streaming, align=1, start=3)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    r_ref = [(x * np.float32(0.5)).astype(np.float32) for x in sets]
    ts = ThresholdSet(gpu_lib, ps, w.copy(), sets, [x.copy() for x in r_ref], 2, ps.flat)
    g_ids = _gradients(streaming)
    thr = np.array([4 * np.median(np.abs(sets[0][L.offset:L.offset + L.n]) / (np.abs(w[L.offset:L.offset + L.n]) + 1e-8))
                    for L in ps.layers], np.float32)
    for t, kernel in enumerate(("k_follow_mask_sum", "k_follow_mask")):
        leaders = np.array([[3 + t, 10], [0, 9]], np.uint32)
        mask, cnt, idx, sm = oracle.step_threshold(w, sets, r_ref, ps.rows(), leaders, thr, 1e-8, float(np.float32(-0.01)), ps.flat,
                                                   accumulate_mask=[i is not None for i in g_ids])
        assert _launches(gpu_lib, kernel, lambda: ts.step(g_ids, leaders, thr, -0.01)) == (1 if together == (t == 0) else 0)
        got, total = ts.download(), int(cnt.sum())
        assert 0 < total < ps.flat and np.array_equal(got["mask"], mask)
        assert np.array_equal(got["idx"][:total], idx) and np.array_equal(bits(got["sum"][:total]), bits(sm))
        assert np.array_equal(bits(got["w"]), bits(w))
        for p in range(W):
            assert np.array_equal(bits(got["r"][p]), bits(r_ref[p])), p


def _step_and_route(gpu_lib, sizes, workers, streaming, start):
    ps = wl.custom_set([(n, (n + 1) // 2) for n in sizes], W=workers, seed=start, align=1, start=start)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(workers)]
    r_ref = [(x * np.float32(0.5)).astype(np.float32) for x in sets]
    gs = GpuSet(gpu_lib, ps, w.copy(), sets, r_np=[x.copy() for x in r_ref], fused=True, hint="none")
    g_ids = [p if p < streaming else None for p in range(workers)]
    lead = (np.arange(len(sizes)) % workers).astype(np.uint32)
    ref = oracle.step(w, sets, r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale), accumulate_mask=[i is not None for i in g_ids])
    launches = _launches(gpu_lib, "k_follow_sum", lambda: gs.step(g_ids, lead))
    assert_step_equal(gs.download(), w, r_ref, *ref, ps.layers)
    return launches


@pytest.mark.parametrize("streaming,last,together", [(6, 1, True), (7, 1023, False), (7, 1024, True), (8, 1023, False), (8, 1024, True)])
def test_short_layers(gpu_lib, streaming, last, together):
    assert _step_and_route(gpu_lib, [1024] * 5 + [last], 9, streaming, 1) == int(together)


@pytest.mark.parametrize("workers", [16, 32])
def test_many_workers_on_packed_layers(gpu_lib, workers):
    """60 packed layers of 270 k elements, 32 workers: 60 us a step in two launches, 72 in one."""
    assert _step_and_route(gpu_lib, [4500] * 60, workers, workers, 3) == 0


@pytest.mark.parametrize("start", range(16))
def test_cut_quads(gpu_lib, start):
    """Layers whose ends cut quads in every way, from layers shorter than a quad on."""
    assert _step_and_route(gpu_lib, [4, 3, 5, 6, 7, 8, 2, 13, 16, 1020, 1021, 1026, 1, 1039, 4093, 4099, 5], 6, 5, start) == 1
