"""GPU parity of the threshold modes, and of the three-call route, where a layer ends within a tile's first chunk of 1024 elements (such tiles take a shorter
path): on the edge and one element to either side, as a layer's only tile and as its last, at every alignment."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, ThresholdSet, assert_step_equal, bits

pytestmark = pytest.mark.gpu
SIZES = [1, 3, 55, 1020, 1023, 1024, 1025, 1027, 2048, 4095, 4096, 4097, 4096 + 1023, 4096 + 1024, 4096 + 1025, 8192 + 5]


@pytest.mark.parametrize("start", [0, 1, 2, 3])
@pytest.mark.parametrize("mode", ["threshold", "random", "layerwise"])
def test_layers_around_the_first_chunk(gpu_lib, start, mode):
    W, n_lead, eps, scale = 3, 2, 1e-8, np.float32(-0.01)
    ps = wl.custom_set([(n, 0) for n in SIZES], W=W, seed=start + 1, align=1, start=start, zero_frac=0.01)
    rng = np.random.default_rng(start)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    r0 = [(rng.standard_t(3, ps.flat) * 1e-3).astype(np.float32) for _ in range(W)]
    nl, cap = len(ps.layers), ps.flat + 8
    ts = ThresholdSet(gpu_lib, ps, w, sets, r0, n_lead, cap)
    w_ref, r_ref = w.copy(), [x.copy() for x in r0]
    for t in range(2):
        ids = [0, None if t else 1, 2]                       # one worker without a gradient in the second step
        g = [sets[i] if i is not None else np.zeros(1, np.float32) for i in ids]
        acc = [i is not None for i in ids]
        chosen = rng.integers(0, W, (nl, n_lead)).astype(np.uint32)
        rnd = (99, t) if mode == "random" else None
        if mode == "layerwise":
            ts.step_layerwise(ids, chosen, 0.05, 1e-4, 1e3, scale)
            thr = np.ascontiguousarray(ts.thr_slots.cpu().numpy().reshape(nl, n_lead))
        else:
            thr = np.full(nl, 0.02, np.float32)
            ts.step(ids, chosen, thr, scale, random=rnd)
        mask, cnt, idx, total = oracle.step_threshold(w_ref, g, r_ref, ps.rows(), chosen, thr, eps, float(scale), cap,
                                                      accumulate_mask=acc, random=rnd)
        got, n = ts.download(), int(cnt.sum())
        tag = "%s start %d step %d" % (mode, start, t)
        assert 0 < n and np.array_equal(got["count"][:nl], cnt) and got["count"][nl] == n, tag
        assert np.array_equal(got["mask"], mask) and np.array_equal(got["idx"][:n], idx), tag
        assert np.array_equal(bits(got["sum"][:n]), bits(total)) and np.array_equal(bits(got["w"]), bits(w_ref)), tag
        for p in range(W):
            assert np.array_equal(bits(got["r"][p]), bits(r_ref[p])), "%s residual %d" % (tag, p)


@pytest.mark.parametrize("start", [0, 1, 2, 3])
def test_three_calls_around_the_first_chunk(gpu_lib, start):
    W = 3
    ps = wl.custom_set([(n, (n + 3) // 4) for n in SIZES], W=W, seed=start + 1, align=1, start=start, zero_frac=0.01)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    gs = GpuSet(gpu_lib, ps, w.copy(), sets, fused=False, hint="none")
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    for t in range(2):
        ids, lead = [(p + t) % W for p in range(W)], wl.leaders(ps, t)
        ref = oracle.step(w, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w, r_ref, *ref, ps.layers, tag="step %d" % t)
