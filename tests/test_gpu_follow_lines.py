"""GPU parity of the followers' tiles whose residuals do not start at a multiple of 64 bytes: every start of a layer in a line,
half of the elements sent (so that all lanes' quads, and the single elements at a tile's ends, hold sent ones), gradients
that start elsewhere in a line than residuals; on tables of both routes of the workers' pass (one launch for all workers on
small ones)."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, ThresholdSet, assert_step_equal, bits

pytestmark = pytest.mark.gpu
SIZES = [2 * 4096 + 5, 4096, 4095, 9 * 4096 + 17, 1, 3, 17, 1023, 1025]
LONG = 260 * 4096 + 11                                         # takes the table past the small ones
W = 3


def _grads_elsewhere(sets, by):
    import torch
    out = []
    for g in sets:
        big = torch.zeros(len(g) + by, dtype=torch.float32, device="cuda:0")
        big[by:].copy_(torch.from_numpy(g))
        out.append(big[by:])
    return out


@pytest.mark.parametrize("small", [True, False])
@pytest.mark.parametrize("start", range(16))
def test_top_k_steps(gpu_lib, start, small):
    ps = wl.custom_set([(n, (n + 1) // 2) for n in SIZES] + [(40000 if small else LONG, 400)], W=W, seed=start + 1, align=1, start=start)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    for fused in (True, False):
        gs = GpuSet(gpu_lib, ps, w, sets, fused=fused, hint="none", grads_dev=_grads_elsewhere(sets, start % 3))
        w_ref = w.copy()
        r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
        for t in range(2):
            lead = wl.leaders(ps, t)
            ids = [(p + t) % W for p in range(W)]
            ref = oracle.step(w_ref, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
            gs.step(ids, lead)
            assert_step_equal(gs.download(), w_ref, r_ref, *ref, ps.layers, tag="start %d step %d" % (start, t))


@pytest.mark.parametrize("small", [True, False])
@pytest.mark.parametrize("start", range(16))
def test_threshold_steps(gpu_lib, start, small):
    sizes = SIZES + ([] if small else [LONG])
    ps = wl.custom_set([(n, 0) for n in sizes], W=W, seed=start + 1, align=1, start=start)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    w_ref = w.copy()
    ts = ThresholdSet(gpu_lib, ps, w, sets, r_ref, 1, ps.flat)
    leaders = np.array([[j % W] for j in range(len(sizes))], np.uint32)
    thr = np.array([np.median(np.abs(sets[j % W][L.offset:L.offset + L.n]) / (np.abs(w[L.offset:L.offset + L.n]) + 1e-8))
                    for j, L in enumerate(ps.layers)], np.float32)
    for t in range(2):
        ts.step(list(range(W)), leaders, thr, -0.01)
        mask, cnt, idx, sm = oracle.step_threshold(w_ref, sets, r_ref, ps.rows(), leaders, thr, 1e-8,
                                                   float(np.float32(-0.01)), ps.flat)
        got, total = ts.download(), int(cnt.sum())
        assert total > ps.flat // 4
        assert np.array_equal(got["idx"][:total], idx) and np.array_equal(bits(got["sum"][:total]), bits(sm))
        assert np.array_equal(bits(got["w"]), bits(w_ref))
        for p in range(W):
            assert np.array_equal(bits(got["r"][p]), bits(r_ref[p]))
