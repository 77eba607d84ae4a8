"""GPU parity of the one-launch route for tables whose layers all have at most 32768 elements, and of the first sizes
beyond it: lengths around a chunk (4096), the two instantiations (16384, 32768) and the line itself; ties at the cut,
zeros of both signs, every element kept; whole steps with layers that keep nothing and workers without a gradient."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, assert_step_equal
from test_gpu_selection_paths import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 63, 4095, 4096, 4097, 16383, 16384, 16385, 32767, 32768, 32769])
@pytest.mark.parametrize("kind", ["spread", "quantised", "zeros"])
def test_single_layers(gpu_lib, n, kind):
    import torch
    rng = np.random.default_rng(n)
    w = (rng.standard_normal(n) * 0.05).astype(np.float32)
    r = (rng.standard_t(3, n) * 1e-3).astype(np.float32)
    g = (rng.standard_t(3, n) * 1e-3).astype(np.float32)
    if kind == "quantised":
        w = np.ones(n, np.float32)
        r, g = np.round(r * 1000).astype(np.float32), np.round(g * 1000).astype(np.float32)
    if kind == "zeros":
        r[n // 20:], g[n // 20:] = 0.0, 0.0
        r[n // 2::3] = -0.0
        g[n // 2::3] = -0.0
    for k in sorted({1, max(1, n // 64), max(1, n // 2), n}):
        _check(gpu_lib, torch, w, g, r, k, "%s n=%d k=%d" % (kind, n, k))


@pytest.mark.parametrize("top", [4096, 16384, 32768, 32769])
@pytest.mark.parametrize("fused", [False, True])
def test_tables(gpu_lib, top, fused):
    sizes = [(top, top // 40), (1, 1), (300, 5), (4097 if top > 4096 else 4095, 100), (700, 0), (top - 1, top - 1), (64, 64)]
    ps = wl.custom_set(sizes, W=3, seed=top, align=1, start=3, zero_frac=0.05)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(3)]
    gs = GpuSet(gpu_lib, ps, w, sets, fused=fused, hint="previous")
    w_ref = w.copy()
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(3)]
    for t in range(3):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % 3 for p in range(3)]
        ref = oracle.step(w_ref, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w_ref, r_ref, *ref, ps.layers, tag="top %d step %d" % (top, t))
