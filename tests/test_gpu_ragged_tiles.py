"""GPU parity of look 1's ragged tiles: the last quad of a layer crossing its end by one, two and three elements, layers of
fewer than four elements on a table that takes the long route, at every alignment of the layer's start."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, assert_step_equal

pytestmark = pytest.mark.gpu
LONG = 9 * 4096


@pytest.mark.parametrize("start", [0, 1, 2, 3])
@pytest.mark.parametrize("fused", [False, True])
def test_ends_of_layers(gpu_lib, start, fused):
    sizes = [(LONG + d, (LONG + d) // 50) for d in (0, 1, 2, 3, 5)] + [(n, 1) for n in (1, 2, 3, 4, 5, 7, 1023, 1025)]
    ps = wl.custom_set(sizes, W=2, seed=start + 1, align=1, start=start, zero_frac=0.01)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(2)]
    gs = GpuSet(gpu_lib, ps, w, sets, fused=fused, hint="none")
    w_ref = w.copy()
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(2)]
    for t in range(2):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % 2 for p in range(2)]
        ref = oracle.step(w_ref, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w_ref, r_ref, *ref, ps.layers, tag="start %d step %d" % (start, t))
