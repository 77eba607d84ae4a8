"""Tables of up to 512 tiles, or 1024 in 16 layers or more, have no sampled mark: the second look reads them again and copies whole bins of the first digit
into roomier slots.  GPU parity on both sides of that line: evenly spread scores, sorted ones, a pattern with the sample's
period (which misleads it above the line), all scores inside one bin (slots overflow); and the workspace of a layer still
serves every shorter one."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, assert_step_equal, sample_plan, sampled_mark
from test_gpu_selection_paths import EPS, TILE, _check


@pytest.mark.gpu
@pytest.mark.parametrize("n", [512 * TILE, 512 * TILE + 1])
@pytest.mark.parametrize("keep", [0.001, 1 / 64, 0.2])
def test_layer_on_both_sides(gpu_lib, n, keep):
    import torch
    rng = np.random.default_rng(n)
    k = int(n * keep)
    w = (rng.standard_normal(n) * 0.05).astype(np.float32)
    one, z = np.ones(n, np.float32), np.zeros(n, np.float32)
    g = (rng.standard_t(3, n) * 1e-4).astype(np.float32)
    _check(gpu_lib, torch, w, g, (np.abs(w) * rng.uniform(-1, 1, n)).astype(np.float32), k, "evenly spread")
    base = (np.abs(rng.standard_t(3, n)) * 1e-3 + 1e-6).astype(np.float32)
    _check(gpu_lib, torch, one, z, np.sort(base), k, "sorted")
    _check(gpu_lib, torch, one, z, rng.uniform(1.0, 1.05, n).astype(np.float32), k, "one bin")
    r = (base * np.float32(1e-3)).astype(np.float32)
    for s in sample_plan(n, k)[0]:
        r[s * 256:s * 256 + 64] = (5.0 + rng.random(64)).astype(np.float32)
    if keep < 0.2:
        assert sampled_mark(one, r, n, k, EPS) > int(np.sort(r.view(np.uint32))[n - k]), "the mark misses candidates"
    _check(gpu_lib, torch, one, z, r, k, "period of the sample")


@pytest.mark.gpu
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("last", [TILE, TILE + 1])
@pytest.mark.parametrize("layers", [4, 15, 16])
def test_table_on_both_sides(gpu_lib, fused, last, layers):
    W = 2
    sizes = [(300 * TILE - 7, 50_000), (100 * TILE, 300), (111 * TILE - 1, 0), (last, last // 2)]
    if layers > 4:                                           # 1024 or 1025 tiles
        sizes = [((512 - (layers - 5)) * TILE, 9000)] + [(TILE - j, 40) for j in range(layers - 5)] + sizes
    ps = wl.custom_set(sizes, W=W, seed=last, align=1, start=1)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    gs = GpuSet(gpu_lib, ps, w, sets, fused=fused, hint="none")
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    for t in range(3):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % W for p in range(W)]
        ref = oracle.step(w, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w, r_ref, *ref, ps.layers, tag="last %d step %d" % (last, t))


def test_a_layers_workspace_serves_shorter_ones():
    from paper_1901_01544_amd import iwp
    for keep in (0.001, 1 / 64, 0.2):
        need = [iwp.workspace_bytes(n, int(n * keep)) for n in range(TILE, 700 * TILE, 16 * TILE)]
        assert all(a <= b for a, b in zip(need, need[1:]))
