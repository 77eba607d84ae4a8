"""Tables of up to 512 tiles, or 1024 in 16 layers or more, have no sampled mark (steps and compressions of a table at momentum 1
without a hint excepted): the second look reads them again and copies whole bins of the first digit
into roomier slots.  GPU parity on both sides of that line: evenly spread scores, sorted ones, a pattern with the sample's
period (which misleads it above the line), all scores inside one bin (slots overflow); tables, and from the selection state that
the call leaves in its workspace that they took the route they are meant to; and the workspace of a layer still
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


def _staging_bins(gs):
    """The first digit from which look 1 copied out, per layer (0xFFFFFFFF: nothing), as the last call left it in its workspace:
    a table of two rows of 56 bytes, the layers' histograms (one copy of the first digit's per 128 tiles, 16 at most, and 1536
    words), nine words of state per layer, each part in whole blocks of 256 bytes."""
    def whole(x):
        return -(-x // 256) * 256
    words = 0
    for L in gs.ps.layers:
        copies = 1
        while L.k and copies < 16 and copies * 128 < -(-L.n // TILE):
            copies *= 2
        words += copies * 4096 + 1536
    at = whole(2 * 56) + whole(4 * words)
    state = gs.ws[at:at + 36 * len(gs.ps.layers)].cpu().numpy().view(np.uint32).reshape(-1, 9)
    return state[:, 6]


@pytest.mark.gpu
@pytest.mark.parametrize("momentum", [1.0, 0.9])
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("last", [TILE, TILE + 1])
@pytest.mark.parametrize("layers", [4, 15, 16])
def test_table_on_both_sides(gpu_lib, fused, last, layers, momentum):
    W = 2
    sizes = [(300 * TILE - 7, 50_000), (100 * TILE, 300), (111 * TILE - 1, 0), (last, last // 2)]
    if layers > 4:                                           # 1024 or 1025 tiles
        sizes = [((512 - (layers - 5)) * TILE, 9000)] + [(TILE - j, 40) for j in range(layers - 5)] + sizes
    ps = wl.custom_set(sizes, W=W, seed=last, align=1, start=1)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    gs = GpuSet(gpu_lib, ps, w, sets, fused=fused, hint="none")
    gs.plan.set_momentum(momentum)
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    tiles = sum(-(-n // TILE) for n, _ in sizes)
    assert tiles in (512, 513, 1024, 1025) and len(sizes) == layers
    sampled = momentum == 1.0 or tiles > (1024 if layers >= 16 else 512)
    for t in range(3):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % W for p in range(W)]
        ref = oracle.step(w, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale), momentum=momentum)
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w, r_ref, *ref, ps.layers, tag="last %d step %d" % (last, t))
        for L, staged in zip(ps.layers, _staging_bins(gs)):
            assert L.k == 0 or (staged != 0xFFFFFFFF) == sampled


def test_a_layers_workspace_serves_shorter_ones():
    from paper_1901_01544_amd import iwp
    for keep in (0.001, 1 / 64, 0.2):
        need = [iwp.workspace_bytes(n, int(n * keep)) for n in range(TILE, 700 * TILE, 16 * TILE)]
        assert all(a <= b for a, b in zip(need, need[1:]))
