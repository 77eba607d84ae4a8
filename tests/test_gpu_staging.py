"""GPU parity where the first look's mark, a key taken from a sample of the layer, can go wrong: lengths around the
sample's regimes (whole layer up to 16 runs of 256 elements, 16 to 64 runs beyond), evenly spread scores as in a long
run, all candidates of a layer in a few tiles (their slots overflow though the copies are complete), keys at the top
of the range (infinite scores, 0 / 0) and NaN among the layer's largest.  Layers of up to 32768 elements are sampled only
beside a longer one (alone, in the first and third test, they take the route that keeps a layer in registers): the last
test puts them there."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, assert_step_equal, sample_plan
from test_gpu_selection_paths import EPS, TILE, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 4095, 4097, 16384, 16385, 70_001, 40 * TILE + 3])
@pytest.mark.parametrize("keep", [0.001, 1 / 64, 0.05, 0.9])
def test_evenly_spread_scores(gpu_lib, n, keep):
    import torch
    rng = np.random.default_rng(n)
    w = (rng.standard_normal(n) * 0.05).astype(np.float32)
    r = (np.abs(w) * rng.uniform(-1, 1, n)).astype(np.float32)
    g = (rng.standard_t(3, n) * 1e-4).astype(np.float32)
    _check(gpu_lib, torch, w, g, r, max(1, int(n * keep)), "n=%d keep=%g" % (n, keep))


@pytest.mark.parametrize("tiles_with", [1, 3])
def test_all_candidates_in_a_few_tiles(gpu_lib, tiles_with):
    import torch
    n = 64 * TILE + 77
    rng = np.random.default_rng(tiles_with)
    w = np.ones(n, np.float32)
    r = (rng.uniform(0.1, 0.2, n)).astype(np.float32)
    for t in range(tiles_with):                              # tiles that the sample's runs pass through
        r[(20 * t + 1) * TILE:(20 * t + 2) * TILE] = rng.uniform(1.0, 1.01, TILE).astype(np.float32)
    for k in (n // 64, tiles_with * TILE, tiles_with * TILE - 1, 100):
        _check(gpu_lib, torch, w, np.zeros(n, np.float32), r, k, "tiles=%d k=%d" % (tiles_with, k))


@pytest.mark.parametrize("n", [3000, 9 * TILE + 5])
def test_keys_at_the_top_of_the_range(gpu_lib, n):
    import torch
    rng = np.random.default_rng(n)
    w = (rng.standard_normal(n) * 0.05).astype(np.float32)
    r = (rng.standard_normal(n)).astype(np.float32)
    zero = rng.choice(n, n // 8, replace=False)
    w[zero] = 0.0                                            # eps = 0: infinite scores ...
    r[zero[::2]] = 0.0                                       # ... and 0 / 0
    r[rng.choice(n, n // 50, replace=False)] = 3.0e38
    for k in (n // 64, n // 16, n // 8, n // 8 + n // 50, n // 2):
        _check(gpu_lib, torch, w, np.zeros(n, np.float32), r, k, "n=%d k=%d" % (n, k), eps=0.0)


SHORT = [1, 255, 256, 257, 3000, 4095, 4096, 4097, 16384, 16385, 20_000]


@pytest.mark.parametrize("route", ["whole_step", "three_calls"])
@pytest.mark.parametrize("keep", [0.001, 1 / 64, 0.05, 0.9])
@pytest.mark.parametrize("kind", ["spread", "top"])
def test_short_layers_beside_a_long_one(gpu_lib, route, keep, kind):
    sizes = [(n, max(1, int(n * keep))) for n in SHORT + [9 * TILE + 5]]
    runs = {n: len(sample_plan(n, k)[0]) for n, k in sizes}
    if keep == 0.001:
        assert runs[16384] == 64 and runs[16385] == 64 and runs[4096] == 16
    ps = wl.custom_set(sizes, W=2, seed=3, align=1, start=1)
    rng = np.random.default_rng(int(keep * 1000))
    w = wl.gen_weights(ps)
    r0 = [(np.abs(w) * rng.uniform(-1, 1, ps.flat)).astype(np.float32) for _ in range(2)]
    sets = [(rng.standard_t(3, ps.flat) * 1e-4).astype(np.float32) for _ in range(2)]
    if kind == "top":                                        # eps = 0: infinite scores and 0 / 0 among the largest
        zero = rng.choice(ps.flat, ps.flat // 8, replace=False)
        w[zero] = 0.0
        for x in r0 + sets:
            x[zero[::2]] = 0.0
    ps.eps = 0.0 if kind == "top" else EPS
    gs = GpuSet(gpu_lib, ps, w, sets, r_np=r0, fused=route == "whole_step", hint="none")
    w_ref, r_ref = w.copy(), [x.copy() for x in r0]
    for t in range(2):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % 2 for p in range(2)]
        ref = oracle.step(w_ref, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w_ref, r_ref, *ref, ps.layers, tag="%s keep=%g step %d" % (kind, keep, t))
