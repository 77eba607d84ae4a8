"""Copies of the first-digit histogram: layers on both sides of the lines where their number changes (with and without a
launch of its own for the pick), and plans that fit the library's static scratch only with fewer copies."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import GpuSet, assert_step_equal, bits

pytestmark = pytest.mark.gpu
TILE = 4096
EPS = 1e-8


@pytest.mark.parametrize("tiles", [[128, 129], [256, 257, 3], [512, 513, 1025, 1]])
def test_edges(gpu_lib, tiles):
    ps = wl.custom_set([(t * TILE - 1, t * 40) for t in tiles], W=2, seed=len(tiles), align=64)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(2)]
    gs = GpuSet(gpu_lib, ps, w, sets, fused=True, hint="previous")
    w_ref = w.copy()
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(2)]
    for t in range(2):
        lead = wl.leaders(ps, t)
        ids = [(p + t) % 2 for p in range(2)]
        ref = oracle.step(w_ref, [sets[i] for i in ids], r_ref, ps.rows(), lead, float(ps.eps), float(ps.scale))
        gs.step(ids, lead)
        assert_step_equal(gs.download(), w_ref, r_ref, *ref, ps.layers, tag="step %d" % t)


def test_largest_plan_of_the_static_scratch(gpu_lib):
    """The longest third layer with which the plan still fits: fits only with the few copies, and gives the oracle's pairs."""
    import torch
    iwp = gpu_lib

    def rows(last):
        out, off, k0 = [], 0, 0
        for n in (513 * TILE, 513 * TILE, last * TILE):
            out.append((off, n, n // 2, k0))
            off, k0 = off + n, k0 + n // 2
        return out

    def fits(last):
        return iwp.Plan(rows(last)).workspace_bytes <= iwp.IWP_STATIC_SCRATCH_BYTES

    lo, hi = 1, 513
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if fits(mid) else (lo, mid)
    few = iwp.Plan(rows(lo))
    # with all copies 16 KiB for each of 6 + 6 (8 instead of 2) and, above 128 tiles, at least one more
    assert few.workspace_bytes + 13 * 16384 > iwp.IWP_STATIC_SCRATCH_BYTES and lo > 128
    n = 2 * 513 * TILE + lo * TILE
    K = n // 2
    rng = np.random.default_rng(3)
    w, g = rng.standard_normal(n).astype(np.float32), rng.standard_t(3, n).astype(np.float32)
    r = np.zeros(n, np.float32)
    d = lambda x: torch.from_numpy(x).to("cuda:0")
    wd, gd, rd = d(w), d(g), d(r)
    idx = torch.full((K,), -1, dtype=torch.int32, device="cuda:0")
    val = torch.zeros(K, dtype=torch.float32, device="cuda:0")
    iwp.compress_segmented_static(few, wd, [gd], [rd], None, EPS, idx, val, None)
    torch.cuda.synchronize()
    score = np.abs(g) / (np.abs(w) + np.float32(EPS))
    want = []
    for off, m, k, _ in rows(lo):
        s = score[off:off + m]
        want.append(off + np.sort(np.argsort(-s, kind="stable")[:k]))
    want = np.concatenate(want)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(bits(val.cpu().numpy()), bits(g[want]))
