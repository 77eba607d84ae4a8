"""Threshold modes: what the chosen nodes hand over from the mask pass (a slot of values per tile and node) on both sides of
the slot's size, with and without an exchange, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import ThresholdSet, bits

pytestmark = pytest.mark.gpu
TILE = 4096
# per tile of the first layer, around the slot's size (64 and four times the capacity over the tiles, 1024 at most); then 700
# elements of which 5; by the tiles of a further layer that sends nothing
SENT = {0: [1023, 1024, 1025, TILE, 0, 1], 300: [123, 124, 125, TILE, 0, 1]}


@pytest.mark.parametrize("short", [0, 1])                      # capacity exactly the total, or one pair less
@pytest.mark.parametrize("n_lead", [1, 2, 3, 4])
@pytest.mark.parametrize("layerwise", [False, True])
@pytest.mark.parametrize("long", [0, 300])                     # a small table, and one past them
def test_slot_edges(gpu_lib, n_lead, short, layerwise, long):
    W = 5
    ps = wl.custom_set([(TILE * len(SENT[long]) + 700, 0), (900, 0)] + [(TILE * long, 0)] * (long > 0), W=W, seed=5, align=1, start=3)
    rng = np.random.default_rng(n_lead)
    L0, L1 = ps.layers[:2]
    w = np.ones(ps.flat, np.float32)
    pool = [(rng.standard_normal(ps.flat) * 1e-3).astype(np.float32) for _ in range(W)]
    r0 = [(rng.standard_normal(ps.flat) * 1e-3).astype(np.float32) for _ in range(W)]
    sent = np.zeros(ps.flat, bool)
    for t, n in enumerate(SENT[long] + [5]):
        room = min(TILE, L0.n - t * TILE)
        sent[L0.offset + t * TILE + rng.choice(room, n, replace=False)] = True
    sent[L1.offset:L1.offset + 3] = True
    leaders = np.array([[0, 1, 2, 3][:n_lead], [3, 0, 3, 2][:n_lead], [1, 1, 0, 2][:n_lead]][:len(ps.layers)], np.uint32)
    lines = np.full(len(ps.layers), 2.0, np.float32)
    for j, L in enumerate(ps.layers[:2]):                          # each sent element lies above the line on one chosen node
        at = L.offset + np.flatnonzero(sent[L.offset:L.offset + L.n])
        for i, p in zip(at, rng.choice(leaders[j], len(at))):
            r0[p][i] += 4.0 if i % 2 else -4.0
    total, cap = int(sent.sum()), int(sent.sum()) - short
    tiles = sum(-(-L.n // TILE) for L in ps.layers)
    assert SENT[long][1] == min(1024, 64 + 4 * -(-cap // tiles))
    g_ids = [0, 1, None, 3, None]                              # node 2: chosen without a gradient; node 4: never chosen
    zero = np.zeros(1, np.float32)
    g_np = [zero if i is None else pool[i] for i in g_ids]
    acc = [i is not None for i in g_ids]
    w_ref, r_ref = w.copy(), [x.copy() for x in r0]
    ts = ThresholdSet(gpu_lib, ps, w, pool, r0, n_lead, cap)
    if layerwise:                                              # the rule gives 2 whatever the statistics are
        ts.step_layerwise(g_ids, leaders, 2.0, 0.0, 1.0, np.float32(-0.01))
        assert np.all(ts.thr_slots.cpu().numpy() == 2.0)
    else:
        ts.step(g_ids, leaders, lines, np.float32(-0.01))
    mask, cnt, idx, sm = oracle.step_threshold(w_ref, g_np, r_ref, ps.rows(), leaders, lines, 1e-8,
                                               float(np.float32(-0.01)), total, accumulate_mask=acc)
    assert int(cnt.sum()) == total
    got = ts.download()
    assert np.array_equal(got["mask"], mask)
    assert got["count"].tolist() == cnt.tolist() + [total, short]
    if short:                                                  # accumulated, nothing exchanged or cleared
        w_ref, r_ref = w.copy(), [x.copy() for x in r0]
        for p in range(W):
            if acc[p]:
                oracle.accumulate(r_ref[p][3:], pool[p][3:])
        assert np.all(got["idx"] == 0xFFFFFFFF) and np.all(np.isnan(got["sum"]))
    else:
        assert np.array_equal(got["idx"][:total], idx)
        assert np.array_equal(bits(got["sum"][:total]), bits(sm))
    assert np.array_equal(bits(got["w"]), bits(w_ref))
    for p in range(W):
        assert np.array_equal(bits(got["r"][p]), bits(r_ref[p])), p
