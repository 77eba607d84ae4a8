"""Four to eight chosen nodes, whose masks are taken by two to four groups of threads in a workgroup: GPU parity for every number
(odd ones leave half a group idle), nodes listed twice inside a group and across groups, nodes without a gradient, tiles that end
within their first chunk, both routes of the workers' pass; and the time against two nodes."""
import statistics

import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import ThresholdSet, bits

pytestmark = pytest.mark.gpu
TILE = 4096


@pytest.mark.parametrize("long", [0, 260])                     # a small table, and one past them
@pytest.mark.parametrize("random", [False, True])
@pytest.mark.parametrize("n_lead", [4, 5, 6, 7, 8])
def test_parity(gpu_lib, n_lead, random, long):
    W = 9
    sizes = [3 * TILE + 17, 900, 1, TILE, 1025] + [long * TILE - 3] * (long > 0)
    ps = wl.custom_set([(n, 0) for n in sizes], W=W, seed=n_lead, align=1, start=3)
    w = wl.gen_weights(ps)
    sets = [wl.gen_gradient(ps, s) for s in range(W)]
    order = [7, 2, 2, 8, 7, 0, 3, 1]                           # 2 twice in a group and 7 in two groups, as far as they are listed
    leaders = np.array([np.roll(order, j)[:n_lead] for j in range(len(sizes))], np.uint32)
    g_ids = [None if p == 3 else p for p in range(W)]
    acc = [i is not None for i in g_ids]
    r_ref = [(s * np.float32(0.5)).astype(np.float32) for s in sets]
    w_ref = w.copy()
    ts = ThresholdSet(gpu_lib, ps, w, sets, [x.copy() for x in r_ref], n_lead, ps.flat)
    thr = np.array([4 * np.median(np.abs(sets[0][L.offset:L.offset + L.n]) / (np.abs(w[L.offset:L.offset + L.n]) + 1e-8))
                    for L in ps.layers], np.float32)
    for t in range(2):
        rnd = (11, t) if random else None
        ts.step(g_ids, leaders, thr, -0.01, random=rnd)
        mask, cnt, idx, sm = oracle.step_threshold(w_ref, sets, r_ref, ps.rows(), leaders, thr, 1e-8, float(np.float32(-0.01)),
                                                   ps.flat, accumulate_mask=acc, random=rnd)
        got, total = ts.download(), int(cnt.sum())
        assert 0 < total < ps.flat
        assert np.array_equal(got["mask"], mask) and got["count"].tolist() == cnt.tolist() + [total, 0]
        assert np.array_equal(got["idx"][:total], idx) and np.array_equal(bits(got["sum"][:total]), bits(sm))
        assert np.array_equal(bits(got["w"]), bits(w_ref))
        for p in range(W):
            assert np.array_equal(bits(got["r"][p]), bits(r_ref[p])), p


def test_time(gpu_lib):
    """1.2 M elements in six layers, eight workers: a step with eight chosen nodes takes at most 1.7 times one with two (1.2
    measured; 2.2 if a workgroup takes the nodes one after the other)."""
    import torch
    iwp, W, dev = gpu_lib, 8, "cuda"
    n, layers = 200_000, 6
    P = n * layers
    plan = iwp.Plan([(j * n, n, 0, 0) for j in range(layers)])
    gen = torch.Generator(device=dev).manual_seed(1)
    w = torch.randn(P, device=dev, generator=gen)
    pool = [torch.randn(P, device=dev, generator=gen) * 1e-3 for _ in range(W)]
    thr = torch.full((layers,), 0.15, device=dev)
    took = {}
    for n_lead in (2, 8):
        leaders = torch.arange(n_lead, dtype=torch.int32, device=dev).repeat(layers)
        r = [torch.zeros(P, device=dev) for _ in range(W)]
        mask = torch.zeros(plan.mask_bytes, dtype=torch.uint8, device=dev)
        count = torch.zeros(layers + 2, dtype=torch.int32, device=dev)
        idx, total = torch.zeros(P, dtype=torch.int32, device=dev), torch.zeros(P, device=dev)
        ws = torch.empty(plan.threshold_workspace_bytes(W, n_lead, P // 2), dtype=torch.uint8, device=dev)

        def steps():
            for _ in range(10):
                iwp.step_threshold_segmented(plan, w, pool, r, leaders, n_lead, thr, 1e-8, 0.0, mask, count, idx, total, P // 2, ws)
        steps()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            steps()
        times = []
        for _ in range(20):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            stop.record()
            stop.synchronize()
            times.append(start.elapsed_time(stop) * 100)
        took[n_lead] = statistics.median(times[3:])
        assert int(count[layers + 1]) == 0 and int(count[layers]) > 0
    print("two nodes %.1f us, eight %.1f us" % (took[2], took[8]))
    assert took[8] < 1.7 * took[2]
