"""compact_pairs on layers of less than a quad, where the ordered split reads the layer itself (half or more of it is kept, or the
record's threshold is zero): only the layer's own elements count, whatever lies behind them.  The layers lie inside a larger buffer."""
import numpy as np
import pytest

import oracle
from harness import bits

pytestmark = pytest.mark.gpu
EPS = 1e-8
BEHIND = 5000                                                   # elements behind the layers


def _expected(keys, key, quota, k):
    ties = np.cumsum(keys == key)
    return np.nonzero((keys > key) | ((keys == key) & (ties <= quota)))[0][:k]


@pytest.mark.parametrize("alone", [True, False])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 4096 + 3])
def test_only_the_layers_own_elements(gpu_lib, n, alone):
    import torch
    iwp = gpu_lib
    rng = np.random.default_rng(n)
    layers = 1 if alone else 3
    at = [7 + j * (n + 1) for j in range(layers)]
    flat = at[-1] + n + BEHIND
    r = rng.uniform(90.0, 99.0, flat).astype(np.float32)         # scores between the layers and behind them: all above the layers' own
    for o in at:
        r[o:o + n] = rng.uniform(1.0, 2.0, n)
    w = np.ones(flat, np.float32)
    wd, rd = torch.from_numpy(w).cuda(), torch.from_numpy(r).cuda()
    keys = [oracle.score(w[o:o + n], r[o:o + n], EPS).view(np.uint32).astype(np.int64) for o in at]
    between = int(np.float32(50.0).view(np.uint32))              # above every score of the layers, below all others
    for k in sorted({n, max(1, n - 1), max(1, n // 2), (n + 1) // 2}):
        plan = iwp.Plan([(o, n, k, j * k) for j, o in enumerate(at)])
        ws = torch.empty(max(plan.workspace_bytes, iwp.workspace_bytes(n, k)), dtype=torch.uint8, device="cuda")
        smallest = int(min(x.min() for x in keys))
        for key, quota in ((between, 0), (between, n), (0, 0), (0, n), (smallest, n), (smallest, 0), (int(keys[0][n // 2]), 1),
                           (0x7FFFFFFF, n), (0x80000000, n), (0xFFFFFFFF, n)):
            thr = torch.tensor([key, 0, quota] * layers, dtype=torch.int64, device="cuda").to(torch.int32)
            idx = torch.full((layers * k,), -1, dtype=torch.int32, device="cuda")
            val = torch.full((layers * k,), -7.0, device="cuda")
            if alone:
                iwp.compact_pairs(wd[at[0]:], rd[at[0]:], EPS, thr, k, idx, val, ws, n=n)
            else:
                iwp.compact_pairs_segmented(plan, wd, rd, EPS, thr, idx, val, ws)
            torch.cuda.synchronize()
            got, gv = idx.cpu().numpy(), val.cpu().numpy()
            for j, o in enumerate(at):
                tag = "n=%d k=%d key=%#x quota=%d layer %d" % (n, k, key, quota, j)
                take = _expected(keys[j], key, quota, k)
                mine, mv = got[j * k:(j + 1) * k], gv[j * k:(j + 1) * k]
                assert np.array_equal(mine[:take.size], take + (0 if alone else o)), tag
                assert np.array_equal(bits(mv[:take.size]), bits(r[o + take])), tag
                assert (mine[take.size:] == -1).all() and (mv[take.size:] == -7.0).all(), tag
    assert np.array_equal(bits(rd.cpu().numpy()), bits(r))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 4097])
@pytest.mark.parametrize("key", [0x7FFFFFFE, 0x7FFFFFFF, 0x80000000, 0xFFFFFFFF])
def test_record_above_every_key_of_a_layer_that_is_read_again(gpu_lib, n, key):
    import torch
    r, w = torch.rand(n, device="cuda"), torch.ones(n, device="cuda")
    for k in {n, (n + 1) // 2}:
        thr = torch.from_numpy(np.array([key, 0, k], np.uint32).view(np.int32)).cuda()
        idx, val = torch.full((k,), -7, dtype=torch.int32, device="cuda"), torch.full((k,), -7.0, device="cuda")
        ws = torch.empty(gpu_lib.workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
        gpu_lib.compact_pairs(w, r, EPS, thr, k, idx, val, ws)
        torch.cuda.synchronize()
        assert bool((idx == -7).all()) and bool((val == -7.0).all()), (n, k)
