"""Tables on both sides of the lines at which look 1 and the records' pass change form: 40 MiB a buffer, 64 and 160 MiB where look 1
accumulates, 160 MiB where it only reads (what is left in the memory-side cache, threads per tile)."""
import numpy as np
import pytest

import oracle
from harness import bits
from test_gpu_selection_paths import _check

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("mib", [40, 64, 160])
@pytest.mark.parametrize("more", [0, 1])
def test_compress_layer(gpu_lib, mib, more):
    import torch
    n = (mib << 18) + more
    rng = np.random.default_rng(mib)
    w = rng.standard_normal(n, dtype=np.float32)
    g = rng.standard_normal(n, dtype=np.float32)
    r = rng.standard_normal(n, dtype=np.float32)
    _check(gpu_lib, torch, w, g, r, n // 100, "%d MiB and %d" % (mib, more))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n", [9 * 4096 - 5, 9 * 4096 + 2049, (40 << 18) - 1, (40 << 18) + 1, (160 << 18) + 1])
def test_threshold_and_pairs(gpu_lib, n):
    import torch
    rng = np.random.default_rng(n)
    w = rng.standard_normal(n, dtype=np.float32)
    r = rng.standard_normal(n, dtype=np.float32)
    k = n // 100
    wd, rd = torch.from_numpy(w).cuda(), torch.from_numpy(r).cuda()
    thr = torch.zeros(3, dtype=torch.int32, device="cuda")
    idx, val = torch.full((k,), -1, dtype=torch.int32, device="cuda"), torch.zeros(k, device="cuda")
    ws = torch.empty(gpu_lib.workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    gpu_lib.select_threshold(wd, rd, k, 1e-8, thr, ws)
    gpu_lib.compact_pairs(wd, rd, 1e-8, thr, k, idx, val, ws)
    torch.cuda.synchronize()
    ref_idx, ref_val, _ = oracle.compress_layer(w, np.zeros(n, np.float32), r.copy(), k, 1e-8)
    assert np.array_equal(idx.cpu().numpy().view(np.uint32), ref_idx)
    assert np.array_equal(bits(val.cpu().numpy()), bits(ref_val))
