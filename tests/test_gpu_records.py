"""Selections whose split finds the threshold's last digit itself, from what the third look left of every tile (up to 512 tiles)
or super-tile: scores that share 22 bits with the threshold, its last digit the lowest, a middle one and the highest of 512, spread
over the layer and crowded at the borders of super-tiles; layers whose records fit their histograms, just do not, and do not."""
import numpy as np
import pytest

import oracle
from harness import bits
from test_gpu_selection_paths import TILE, _check

pytestmark = pytest.mark.gpu
GROUP = np.uint32(0x3F840000)                                   # 1.03125: the first of 512 keys that share 22 bits


def _scores(rng, n, where):
    """A tenth of the elements in the group, or 1600 at every border between super-tiles; a hundredth above it, the rest below."""
    r = rng.uniform(0.1, 0.9, n).astype(np.float32)
    at = rng.choice(n, n // 10, replace=False) if where == "spread" else np.flatnonzero((np.arange(n) + 800) % (8 * TILE) < 1600)
    r[at] = (GROUP + rng.integers(0, 512, at.size).astype(np.uint32)).view(np.float32)
    r[rng.choice(n, n // 100, replace=False)] = np.float32(2.0)
    return r


@pytest.mark.timeout(300)
@pytest.mark.parametrize("where", ["spread", "borders"])
@pytest.mark.parametrize("tiles", [9, 512, 513, 2047, 2049, 2600])
def test_last_digit(gpu_lib, tiles, where):
    import torch
    n = tiles * TILE - 3
    rng = np.random.default_rng(tiles)
    one, z = np.ones(n, np.float32), np.zeros(n, np.float32)
    r = _scores(rng, n, where)
    key = r.view(np.uint32)
    above, low = int((key >= GROUP + 512).sum()), key[(key >= GROUP) & (key < GROUP + 512)] - GROUP
    for digit in (0, 200, 511):                                  # k ends among the elements of that digit
        k = above + int((low > digit).sum()) + int((low == digit).sum()) // 2
        assert k * 8 < n                                         # slots few enough for the records
        _check(gpu_lib, torch, one, z, r, k, "tiles=%d %s digit %d" % (tiles, where, digit))


@pytest.mark.parametrize("keep", [0.12, 0.13])
def test_both_sides_of_the_line(gpu_lib, keep):
    """Tables that keep an eighth of a layer or less go by the records, others count the tiles in a launch of their own."""
    import torch
    iwp = gpu_lib
    rng = np.random.default_rng(5)
    sizes = [600 * TILE + 5, 7, 40 * TILE]
    rows, off, out = [], 0, 0
    for n in sizes:
        k = max(1, int(n * keep)) if n > 7 else 0
        rows.append((off, n, k, out))
        off, out = off + n, out + k
    w, r = np.ones(off, np.float32), _scores(rng, off, "spread")
    plan = iwp.Plan(rows)
    d = lambda x: torch.from_numpy(x).cuda()
    wd, rd = d(w), d(r)
    idx, val = torch.full((out,), -1, dtype=torch.int32, device="cuda"), torch.zeros(out, device="cuda")
    thr = torch.zeros(3 * len(rows), dtype=torch.int32, device="cuda")
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
    for kernel, by_records in (("k_split", True), ("k_count", False)):
        iwp.timing_enable(kernel)
        iwp.compress_segmented(plan, wd, [None], [rd], None, 1e-8, idx, val, thr, ws)
        assert iwp.timing_collect()[1] == (1 if by_records == (keep < 0.125) else 0)
    torch.cuda.synchronize()
    for o, n, k, at in rows:
        if k:
            ref_idx, ref_val, _ = oracle.compress_layer(w[o:o + n], np.zeros(n, np.float32), r[o:o + n].copy(), k, 1e-8)
            assert np.array_equal(idx[at:at + k].cpu().numpy().view(np.uint32), ref_idx + np.uint32(o))
            assert np.array_equal(bits(val[at:at + k].cpu().numpy()), bits(ref_val))
