"""Layers on both sides of 4096 super-tiles, beyond which the super-tiles' counts are scanned by a launch of their own: slots of few and of
many entries, tiles of equal scores at, above and below the threshold, tiles that overflow their slots, behind the long one a short layer
that keeps too many for the kernels that take a super-tile by a wavefront (test_gpu_long_layers_led.py has those).  Weights of one and no eps: the
score is |r| itself."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]
TILE, STILE = 4096, 8 * 4096


def _residuals(torch, n, kind):
    gen = torch.Generator(device="cuda").manual_seed(n + len(kind))
    r = torch.empty(n, device="cuda").uniform_(-1.0, 1.0, generator=gen)
    if kind == "blocks":
        tile = torch.arange(n, device="cuda") // TILE
        r[tile % 97 == 3] = 0.0
        r[tile % 1001 == 5] = 2.0                              # tiles of equal scores above the threshold
        dense = tile % 2003 == 7
        r[dense] = torch.empty(int(dense.sum()), device="cuda").uniform_(0.995, 1.0, generator=gen)
    if kind == "ties":
        r = torch.where(r.abs() > 0.5, r.sign(), r)            # half of all tie with the threshold
    return r


def _expected(torch, r, k):
    score = r.abs()
    line = torch.kthvalue(score, score.numel() - k + 1).values
    keep = score > line
    keep[(score == line).nonzero().flatten()[:k - int(keep.sum())]] = True
    return keep.nonzero().flatten(), line


@pytest.mark.parametrize("stiles", [4096, 4097])
@pytest.mark.parametrize("kind,share", [("plain", 1000), ("plain", 30), ("blocks", 300), ("ties", 400)])
def test_step_and_pairs(gpu_lib, stiles, kind, share):
    import torch
    iwp = gpu_lib
    n, n2 = stiles * STILE - 4096 * 3 - 5, 50001
    k, k2 = n // share, 700
    rows = [(1, n, k, 0), (1 + n, n2, k2, k)]
    plan = iwp.Plan(rows)
    r = torch.cat([torch.full((1,), 9.0, device="cuda"), _residuals(torch, n, kind), _residuals(torch, n2, "plain")])
    w = torch.ones_like(r)
    want = [_expected(torch, r[o:o + m], kk) for o, m, kk, _ in rows]
    idx_ref = torch.cat([x[0] + o for x, (o, _, _, _) in zip(want, rows)])
    idx, val = torch.full((k + k2,), -1, dtype=torch.int32, device="cuda"), torch.zeros(k + k2, device="cuda")
    total, thr = torch.zeros(k + k2, device="cuda"), torch.zeros(6, dtype=torch.int32, device="cuda")
    ws = torch.empty(plan.step_workspace_bytes(1), dtype=torch.uint8, device="cuda")
    iwp.select_threshold_segmented(plan, w, r, 0.0, thr, ws)
    assert torch.equal(thr.view(torch.float32)[0::3], torch.stack([x[1] for x in want]))
    iwp.compact_pairs_segmented(plan, w, r, 0.0, thr, idx, val, ws)
    assert torch.equal(idx.long(), idx_ref) and torch.equal(val, r[idx_ref])
    idx.fill_(-1)
    val.zero_()
    r_ref, w_ref = r.clone(), w.clone()
    r_ref[idx_ref] = 0.0
    w_ref[idx_ref] += -0.5 * r[idx_ref]
    val_ref = r[idx_ref]
    iwp.step_segmented(plan, w, [None], [r], None, 0.0, -0.5, idx, val, total, thr, ws)
    torch.cuda.synchronize()
    assert torch.equal(idx.long(), idx_ref) and torch.equal(val, val_ref) and torch.equal(total, val_ref)
    assert torch.equal(r, r_ref) and torch.equal(w, w_ref)
