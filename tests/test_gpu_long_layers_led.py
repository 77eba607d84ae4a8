"""Layers on both sides of 4096 super-tiles, led by the second of two workers, behind them a short layer that keeps as little: counts and
pairs by a wavefront per super-tile where at most one of 170 is kept and the layer is long enough, otherwise by workgroups.  The leader's
residual is selected from and cleared, the sums run over both workers in order."""
import pytest

from test_gpu_long_layers import STILE, _expected, _residuals

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


@pytest.mark.parametrize("streaming", [False, True])
@pytest.mark.parametrize("kind,share,stiles,by_wavefronts", [("plain", 1000, 4097, 1), ("blocks", 300, 4097, 1), ("ties", 400, 4097, 1),
                                                             ("blocks", 300, 4096, 0), ("plain", 30, 4097, 0)])
def test_leader_is_the_second_worker(gpu_lib, kind, share, stiles, by_wavefronts, streaming):
    import torch
    iwp = gpu_lib
    n, n2 = stiles * STILE - 4096 * 3 - 5, 50001
    k, k2 = n // share, 200
    rows = [(1, n, k, 0), (1 + n, n2, k2, k)]
    plan = iwp.Plan(rows)
    edge = torch.full((1,), 9.0, device="cuda")
    r = [torch.cat([edge, _residuals(torch, n, kind if p else "plain"), _residuals(torch, n2, "plain")]) for p in range(2)]
    g = [None, None]
    if streaming:
        gen = torch.Generator(device="cuda").manual_seed(share)
        g = [(torch.rand(r[0].numel(), device="cuda", generator=gen) < 0.5).float().div_(8.0) for _ in range(2)]
        for x in g:
            x[0] = 0.0                                          # belongs to no layer
    w = torch.ones_like(r[0])
    lead = [1, 0]
    leader = torch.tensor(lead, dtype=torch.int32, device="cuda")
    r_ref = [x + y if streaming else x.clone() for x, y in zip(r, g)]
    idx_ref = torch.cat([_expected(torch, r_ref[p][o:o + m], kk)[0] + o for p, (o, m, kk, _) in zip(lead, rows)])
    val_ref = torch.cat([r_ref[p][idx_ref[out:out + kk]] for p, (_, _, kk, out) in zip(lead, rows)])
    idx, val = torch.full((k + k2,), -1, dtype=torch.int32, device="cuda"), torch.zeros(k + k2, device="cuda")
    total, thr = torch.zeros(k + k2, device="cuda"), torch.zeros(6, dtype=torch.int32, device="cuda")
    ws = torch.empty(plan.step_workspace_bytes(2), dtype=torch.uint8, device="cuda")

    mine = [x.clone() for x in r]
    iwp.timing_enable("k_write_stiles")
    iwp.compress_segmented(plan, w, g, mine, leader, 0.0, idx, val, thr, ws)
    torch.cuda.synchronize()
    assert iwp.timing_collect()[1] == by_wavefronts
    assert torch.equal(idx.long(), idx_ref) and torch.equal(val, val_ref)
    assert all(torch.equal(x, y) for x, y in zip(mine, r_ref))
    del mine
    idx.fill_(-1)
    val.zero_()
    iwp.timing_enable("k_count_stiles")
    iwp.step_segmented(plan, w, g, r, leader, 0.0, -0.5, idx, val, total, thr, ws)
    torch.cuda.synchronize()
    assert iwp.timing_collect()[1] == by_wavefronts
    assert torch.equal(idx.long(), idx_ref) and torch.equal(val, val_ref)
    assert torch.equal(total, r_ref[0][idx_ref] + r_ref[1][idx_ref])
    w_ref = torch.ones_like(w)
    w_ref[idx_ref] += -0.5 * total
    for x in r_ref:
        x[idx_ref] = 0.0
    assert torch.equal(w, w_ref) and all(torch.equal(x, y) for x, y in zip(r, r_ref))
