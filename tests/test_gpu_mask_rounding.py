"""Threshold masks where the rounding of the score decides: scores at a threshold and a few units in the last place to either side of it,
infinite and NaN scores, weights of zero with and without eps, and thresholds for which the short form is no proof (zero,
negative, subnormal, just above 2^-100, infinite, NaN)."""
import numpy as np
import pytest

import oracle
from paper_1901_01544_amd import workloads as wl
from harness import ThresholdSet, bits

pytestmark = pytest.mark.gpu
W = 4


def _near(rng, w, t, eps):
    """Residuals whose scores lie within a few units of t, a tenth of them; the others anywhere below twice t."""
    d = (np.abs(w) + np.float32(eps)).astype(np.float32)
    r = (d * np.float32(t)).astype(np.float32)
    r = (r.view(np.int32) + rng.integers(-4, 5, r.size).astype(np.int32)).view(np.float32)
    far = rng.random(r.size) < 0.9
    r[far] = (rng.uniform(0.0, 2.0, int(far.sum())) * d[far] * np.float32(t)).astype(np.float32)
    return np.where(rng.random(r.size) < 0.5, r, -r).astype(np.float32)


@pytest.mark.parametrize("eps", [0.0, 1e-8])
@pytest.mark.parametrize("n_lead", [1, 2, 3, 4])
@pytest.mark.parametrize("case", ["near", "far", "odd thresholds"])
def test_mask(gpu_lib, case, n_lead, eps):
    rng = np.random.default_rng(n_lead)
    thr = {"near": [0.7, 1.0, 3.0e-5, 1234.5], "far": [0.7, 1e-30, 1e30, 3e38],
           "odd thresholds": [0.0, -1.0, 1e-42, 7.9e-31, np.inf, np.nan, -0.0]}[case]
    sizes = [4096 + 7, 3, 1023, 9000][:len(thr)] + [2050] * (len(thr) - 4)
    ps = wl.custom_set([(n, 0) for n in sizes], W=W, seed=n_lead, align=1, start=1)
    w = wl.gen_weights(ps)
    r_ref = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    for L, t in zip(ps.layers, thr):
        at = slice(L.offset, L.offset + L.n)
        w[at][rng.random(L.n) < 0.01] = 0.0
        for p in range(W):
            r_ref[p][at] = _near(rng, w[at], abs(t) if np.isfinite(t) else 1.0, eps)
            if case == "far":
                r_ref[p][at][rng.random(L.n) < 0.01] = rng.choice(np.array([np.inf, -np.inf, 0.0, 1e-45, 3e38], np.float32))
    sets = [np.zeros(ps.flat, np.float32) for _ in range(W)]
    ts = ThresholdSet(gpu_lib, ps, w, sets, r_ref, n_lead, ps.flat)
    ts.eps = eps
    leaders = np.array([[(j + q) % W for q in range(n_lead)] for j in range(len(sizes))], np.uint32)
    thr = np.array(thr, np.float32)
    ts.step(list(range(W)), leaders, thr, -0.01)
    mask, cnt, idx, sm = oracle.step_threshold(w, sets, r_ref, ps.rows(), leaders, thr, eps, float(np.float32(-0.01)), ps.flat)
    got, total = ts.download(), int(cnt.sum())
    assert np.array_equal(got["idx"][:total], idx)
    same = (bits(got["sum"][:total]) == bits(sm)) | (np.isnan(got["sum"][:total]) & np.isnan(sm))
    assert same.all()
    for p in range(W):
        assert np.array_equal(bits(got["r"][p]), bits(r_ref[p]))
