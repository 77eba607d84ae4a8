"""Layers that one workgroup takes whole: scores that part only in one digit of their keys, at the digits' borders of both forms
(11 + 10 + 10 bits up to 4096 elements, 12 + 10 + 9 beyond), and lengths whose last quad is cut, the largest scores in it."""
import numpy as np
import pytest

from test_gpu_selection_paths import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 258, 1021, 1023, 1026, 4095, 4099, 12285, 20002, 28673])
def test_digits_and_cut_quads(gpu_lib, n):
    import torch
    rng = np.random.default_rng(n)
    one, z = np.ones(n, np.float32), np.zeros(n, np.float32)
    for low, bits in ((0, 9), (0, 10), (9, 10), (10, 10), (19, 9), (20, 8)):    # keys from 1.0 up that differ in these bits only
        key = np.uint32(0x3F800000) + (rng.integers(0, 1 << bits, n) << low).astype(np.uint32)
        r = np.minimum(key, np.uint32(0x7F000000)).view(np.float32)
        for k in sorted({1, max(1, n // 64), n // 2, n - 1, n}):
            _check(gpu_lib, torch, one, z, r, k, "n=%d bits %d to %d k=%d" % (n, low, low + bits, k))
    r = rng.uniform(0.1, 0.9, n).astype(np.float32)
    r[-3:] = (5.0, -7.0, 6.0)
    for k in (1, 2, 3, 4):
        _check(gpu_lib, torch, one, z, r, k, "n=%d last quad k=%d" % (n, k))
