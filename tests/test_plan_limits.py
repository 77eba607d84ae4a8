"""The largest layer tables that a plan takes: as many histograms as 32 bits address.  No GPU: a table that passes the checks ends in
a HIP error here, or in a plan."""
import ctypes

import numpy as np
import pytest

from paper_1901_01544_amd import iwp

ROW = np.dtype([("offset", "<i8"), ("n", "<u4"), ("k", "<u4"), ("out_offset", "<u4"), ("pad", "<u4")])
ONE_COPY = 4096 + 1024 + 512                                   # words of a layer's histograms


@pytest.mark.parametrize("spare,tiles,code", [(0, 1, None), (0, 129, None), (0, 512, None), (0, 513, iwp.IWP_ERANGE),
                                              (-1, 1, iwp.IWP_ERANGE)])
def test_histograms_of_32_bits(spare, tiles, code):
    """One-element layers and a last one of `tiles` tiles.  Up to 512 tiles it can do with one copy of its first-digit histogram,
    though it has more where there is room for them."""
    L = iwp.load()
    layers = 0xFFFFFFFF // ONE_COPY - spare
    rows = np.zeros(layers, ROW)
    rows["n"] = rows["k"] = 1
    rows["offset"] = rows["out_offset"] = np.arange(layers)
    rows["n"][-1] = tiles * 4096
    table = (iwp.Layer * layers)()
    ctypes.memmove(table, rows.ctypes.data, rows.nbytes)
    plan = ctypes.c_void_p()
    got = L.iwp_plan_create(table, layers, ctypes.byref(plan))
    assert got == code if code is not None else got in (iwp.IWP_OK, iwp.IWP_EHIP)
    if plan.value:
        L.iwp_plan_destroy(plan)
