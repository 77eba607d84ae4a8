"""The layer-wise rule where the masks' launch merges the tiles' statistics itself (layers of up to 64 tiles, 1024 tiles over all chosen
nodes) and where a launch of its own does: both sides of both lines, layers without elements, nodes listed twice."""
import numpy as np
import pytest

from paper_1901_01544_amd import workloads as wl
from test_gpu_layerwise import _run

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]
TILE = 4096


@pytest.mark.parametrize("sizes,n_lead", [([64 * TILE, 0, 5, 9000], 2), ([64 * TILE + 1, 0, 5, 9000], 2),
                                          ([64 * TILE - 1, 0, 1, 0, 4097], 1), ([3 * TILE] * 85 + [1], 4),
                                          ([3 * TILE] * 85 + [1, 1], 4), ([7, 0, 0, 1023], 8)])
def test_merge(gpu_lib, sizes, n_lead):
    W = 8
    ps = wl.custom_set([(n, 0) for n in sizes], W=W, seed=len(sizes), align=1, start=1)
    _run(gpu_lib, ps, W, n_lead, 2, seed=n_lead)
