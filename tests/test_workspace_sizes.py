"""Bytes of the workspace: what fits a layer fits shorter and sparser ones, and layers too long for records hold room for no more of them
than the longest layer that has them."""
import pytest

TILE, STILE = 4096, 8 * 4096
RECORD_MAX_STILES = 4096


def test_fits_shorter_and_sparser_layers():
    from paper_1901_01544_amd import iwp
    around = [m * STILE + d for m in (1, 17, 255, 257, 4095, 4096, 4097, 5000, 30000) for d in (-1, 0, 1)]
    for keep in (1e-6, 0.001, 1 / 64, 0.124, 0.126, 1.0):
        need = [iwp.workspace_bytes(n, max(1, int(n * keep))) for n in around]
        assert all(a <= b for a, b in zip(need, need[1:])), keep
    for n in (70_000, 1_000_000, 4096 * STILE, 4097 * STILE):
        need = [iwp.workspace_bytes(n, max(1, n * i // 1000)) for i in range(1001)]
        assert all(a <= b for a, b in zip(need, need[1:])), n


@pytest.mark.parametrize("share", [1000, 64, 4])
def test_no_records_beyond_the_longest_layer_that_has_them(share):
    from paper_1901_01544_amd import iwp
    n0, more = RECORD_MAX_STILES * STILE, 5000
    cap = min(TILE, 64 + 3 * -(-TILE // share))
    stile = 8 * (12 * cap + 16) + 8                             # slots, tiles' words and the super-tile's own
    n = n0 + more * STILE
    grown = iwp.workspace_bytes(n, n // share) - iwp.workspace_bytes(n0, n0 // share)
    assert grown <= more * stile + 16 * 256                     # each array is whole 256-byte blocks
