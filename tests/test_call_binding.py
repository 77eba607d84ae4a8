"""The module that converts the hot calls' arguments: what it takes, what it turns away, and that numbers and tables arrive.
No GPU: calls that end in the library's argument checks, or with nothing to do."""
import ctypes

import pytest
import torch

from paper_1901_01544_amd import iwp


class NoStream:
    cuda_stream = 0


S = NoStream()


def test_numbers_and_codes():
    iwp.load()
    assert iwp.compress_layer(None, 16, None, 0, 1e-8, None, None, None, S, n=0) is None          # nothing to do
    for n, k, eps, code in ((4, 5, 1e-8, iwp.IWP_EINVAL), (4, 2, -1.0, iwp.IWP_EINVAL), (2 ** 32 - 1, 1, 0.0, iwp.IWP_ERANGE)):
        with pytest.raises(iwp.IwpError) as e:
            iwp.compress_layer(16, 16, 16, k, eps, 16, 16, None, S, n=n)
        assert e.value.code == code
    with pytest.raises(iwp.IwpError) as e:                       # 256-byte alignment of the workspace, given as an address
        iwp._check(iwp._hot().compress_layer(16, 16, 16, 8, 1, 0.0, 16, 16, 16, 1 << 30, None), "x")
    assert e.value.code == iwp.IWP_EALIGN


def test_tables():
    iwp.load()
    iwp.gather_sum_at_indices([16, 32], None, 0, None, S)         # no pairs
    iwp.apply_sparse_update(None, None, None, 0, 1.0, (), S)
    for table, code in (([], iwp.IWP_EINVAL), ([16] * 33, iwp.IWP_EINVAL), ([16, None], iwp.IWP_EINVAL),
                        ((16, 18), iwp.IWP_EALIGN), ([16] * 100, iwp.IWP_EINVAL)):
        with pytest.raises(iwp.IwpError) as e:
            iwp.gather_sum_at_indices(table, 16, 4, 16, S)
        assert e.value.code == code


def test_turned_away():
    iwp.load()
    host = torch.zeros(8)
    with pytest.raises(AssertionError):
        iwp.compress_layer(host, host, host, 1, 0.0, host, host, None, S)
    with pytest.raises(AssertionError):
        iwp.gather_sum_at_indices([16, host], 16, 4, 16, S)
    with pytest.raises(AttributeError):
        iwp.gather_sum_at_indices(["x"], 16, 4, 16, S)
    with pytest.raises(TypeError):
        iwp.gather_sum_at_indices([16], 16, 4.0, 16, S)
    with pytest.raises(TypeError):
        iwp.compress_layer(16, 16, 16, 1, "eps", 16, 16, None, S, n=4)
    with pytest.raises(TypeError):
        iwp._hot().gather_sum_at_indices(1, 2)


def test_bound_to_the_library():
    L = iwp.load()
    at = {name: ctypes.cast(getattr(L, name), ctypes.c_void_p).value for name in iwp._hot().names()}
    assert len(set(at.values())) == len(at) == 13
    with pytest.raises(KeyError):
        iwp._hot().bind({})
    iwp._hot().bind(at)
