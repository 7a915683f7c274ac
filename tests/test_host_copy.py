"""Results leave the server's pool in slices by several threads: sizes around
the slices and the page rounding, every byte in its place and none beyond.
"""
import ctypes

import numpy as np
import pytest

from paper_1309_3458_amd._native import lib


@pytest.mark.parametrize("nbytes", [0, 1, 4095, (1 << 20) - 1, 1 << 20, (2 << 20) - 1, 2 << 20,
                                    (2 << 20) + 1, (3 << 20) + 4097, (4 << 20) + 8, 12345678])
def test_every_byte_once(nbytes):
    src = np.random.default_rng(nbytes).integers(0, 256, nbytes + 16).astype(np.uint8)
    dst = np.full(nbytes + 16, 0xA5, np.uint8)
    code = lib().ddm_host_copy(dst.ctypes.data_as(ctypes.c_void_p),
                               src.ctypes.data_as(ctypes.c_void_p), nbytes)
    assert code == 0
    assert np.array_equal(dst[:nbytes], src[:nbytes])
    assert (dst[nbytes:] == 0xA5).all()
