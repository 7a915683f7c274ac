"""Small sets take kernels of their own (keys and sort in one workgroup, the
update order in one workgroup, the offsets in one workgroup): the sizes at
which each begins and ends, equal lower bounds (the sort is stable), extents
that are not valid, and the largest scan's separate pass over the tile sums.
Pairs are whole numbers: equal or wrong.
"""
import numpy as np
import pytest

import oracle
from paper_1309_3458_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _match(s_lo, s_hi, u_lo, u_hi):
    import paper_1309_3458_amd as P
    t = P.build(dev(s_lo), dev(s_hi))
    try:
        return P.match(t, dev(u_lo), dev(u_hi)).cpu().numpy().view(np.uint64)
    finally:
        t.free()


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 2047, 2049, 5121, 6145, 8191, 8192, 8193])
def test_sort_sizes(d, n):
    inst = W.uniform_instance(3000 + n, n, 300, d, 0.3e6)
    # many equal lower bounds in every dimension
    s_lo = np.floor(inst.s_lo / 1e5).astype(np.float32) * np.float32(1e5)
    s_hi = np.maximum(inst.s_hi, s_lo)
    want = oracle.itm(s_lo, s_hi, inst.u_lo, inst.u_hi)
    assert np.array_equal(_match(s_lo, s_hi, inst.u_lo, inst.u_hi), want)


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("m", [1, 1023, 1025, 8191, 8192, 8193, 16384, 16385])
def test_order_sizes(d, m):
    inst = W.uniform_instance(4000 + m, 2000, m, d, 0.02e6)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi)
    assert np.array_equal(_match(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi), want)


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [100, 8192, 9000])
def test_invalid_extents(d, n):
    import paper_1309_3458_amd as P
    inst = W.uniform_instance(5000 + n, n, n, d, 0.02e6)
    for side in (0, 1):
        arrs = [inst.s_lo.copy(), inst.s_hi.copy(), inst.u_lo.copy(), inst.u_hi.copy()]
        arrs[2 * side][d - 1, n - 1] = np.nan
        with pytest.raises(P.DDMError):
            _match(*arrs)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi)
    assert np.array_equal(_match(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi), want)


def test_largest_scan():
    inst = W.uniform_instance(6000, 500, 4096 * 1024 + 77, 2, 1.0e4)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    assert np.array_equal(_match(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi), want)
