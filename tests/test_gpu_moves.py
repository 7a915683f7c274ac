"""Moves of resident extents by merging: move counts around the workgroup sizes
and where the general path takes over, moves that put everything into one tile,
ties of the lower bounds, results that start or end empty, rows beyond the one
workgroup's sort, and refused moves that must change nothing.  Pairs are whole
numbers: equal or wrong.
"""
import numpy as np
import pytest

import oracle
from paper_1309_3458_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Pair:
    """A dynamic matcher and the sets it should hold."""

    def __init__(self, inst):
        import paper_1309_3458_amd as P
        self.P = P
        self.sets = [[inst.s_lo.copy(), inst.s_hi.copy()], [inst.u_lo.copy(), inst.u_hi.copy()]]
        self.dyn = P.Dynamic(dev(inst.s_lo), dev(inst.s_hi), dev(inst.u_lo), dev(inst.u_hi))

    def move(self, which, ids, lo, hi):
        which_c = self.P.Dynamic.SUBSCRIPTIONS if which == 0 else self.P.Dynamic.UPDATES
        k = self.dyn.move(which_c, dev(ids.astype(np.int32)), dev(lo), dev(hi))
        self.sets[which][0][:, ids] = lo
        self.sets[which][1][:, ids] = hi
        self.check(k)

    def check(self, k=None):
        (s_lo, s_hi), (u_lo, u_hi) = self.sets
        want = oracle.itm(s_lo, s_hi, u_lo, u_hi, threads=8)
        got = self.dyn.pairs().cpu().numpy().view(np.uint64)
        assert np.array_equal(got, want)
        if k is not None:
            assert k == len(want)


def extents(rng, d, c, side, quantum=0.0):
    lo = rng.uniform(0.0, 1e6, (d, c)).astype(np.float32)
    if quantum:
        lo = (np.floor(lo / quantum) * quantum).astype(np.float32)
    return lo, (lo + np.float32(side)).astype(np.float32)


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("count", [1, 2, 1023, 1025, 4097, 8192, 8193])
def test_counts(d, count):
    side = {1: 60.0, 2: 8e3, 3: 4e4, 4: 9e4}[d]
    p = Pair(W.uniform_instance(7000 + count, 9001, 8500, d, side))
    rng = np.random.default_rng(count)
    for which, n in ((0, 9001), (1, 8500), (0, 9001)):
        ids = rng.permutation(n)[:count]
        p.move(which, ids, *extents(rng, d, count, side))


@pytest.mark.parametrize("d", [2, 3])
def test_ties(d):
    """Many equal lower bounds, moved onto each other and onto themselves."""
    inst = W.uniform_instance(11, 5000, 4000, d, 2e4)
    for a in (inst.s_lo, inst.u_lo):
        a[:] = np.floor(a / 5e4) * np.float32(5e4)
    inst.s_hi[:] = inst.s_lo + np.float32(2e4)
    inst.u_hi[:] = inst.u_lo + np.float32(2e4)
    p = Pair(inst)
    rng = np.random.default_rng(5)
    for which, n in ((0, 5000), (1, 4000)):
        ids = rng.permutation(n)[:700]
        p.move(which, ids, *extents(rng, d, 700, 2e4, 5e4))
        # the same extents again: nothing may change
        p.move(which, ids, p.sets[which][0][:, ids].copy(), p.sets[which][1][:, ids].copy())


def test_all_into_one_tile_and_back():
    d, n = 2, 6000
    p = Pair(W.uniform_instance(13, n, n, d, 5e3))
    rng = np.random.default_rng(6)
    ids = rng.permutation(n)[:3000]
    old = [a[:, ids].copy() for a in p.sets[0]]
    lo = rng.uniform(4.99e5, 5.0e5, (d, 3000)).astype(np.float32)
    p.move(0, ids, lo, lo + np.float32(200.0))
    p.move(0, ids, *old)
    ids = np.arange(n)  # every extent
    p.move(1, ids, *extents(rng, d, n, 5e3))


def test_empty_results_and_many_rows():
    d = 2
    p = Pair(W.uniform_instance(17, 3000, 3000, d, 5e3))
    ids = np.arange(3000)
    far = np.full((d, 3000), 5e6, np.float32)
    p.move(0, ids, far, far + np.float32(1.0))
    assert p.dyn.pairs().numel() == 0
    rng = np.random.default_rng(8)
    p.move(0, ids[:5], *extents(rng, d, 5, 1e5))
    for side in (2e4, 5e4):  # rows within and beyond one workgroup's sort
        p.move(0, ids, *extents(rng, d, 3000, side))


@pytest.mark.parametrize("d", [1, 2])
def test_refused_moves_change_nothing(d):
    p = Pair(W.uniform_instance(19, 4000, 4000, d, 3e3))
    rng = np.random.default_rng(9)
    lo, hi = extents(rng, d, 300, 3e3)
    good = rng.permutation(4000)[:300]
    for bad in ("range", "repeat", "nan", "order"):
        ids, a, b = good.copy(), lo.copy(), hi.copy()
        if bad == "range":
            ids[7] = 4000
        elif bad == "repeat":
            ids[7] = ids[200]
        elif bad == "nan":
            a[d - 1, 11] = np.nan
        else:
            b[0, 11] = a[0, 11] - np.float32(1.0)
        for which in (0, 1):
            with pytest.raises(p.P.DDMError):
                p.dyn.move(which, dev(ids.astype(np.int32)), dev(a), dev(b))
            p.check()
    p.move(1, good, lo, hi)
