"""Which kernels a match runs, read from the library's kernel timing records:
work that is thrown away shows there and not in the pairs (which are compared
with the oracle all the same)."""
import numpy as np
import pytest

import oracle
from paper_1309_3458_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def recorded(fn):
    """fn's result and the kernels that it recorded: {name: launches}."""
    import paper_1309_3458_amd as P
    P.prof_enable(True)
    P.prof_read()
    try:
        res = fn()
        rec = {k: v[1] for k, v in P.prof_read().items()}
    finally:
        P.prof_enable(False)
    return res, rec


def match(inst):
    import paper_1309_3458_amd as P
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    t = P.build(dev(inst.s_lo), dev(inst.s_hi))
    keys, rec = recorded(lambda: P.match(t, dev(inst.u_lo), dev(inst.u_hi)))
    assert np.array_equal(keys.cpu().numpy().view(np.uint64), want)
    t.free()
    return len(want), rec


@pytest.mark.parametrize("m", [700, 9001])
def test_one_count_where_the_dense_form_is_not_allowed(m):
    """A dense set of more than 2^20 subscriptions: its first traversal counts
    (it used to list candidates that nothing read, and count in a second one)."""
    K, rec = match(W.uniform_instance(32, (1 << 20) + 77, m, 2, 9000.0))
    assert K > 100 * m
    assert rec["traverse_tile_count_stash"] == 1 and "traverse_tile_count" not in rec


@pytest.mark.parametrize("which", [0, 1])
def test_refused_move_matches_nothing(which):
    """A move with a repeated id leaves gaps in the gathered extents; what the
    scratch held there (the wide extents of the move before) must not be matched."""
    import paper_1309_3458_amd as P
    n, c = 60000, 64
    inst = W.uniform_instance(33, n, n, 2, 300.0)
    dyn = P.Dynamic(dev(inst.s_lo), dev(inst.s_hi), dev(inst.u_lo), dev(inst.u_hi))
    lo = dev(np.zeros((2, c), np.float32))
    hi = dev(np.full((2, c), 2e6, np.float32))
    ids = dev(np.arange(c, dtype=np.int32))
    for _ in range(3):  # the last one finds its scratch where the one before had it
        K = dyn.move(which, ids, lo, hi)
    assert K >= c * (n - c)
    before = dyn.pairs()

    def refused():
        with pytest.raises(P.DDMError):
            dyn.move(which, dev(np.full(c, 5, np.int32)), lo, hi)

    _, rec = recorded(refused)
    assert "listsort" not in rec and "traverse_tile_fill_units" not in rec
    assert bool((dyn.pairs() == before).all())
    dyn.free()
