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


def diagonal(seed, n, m, d, side):
    """Extents along the diagonal: the sample takes the dimensions as
    independent and expects few hits."""
    rng = np.random.default_rng(seed)

    def draw(count):
        c = rng.uniform(0, 1e6, count)
        lo = np.stack([(c + rng.uniform(0, 100, count)) for _ in range(d)]).astype(np.float32)
        return lo, (lo + np.float32(side)).astype(np.float32)

    u = draw(m)
    s = draw(n)
    return W.Instance(s[0], s[1], u[0], u[1])


FILLS = ("traverse_tile_fill", "traverse_tile_fill_balanced")


@pytest.mark.parametrize("d", [2, 3])
def test_overflowing_stash_takes_the_dense_form(d):
    K, rec = match(diagonal(34, 150000, 20000, d, 1500.0))
    assert K > 100 * 20000
    assert rec["traverse_tile_count_stash"] == 1 and rec["dense_expand"] == 1
    assert not any(k in rec for k in FILLS)


@pytest.mark.parametrize("m, side", [(8000, 600.0), (20000, 150.0)])
def test_overflowing_stash_fills_where_the_dense_form_is_not_allowed(m, side):
    """More than 2^20 subscriptions, more hits than the stash has room for."""
    K, rec = match(diagonal(35, (1 << 20) + 5, m, 2, side))
    assert K > 100 * m
    assert rec["traverse_tile_count_stash"] == 1 and "stash_scatter" not in rec
    assert any(k in rec for k in FILLS) and "dense_expand" not in rec
    assert "traverse_tile1_fill" not in rec


@pytest.mark.parametrize("m", [300, 8192, 20000])
def test_name_of_a_plain_fill(m):
    """One update to a tile is not the refill of overflowed slots."""
    K, rec = match(W.uniform_instance(36, 50000, m, 1, 60.0))
    assert K > 0 and any(k in rec for k in FILLS) and "traverse_tile1_fill" not in rec


def test_name_of_a_refill():
    """A predictor that gives every update two slots: the others are refilled."""
    import paper_1309_3458_amd as P
    from oracle import mlp_ref
    p = P.Predictor(0)
    w = np.zeros(mlp_ref.N_PARAMS, np.float32)
    w[-1] = np.log1p(2.0)
    p.set_params(w, 0.0)
    inst = W.uniform_instance(37, 20000, 9001, 2, 9000.0)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    t = P.build(dev(inst.s_lo), dev(inst.s_hi))
    keys, rec = recorded(lambda: P.match_learned(t, dev(inst.u_lo), dev(inst.u_hi), p))
    assert np.array_equal(keys.cpu().numpy().view(np.uint64), want)
    assert rec["traverse_tile1_fill"] == 1 and rec["traverse_tile_fill_balanced"] == 1
    assert "dense_expand" not in rec
    t.free()
    p.free()


@pytest.mark.parametrize("n, m, hits, dense", [
    (20000, 8000, 1200, False),       # one update to a tile
    (100000, 700000, 14, False),      # many updates, few hits each
    (100000, 60000, 167, False),      # tiles of 8: from 2^24 pairs
    (100000, 60000, 400, True),
    (20000, 154000, 62, True),        # tiles of 32: from 2^23 pairs
    (3000, 4000, 2200, True),         # more than half of all pairs
])
def test_one_dimension_takes_the_dense_form_where_it_pays(n, m, hits, dense):
    f = hits / n
    side = 1e6 * (1.0 - (1.0 - f) ** 0.5)
    K, rec = match(W.uniform_instance(38, n, m, 1, side))
    assert K > (1 << 23)
    assert ("dense_expand" in rec) == dense and any(k in rec for k in FILLS) != dense


@pytest.mark.parametrize("d", [1, 2])
def test_a_result_beyond_the_capacity_is_only_counted(d):
    """The number of pairs is known before the dense form is begun."""
    import paper_1309_3458_amd as P
    import torch
    inst = diagonal(39, 150000, 154000, d, 400.0)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    t = P.build(dev(inst.s_lo), dev(inst.s_hi))
    out = torch.full((1000,), -1, dtype=torch.int64, device="cuda")

    def refused():
        with pytest.raises(P.DDMError) as e:
            P.match_into(t, dev(inst.u_lo), dev(inst.u_hi), out)
        assert str(len(want)) in str(e.value)

    _, rec = recorded(refused)
    assert "listsort" not in rec and bool((out == -1).all())
    big = torch.empty(len(want), dtype=torch.int64, device="cuda")
    K, rec = recorded(lambda: P.match_into(t, dev(inst.u_lo), dev(inst.u_hi), big))
    assert rec["dense_expand"] == 1
    assert np.array_equal(big[:K].cpu().numpy().view(np.uint64), want)
    t.free()


@pytest.mark.parametrize("d, long, short, n, m, hits", [
    (2, 2e4, 200.0, 18000, 250000, 3.8), (2, 2e4, 200.0, 100000, 8000, 21.0),
    (3, 6e4, 3e3, 250000, 250000, 3.5), (4, 3e5, 2e4, 40000, 250000, 3.0)])
def test_hits_of_mixed_lengths_are_kept(d, long, short, n, m, hits):
    """Half of the boxes long in one dimension, half in another: three to four times
    as many hits were all subscriptions as long as the longest."""
    rng = np.random.default_rng(37)

    def boxes(count):
        side = np.full((d, count), short)
        side[rng.integers(0, 2, count), np.arange(count)] = long
        lo = rng.uniform(0, 1e6, (d, count)).astype(np.float32)
        return lo, (lo + side).astype(np.float32)

    import paper_1309_3458_amd as P
    inst = W.Instance(*boxes(n), *boxes(m))
    t = P.build(dev(inst.s_lo), dev(inst.s_hi))
    keys, rec = recorded(lambda: P.match(t, dev(inst.u_lo), dev(inst.u_hi)))
    t.free()
    keys = keys.cpu().numpy().view(np.uint64)
    # (the oracle takes a minute for all of them)
    some = 1000
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo[:, :some], inst.u_hi[:, :some], threads=8)
    assert np.array_equal(keys[:len(want)], want) and keys[len(want)] >> np.uint64(32) >= some
    assert 0.8 * hits < len(keys) / m < 1.2 * hits
    assert rec["stash_scatter"] == 1 and "dense_expand" not in rec


def test_hits_of_dependent_dimensions_are_kept():
    """Boxes on a plane in three dimensions: the sample expects a hundredth of their
    24 hits each, and the stash has room for them."""
    rng = np.random.default_rng(38)

    def boxes(count):
        p, q = rng.uniform(0, 1e6, (2, count))
        lo = np.stack([p, p + rng.uniform(0, 100, count), q]).astype(np.float32)
        return lo, (lo + np.float32([[1000], [1000], [11000]])).astype(np.float32)

    import paper_1309_3458_amd as P
    m = 200000
    inst = W.Instance(*boxes(600000), *boxes(m))
    t = P.build(dev(inst.s_lo), dev(inst.s_hi))
    keys, rec = recorded(lambda: P.match(t, dev(inst.u_lo), dev(inst.u_hi)))
    t.free()
    keys = keys.cpu().numpy().view(np.uint64)
    some = 1000
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo[:, :some], inst.u_hi[:, :some], threads=8)
    assert np.array_equal(keys[:len(want)], want) and keys[len(want)] >> np.uint64(32) >= some
    assert 22 < len(keys) / m < 28
    assert rec["stash_scatter"] == 1 and "dense_expand" not in rec
