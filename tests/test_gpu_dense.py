"""Dense sets: the tiles' candidate lists sorted by id, the hits tested in id
order and expanded (csrc/dense.h), against the oracle where the form can go
wrong: list lengths around a unit of 1024 candidates and a batch of 64, update
counts around the tile sizes, sets whose density the sample misjudges, and
lists the predictor sizes too small.  Pairs are whole numbers: equal or wrong.
"""
import numpy as np
import pytest

import oracle
from paper_1309_3458_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _match(inst, learned=None, info=None):
    import paper_1309_3458_amd as P
    t = P.build(dev(inst.s_lo), dev(inst.s_hi))
    P.prof_enable(True)
    P.prof_read()
    try:
        if learned is None:
            keys = P.match(t, dev(inst.u_lo), dev(inst.u_hi))
        else:
            keys = P.match_learned(t, dev(inst.u_lo), dev(inst.u_hi), learned, info=info)
        got = keys.cpu().numpy().view(np.uint64)
        rec = P.prof_read()
    finally:
        P.prof_enable(False)
    t.free()
    return got, rec


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [63, 64, 65, 1023, 1024, 1025, 2049, 5000])
def test_list_lengths(d, n):
    """Long extents: every list holds about every id, and there are updates
    enough for the dense form."""
    side = 0.9e6 if n < 1000 else 0.5e6
    hits = n * (0.98 if n < 1000 else 0.74) ** d
    m = 131 + int(9.5e6 / hits if d == 1 else 1.4 * (3000.0 * d / hits) ** 2)
    inst = W.uniform_instance(1000 + n, n, m, d, side)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    got, rec = _match(inst)
    assert "traverse_tile_fill_units" in rec
    assert np.array_equal(got, want)


@pytest.mark.parametrize("m", [1, 4, 5, 255, 32768, 32769, 65537])
def test_update_counts(m):
    """Tiles of 4, 8 and 16 updates, full and partial."""
    inst = W.uniform_instance(2000 + m, 3000 if m > 255 else 20000, m, 2,
                              130000.0 if m > 255 else 0.5e6)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    got, rec = _match(inst)
    assert "traverse_tile_fill_units" in rec
    assert np.array_equal(got, want)


def _diagonal(seed, n, m, d):
    """Extents along the diagonal: the dimensions are anything but independent."""
    rng = np.random.default_rng(seed)

    def draw(count):
        c = rng.uniform(0, 1e6, count)
        lo = np.stack([(c + rng.uniform(0, 100, count)) for _ in range(d)]).astype(np.float32)
        return lo, (lo + np.float32(1500.0)).astype(np.float32)

    u = draw(m)
    s = draw(n)
    return W.Instance(s[0], s[1], u[0], u[1])


@pytest.mark.parametrize("d", [2, 3])
def test_correlated_set_overflows_the_stash(d):
    inst = _diagonal(7 + d, 150000, 20000, d)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    assert len(want) > 100 * inst.m
    got, _ = _match(inst)
    assert np.array_equal(got, want)


def test_ids_beyond_the_bitmap_window():
    """More than 2^20 subscriptions: counted, filled and sorted instead."""
    inst = W.uniform_instance(31, (1 << 20) + 77, 700, 2, 9000.0)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    got, rec = _match(inst)
    assert len(want) > 100 * inst.m and "traverse_tile_fill_units" not in rec
    assert np.array_equal(got, want)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("hits", [60.0, 4000.0])
def test_learned_lists(d, hits):
    """A predictor that says `hits` for every extent: too little for the tiles'
    lists (the lists are made again from the counts) and more than enough."""
    import paper_1309_3458_amd as P
    from oracle import mlp_ref
    p = P.Predictor(0)
    w = np.zeros(mlp_ref.N_PARAMS, np.float32)
    w[-1] = np.log1p(hits)
    p.set_params(w, 0.0)
    inst = W.uniform_instance(50 + d, 4000, 9001, d, 150000.0 if d == 2 else 300000.0)
    want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
    info = {}
    got, rec = _match(inst, p, info)
    assert "traverse_tile_fill_balanced" in rec and "candidate_lists" in rec
    assert np.array_equal(got, want)
    counts = oracle.counts_per_update(want, inst.m)
    assert info["slots"] == info["budget"]
    cap = info["slots"] // inst.m
    assert info["overflowed"] == int((counts > cap).sum())
    p.free()
