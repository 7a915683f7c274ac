"""The order that updates are matched in, on sets that a grid of equal cells does
not fit: extents long in one dimension or another, along a line or a plane, in
clusters.  Pairs are whole numbers (equal or wrong); the count traversal's time
is compared with that of a uniform set of the same size, since an order that does
not fit shows only there (by factors of 6 to 60)."""
import numpy as np
import pytest

import oracle
from paper_1309_3458_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def boxes(rng, d, count, side):
    lo = rng.uniform(0, 1e6, (d, count)).astype(np.float32)
    return lo, (lo + np.asarray(side, np.float32)).astype(np.float32)


def either_way(rng, d, count, long, short):
    """Half long in the first dimension, half in the second."""
    side = np.full((d, count), short)
    side[rng.integers(0, 2, count), np.arange(count)] = long
    return boxes(rng, d, count, side)


def line(rng, d, count, side):
    lo = rng.uniform(0, 1e6, (1, count)) + rng.uniform(0, 100, (d, count))
    return lo.astype(np.float32), (lo + side).astype(np.float32)


def plane(rng, d, count, side):
    p, q = rng.uniform(0, 1e6, (2, count))
    lo = np.stack([p, p, q, q])[:d] + rng.uniform(0, 1000, (d, count))
    return lo.astype(np.float32), (lo + side).astype(np.float32)


def clusters(rng, d, count, side, spread, centres):
    lo = centres[:, rng.integers(0, centres.shape[1], count)] + \
        spread * rng.standard_normal((d, count))
    return lo.astype(np.float32), (lo + side).astype(np.float32)


def instance(kind, seed, n, m, d):
    rng = np.random.default_rng(seed)
    if kind == "uniform":
        side = 1e6 * (0.01 / (n + m)) ** (1.0 / d)
        s, u = boxes(rng, d, n, side), boxes(rng, d, m, side)
    elif kind == "long updates":  # all in the first dimension
        side = np.full((d, 1), 20.0)
        s = boxes(rng, d, n, side)
        side[0] = 2e5
        u = boxes(rng, d, m, side)
    elif kind == "long either way":
        s, u = boxes(rng, d, n, 20.0), either_way(rng, d, m, 2e5, 20.0)
    elif kind == "all long either way":
        s, u = either_way(rng, d, n, 4e5, 1e3), either_way(rng, d, m, 4e5, 1e3)
    elif kind == "line":
        s, u = line(rng, d, n, 20.0), line(rng, d, m, 20.0)
    elif kind == "plane":
        s, u = plane(rng, d, n, 1000.0), plane(rng, d, m, 1000.0)
    else:
        c = rng.uniform(0, 1e6, (d, 16 if kind == "16 clusters" else 100))
        spread = 2e4 if kind == "16 clusters" else 3e3
        side = {2: 200.0, 3: 500.0, 4: 1000.0}[d]
        s, u = clusters(rng, d, n, side, spread, c), clusters(rng, d, m, side, spread, c)
    return W.Instance(s[0], s[1], u[0], u[1])


KINDS = ["long either way", "all long either way", "line", "plane", "16 clusters", "100 clusters"]


@pytest.mark.parametrize("d", [2, 3, 4])
@pytest.mark.parametrize("kind", KINDS)
def test_pairs(kind, d):
    """Also where classes, cells and tiles are few, and by every path that orders."""
    import paper_1309_3458_amd as P
    for n, m in ((3000, 8193), (30011, 20001)):
        inst = instance(kind, 100 + d, n, m, d)
        want = oracle.itm(inst.s_lo, inst.s_hi, inst.u_lo, inst.u_hi, threads=8)
        t = P.build(dev(inst.s_lo), dev(inst.s_hi))
        u = dev(inst.u_lo), dev(inst.u_hi)
        assert np.array_equal(P.match(t, *u).cpu().numpy().view(np.uint64), want)
        assert np.array_equal(P.match(t, *u, traversal="lane").cpu().numpy().view(np.uint64), want)
        counts, K = P.count(t, *u)
        assert K == len(want)
        assert np.array_equal(counts.cpu().numpy(), oracle.counts_per_update(want, m))
        t.free()


def count_us(inst):
    """The count traversal's time, the least of some."""
    import paper_1309_3458_amd as P
    t = P.build(dev(inst.s_lo), dev(inst.s_hi))
    u = dev(inst.u_lo), dev(inst.u_hi)
    best = np.inf
    P.match(t, *u)
    P.prof_enable(True, only="traverse_tile_count_stash")
    for _ in range(7):
        P.prof_read()
        P.match(t, *u)
        best = min(best, 1e3 * P.prof_read()["traverse_tile_count_stash"][0])
    P.prof_enable(False)
    t.free()
    return best


@pytest.mark.parametrize("kind, d, like, factor", [
    ("long either way", 2, "long updates", 3.0),
    ("all long either way", 3, "uniform", 3.0),
    ("line", 3, "uniform", 3.0),
    ("line", 4, "uniform", 3.0),
    ("plane", 4, "uniform", 3.0),
    ("16 clusters", 2, "uniform", 3.0),
    ("16 clusters", 3, "uniform", 5.0),
    ("100 clusters", 3, "uniform", 5.0),
])
def test_order_fits(kind, d, like, factor):
    n, m = 250000, 200000
    got = count_us(instance(kind, 200 + d, n, m, d))
    ref = count_us(instance(like, 300 + d, n, m, d))
    print(f"{kind} d={d}: {got:.0f} us, {like} {ref:.0f} us")
    assert got < factor * ref


@pytest.mark.parametrize("use_graph", [False, True])
def test_batch_pairs(use_graph):
    """Sets of every kind in one batch, of sizes around a class's few cells."""
    import paper_1309_3458_amd as P
    insts = [instance(kind, 400 + 10 * d + i, 700 + 900 * i, m, d) for d in (2, 3, 4)
             for i, kind in enumerate(KINDS + ["uniform"]) for m in (1, 63, 256, 5000 + 1000 * i)]
    want = [oracle.itm(i.s_lo, i.s_hi, i.u_lo, i.u_hi, threads=8) for i in insts]
    tens = [(dev(i.s_lo), dev(i.s_hi), dev(i.u_lo), dev(i.u_hi)) for i in insts]
    b = P.Batch(tens, sum(len(w) for w in want), use_graph=use_graph)
    for _ in range(3):
        b.out.fill_(-1)
        b.run()
        b.result()
        for i, w in enumerate(want):
            assert np.array_equal(b.pairs(i).cpu().numpy().view(np.uint64), w), i
    b.free()


def batch_count_us(insts):
    import paper_1309_3458_amd as P
    tens = [(dev(i.s_lo), dev(i.s_hi), dev(i.u_lo), dev(i.u_hi)) for i in insts]
    b = P.Batch(tens, 1 << 25, use_graph=False)
    best = np.inf
    b.run()
    P.prof_enable(True, only="batch_traverse_count")
    for _ in range(7):
        P.prof_read()
        b.run()
        best = min(best, 1e3 * P.prof_read()["batch_traverse_count"][0])
    P.prof_enable(False)
    b.result()
    b.free()
    return best


@pytest.mark.parametrize("kind, d, factor", [
    ("all long either way", 3, 4.0), ("long either way", 4, 4.0), ("line", 3, 4.0),
    ("plane", 4, 4.0), ("16 clusters", 2, 4.0), ("100 clusters", 3, 5.0)])
def test_batch_order_fits(kind, d, factor):
    n, m = 50000, 40000
    got = batch_count_us([instance(kind, 500 + i, n, m, d) for i in range(4)])
    ref = batch_count_us([instance("uniform", 600 + i, n, m, d) for i in range(4)])
    print(f"{kind} d={d}: {got:.0f} us, uniform {ref:.0f} us")
    assert got < factor * ref
