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
