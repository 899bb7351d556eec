"""Motif families over every kind of weight set and mix of members: trees of up
to five vertices and larger ones, 64-bit sets, 128-bit ones whose list tables
stayed 64-bit and ones rebuilt in 128 bits, counts below and above the one
that sorts roots, members with general runs (which go one by one) between
others (up to four a pass).  Every member equals the oracle's own run, or where
the oracle would take minutes (its weights are quadratic in a vertex's edges)
the library's own."""
import numpy as np
import pytest

import oracle as O
from paper_2507_20441_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


def path(n):
    return tuple((i, i + 1) for i in range(n - 1))


def star(n):
    return tuple((0, i) for i in range(1, n))


def hub(degree, others, n, span, seed):
    """A vertex 0 with `degree` edges to the others, and `others` edges from those."""
    rng = np.random.default_rng(seed)
    u = np.r_[np.zeros(degree, np.int64), rng.integers(1, n, others)]
    v = np.r_[rng.integers(1, n, degree), rng.integers(0, n, others)]
    t = rng.integers(0, span, degree + others)
    e = np.unique(np.stack([u, v, t], 1)[u != v], axis=0)
    e = e[rng.permutation(len(e))]
    return e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2].astype(np.int64), n


def small():
    g = W.small_graph(20_000, 51, n=300, span=200_000)
    return g.src, g.dst, g.t, g.n


# tree, its center's index, graph, delta; wide: the set's width (its list
# tables' width is not visible: products above 2^64 need 128-bit ones)
SETS = {
    "five_vertices": (path(5), 2, small, 3000, False),
    "six_vertices": (path(6), 2, small, 3000, False),
    "eight_vertices": (path(8), 3, small, 900, False),
    "wide_small_tree": (star(5), 0, lambda: hub(110_000, 60_000, 400, 10**6, 71), 10**6, True),
    "wide_totals": (star(7), 0, lambda: hub(3000, 30_000, 60, 5000, 72), 5000, True),
    "wide_products": (star(7), 0, lambda: hub(8000, 30_000, 60, 5000, 73), 5000, True),
}


def members(tree):
    """Members by name: g_ with general runs (edges before the tree and after
    it, or three in a row)."""
    a, b, c = len(set(x for e in tree for x in e)) - 1, 1, 2  # some vertices no tree edge joins
    pairs = [p for p in ((a, 0), (a, b), (b, a), (c, 0), (a, c), (2, 1)) if p not in tree]
    p, q, r = pairs[:3]
    mid = len(tree) // 2
    return [("tree", tree), ("one", tree + (p,)), ("lead", (q,) + tree), ("g_around", (p,) + tree + (q,)),
            ("between", tree[:mid] + (p,) + tree[mid:]), ("two", tree + (p, q)), ("g_three", tree + (p, q, r)),
            ("two_lead", (q, r) + tree), ("apart", tree[:1] + (q,) + tree[1:mid] + (r,) + tree[mid:]),
            ("other", tree + (r,)), ("again", tree + (q,))]


@pytest.mark.parametrize("k", [9_001, 70_001])
@pytest.mark.parametrize("name", SETS)
def test_every_member_equals_the_oracle(T, name, k):
    tree, center, make, delta, wide = SETS[name]
    u, v, t, n = make()
    tg = T.Graph(u, v, t, n)
    og = O.Graph(u, v, t, n) if not wide or (k < 10_000 and len(u) < 100_000) else None
    w = T.Weights(tg, T.make_motif(tree, delta), T.make_tree(list(range(len(tree))), center))
    assert w.info()["wide"] == wide and w.W > 0
    fam = members(tree)
    want = []
    for nm, edges in fam:
        idx = [edges.index(e) for e in tree]
        if og is None:
            alone = T.Weights(tg, T.make_motif(edges, delta), T.make_tree(idx, idx[center]))
            want.append(alone.sample(13, k)[0])
            alone.close()
            continue
        P = O.Prep(og, O.make_motif(edges, delta), O.make_tree(idx, idx[center]))
        assert P.W == w.W
        want.append(P.sample(13, k)[0])
    print("[family]", name, k, w.W, [r.n_nonzero for r in want], flush=True)
    # all together, then prefixes: passes of one to four members
    for take in ([len(fam)] if name.startswith("wide") else [len(fam), 1, 2, 3, 5]):
        got = T.sample_family(w, [T.make_motif(e, delta) for _, e in fam[:take]], 13, k)
        for (nm, _), r, o in zip(fam, got, want):
            assert r.status == 0, nm
            assert (r.acc2.value, r.acc2_sq.value, r.n_valid, r.n_bad_vertex, r.n_bad_delta, r.n_bad_order,
                    r.n_nonzero, r.estimate, r.std_error) == \
                   (o.acc2.value, o.acc2_sq.value, o.n_valid, o.n_bad_vertex, o.n_bad_delta, o.n_bad_order,
                    o.n_nonzero, o.estimate, o.std_error), (nm, take)
