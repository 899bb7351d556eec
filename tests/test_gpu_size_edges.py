"""Graph arrays and weights on both sides of 2^22 edges, where the list sorts of
the two directions run together or in turn and the scans of the weights take
their tile sums in one launch or in groups: the arrays against numpy's stable
sorts, with 32-bit and 64-bit times, and the totals of a 64-bit and a 128-bit
weight set on a graph whose weights are known."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EDGE = 1 << 22


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


@pytest.mark.parametrize("span", [2**31, 2**36])
@pytest.mark.parametrize("m", [EDGE, EDGE + 1])
def test_graph_arrays(T, m, span):
    print("[size edges]", m, span, flush=True)
    n = 40_000
    rng = np.random.default_rng(98)
    u, v = rng.integers(0, n, m), rng.integers(0, n - 1, m)
    v = np.where(v >= u, v + 1, v)
    t = np.sort(rng.integers(0, span - m, m)) + np.arange(m)  # distinct times
    t = t[rng.permutation(m)]
    t[0], t[1] = 0, span
    u, v = u.astype(np.int32), v.astype(np.int32)
    tg = T.Graph(u, v, t, n)
    order = np.argsort(t, kind="stable")
    s, d, t = u[order], v[order], t[order]
    bt = int(t.max()).bit_length()
    for name, own, nbr in (("out", s, d), ("in", d, s)):
        eid = np.argsort(own, kind="stable")
        assert (tg.export(f"{name}_eid") == eid).all(), name
        assert (tg.export(f"{name}_t") == t[eid]).all() and (tg.export(f"{name}_nbr") == nbr[eid]).all(), name
        pos = np.empty(m, np.int64)
        pos[eid] = np.arange(m)
        assert (tg.export(f"{name}_pos") == pos).all(), name
        neid = np.argsort(own.astype(np.int64) * n + nbr, kind="stable")
        assert (tg.export(f"{name}n_eid") == neid).all(), name
        assert (tg.export(f"{name}n_pos") == pos[neid]).all(), name
        key = (nbr[neid].astype(np.uint64) << np.uint64(bt)) | t[neid].astype(np.uint64)
        assert (tg.export(f"{name}n_key") == key).all(), name


@pytest.mark.parametrize("m", [EDGE, EDGE + 1])
def test_weights(T, m):
    """Disjoint paths of three edges, each one partial match in two intervals,
    and in the first interval x -> a, then `hub` times a -> h, then h -> `hub`
    others: below a -> h five edges out of h give hub^5 each, which is a 64-bit
    product, and hub^6 in all, which is not."""
    print("[size edges] weights", m, flush=True)
    hub, delta = 5000, 12_000
    paths = (m - 2 * hub - 1) // 3
    k, h = np.arange(paths), np.arange(hub)
    base = hub + 3
    u = [base + 4 * k + i for i in range(3)] + [np.zeros(1, np.int64), np.ones(hub, np.int64), np.full(hub, 2)]
    v = [base + 4 * k + i + 1 for i in range(3)] + [np.ones(1, np.int64), np.full(hub, 2), 3 + h]
    t = [20_000 + 4 * k + i for i in range(3)] + [np.zeros(1, np.int64), 1 + h, 6000 + h]
    u, v, t = (np.concatenate(x) for x in (u, v, t))
    # single edges up to m
    rest = m - len(u)
    n = base + 4 * paths + 2 * rest
    i = np.arange(rest)
    u, v, t = np.r_[u, n - 1 - 2 * i], np.r_[v, n - 2 - 2 * i], np.r_[t, 30_000 + i]
    assert len(u) == m
    order = np.random.default_rng(99).permutation(m)
    u, v, t = u[order].astype(np.int32), v[order].astype(np.int32), t[order].astype(np.int64)
    tg = T.Graph(u, v, t, n)
    w = T.Weights(tg, T.make_motif(((0, 1), (1, 2), (2, 3)), delta), T.make_tree([0, 1, 2], 0))
    assert not w.info()["wide"] and w.W == 2 * paths + hub * hub
    w.close()
    star = ((0, 1), (1, 2)) + tuple((2, 3 + i) for i in range(5))
    w = T.Weights(tg, T.make_motif(star, delta), T.make_tree(list(range(7)), 0))
    assert w.info()["wide"] and w.W == 2 * paths + hub**6
    r, _ = w.sample(3, 100_000)
    # every sample is a match of the hub's, its five ends distinct or not
    assert r.n_valid + r.n_bad_vertex + r.n_bad_order == 100_000 and r.n_valid > 0
    w.close()
