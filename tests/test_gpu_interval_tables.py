"""Interval bounds and the prefix of the interval weights at the sizes where
their kernels change (one chunk of a block, waves or lanes per search), around
a whole scan tile of edges, and for a delta near the largest, against the
oracle."""
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


def check(T, u, v, t, n, delta, q):
    og, tg = O.Graph(u, v, t, n), T.Graph(u, v, t, n)
    for name in ("4star", "4cycle"):
        P = O.Prep(og, O.make_motif(W.MOTIFS[name], delta))
        Wt = T.Weights(tg, T.make_motif(W.MOTIFS[name], delta))
        assert P.q == Wt.info()["q"] == q
        assert Wt.W == P.W and Wt.interval_weights() == P.interval_weights()
        ro, reco = P.sample(7, 2000, records=True)
        rg, recg = Wt.sample(7, 2000, records=True)
        assert (reco == recg).all() and rg.estimate == ro.estimate


@pytest.mark.parametrize("q", [1, 2, 63, 64, 65, 4095, 4096, 4097, 16384, 16385])
def test_interval_counts(T, q):
    print("[intervals]", q, flush=True)
    delta = 40
    g = W.small_graph(3000, 51, n=60, span=20000)
    t = (g.t - g.t.min()) * ((q - 1) * delta + delta // 2) // (g.t.max() - g.t.min())
    e = np.unique(np.stack([g.src, g.dst, t], 1), axis=0)
    e[np.argmax(e[:, 2]), 2] = (q - 1) * delta + delta // 2
    e[np.argmin(e[:, 2]), 2] = 0
    e = np.unique(e, axis=0)
    check(T, e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2].astype(np.int64), 60, delta, q)


@pytest.mark.parametrize("m", [1, 2, 2047, 2048, 2049, 4096])
def test_edge_counts(T, m):
    print("[intervals] edges", m, flush=True)
    g = W.small_graph(m, 52, n=max(2, m // 30), span=5000)
    check(T, g.src, g.dst, g.t, g.n, 300, int(g.t.max() - g.t.min()) // 300 + 1)


@pytest.mark.parametrize("delta", [2**31, 2**61 + 12345, 2**62 - 1])
def test_delta_near_the_largest(T, delta):
    # one or two intervals whose ends lie far past every time
    print("[intervals] delta", delta, flush=True)
    g = W.small_graph(2000, 53, n=60, span=5000)
    check(T, g.src, g.dst, g.t, g.n, delta, 1)
    if delta < 2**61:
        t = g.t - g.t.min()
        t = np.where(t > 2500, t + delta, t)
        check(T, g.src, g.dst, t, g.n, delta, 2)
