"""Pair ranks (an edge's place in its lists' other orders, and the gaps to its
pair's neighbouring edges) against the oracle: graphs one edge below the size
that keeps them and just at it, pairs that meet many times (gaps below, at and
above delta, in both directions), with 32-bit and 64-bit times."""
import numpy as np
import pytest

import oracle as O
from paper_2507_20441_amd import workloads as W

pytestmark = pytest.mark.gpu

KEEP_FROM = 1 << 19


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


def graph(m, n, scale, seed):
    """m distinct edges over n vertices; a third of them answer an earlier edge
    of the reversed pair at the same time, or repeat their own pair, within a
    few seconds."""
    rng = np.random.default_rng(seed)
    g = W.small_graph(m, seed, n=n, span=m // 16)
    u, v, t = g.src.astype(np.int64), g.dst.astype(np.int64), g.t.copy()
    pick = rng.choice(m, m // 3, replace=False)
    rev = rng.random(pick.size) < 0.5
    u2, v2 = np.where(rev, v[pick], u[pick]), np.where(rev, u[pick], v[pick])
    e = np.stack([np.r_[u, u2], np.r_[v, v2], np.r_[t, t[pick] + rng.integers(0, 8, pick.size)]], 1)
    e = np.unique(e, axis=0)
    e = e[rng.permutation(len(e))[:m]]
    return e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2] * scale, n


# (the largest graph's times need 64 bits)
@pytest.mark.parametrize("m,n,scale", [(KEEP_FROM - 1, 3000, 1), (KEEP_FROM, 3000, 1), (KEEP_FROM + 77, 150, 1),
                                       (KEEP_FROM + 4096, 3000, 1 << 20)])
def test_weights_and_samples_match_oracle(T, m, n, scale):
    u, v, t, n = graph(m, n, scale, 41)
    print("[ranks]", m, n, scale, flush=True)
    og, tg = O.Graph(u, v, t, n), T.Graph(u, v, t, n)
    for name, delta in (("scatter_gather", 60), ("6chain", 100), ("4cycle", 20)):
        P = O.Prep(og, O.make_motif(W.MOTIFS[name], delta * scale))
        Wt = T.Weights(tg, T.make_motif(W.MOTIFS[name], delta * scale))
        assert Wt.W == P.W and P.W > 0
        assert Wt.interval_weights() == P.interval_weights()
        ro, reco = P.sample(3, 70_000, records=True)
        rg, recg = Wt.sample(3, 70_000, records=True)
        assert (reco == recg).all() and rg.estimate == ro.estimate
    # children a partial order leaves unordered with their parent
    edges, before = W.PO_MOTIFS["po_diamond"]
    P = O.Prep(og, O.make_motif(edges, 30 * scale, before=before))
    Wt = T.Weights(tg, T.make_motif(edges, 30 * scale, before=before))
    assert Wt.W == P.W
    ro, reco = P.sample(3, 20_000, records=True)
    rg, recg = Wt.sample(3, 20_000, records=True)
    assert (reco == recg).all() and rg.estimate == ro.estimate


@pytest.mark.parametrize("n,scale", [(3000, 1), (150, 1), (3000, 1 << 20)])
def test_served_samples_match_oracle(T, n, scale):
    """A server's sets keep no windows: its samples search them, with the pair
    ranks for the excluded runs."""
    u, v, t, n = graph(KEEP_FROM + 5, n, scale, 43)
    print("[ranks] served", n, scale, flush=True)
    og, tg = O.Graph(u, v, t, n), T.Graph(u, v, t, n)
    with T.Server(8 << 30) as server:
        gid = server.add_graph(tg)
        for name, delta in (("scatter_gather", 60), ("6chain", 100), ("4cycle", 20)):
            r, _ = server.wait(server.submit(gid, T.make_motif(W.MOTIFS[name], delta * scale), 70_000, 3))
            ro, _ = O.Prep(og, O.make_motif(W.MOTIFS[name], delta * scale)).sample(3, 70_000)
            for f in ("W", "acc2", "acc2_sq"):
                assert getattr(r, f).value == getattr(ro, f).value, (name, f)
            assert (r.n_valid, r.n_bad_vertex, r.n_bad_order) == (ro.n_valid, ro.n_bad_vertex, ro.n_bad_order), name
            assert r.estimate == ro.estimate, name
