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
