"""When a graph gets its pair ranks: not with the graph, but with the first call
that they pay for (eight level launches of one graph in all, or from 2^22 edges
on a set of three); a build that cannot have their memory goes on without;
threads and recorded plans that meet a graph for the first time agree with one
that has them, and so does the oracle."""
import threading

import numpy as np
import pytest

import oracle as O
from paper_2507_20441_amd import workloads as W

pytestmark = pytest.mark.gpu

M = (1 << 19) + 11
RANKS = 2 * ((16 * M + 255) // 256 * 256)
PATH2 = ((0, 1), (1, 2))  # one level launch
AT_ONCE = 1 << 22


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


@pytest.fixture(scope="module")
def edges():
    g = W.small_graph(M, 44, n=4000, span=M // 8)
    return g.src, g.dst, g.t, g.n


def fields(r):
    return (r.W.value, r.acc2.value, r.acc2_sq.value, r.n_valid, r.n_bad_vertex, r.n_bad_order, r.n_nonzero)


def test_the_build_that_pays_makes_them(T, edges):
    g = T.Graph(*edges)
    alone = g.info()["bytes"]
    chain = T.make_motif(W.MOTIFS["6chain"], 50)
    path = T.make_motif(PATH2, 50)
    for _ in range(7):
        T.Weights(g, path).close()
        assert g.info()["bytes"] == alone
    w0 = T.Weights(g, path)  # the eighth launch
    assert g.info()["bytes"] == alone + RANKS
    h = T.Graph(*edges)
    w1 = T.Weights(h, path)  # the same set without them
    assert h.info()["bytes"] == alone
    assert fields(w0.sample(5, 100_000)[0]) == fields(w1.sample(5, 100_000)[0])
    w2 = T.Weights(h, chain)  # four launches more
    assert h.info()["bytes"] == alone
    w3 = T.Weights(h, chain)
    assert h.info()["bytes"] == alone + RANKS and w3.W == w2.W
    # a set that was there before reads them from now on
    assert fields(w0.sample(6, 100_000)[0]) == fields(w1.sample(6, 100_000)[0])
    assert fields(T.Weights(g, chain).sample(5, 100_000)[0]) == fields(w2.sample(5, 100_000)[0])
    e = T.Graph(*edges)
    for rep in range(3):
        assert fields(T.estimate(e, chain, 100_000, 5)) == fields(w2.sample(5, 100_000)[0])
        assert e.info()["bytes"] == alone + (RANKS if rep else 0)
    c = T.Graph(*edges)
    T.choose_tree(c, chain, 2)  # eight launches of one call
    assert c.info()["bytes"] == alone + RANKS


def test_a_graph_below_the_size_has_none(T):
    g = W.small_graph((1 << 19) - 1, 44, n=4000, span=M // 8)
    tg = T.Graph(g.src, g.dst, g.t, g.n)
    alone = tg.info()["bytes"]
    T.Weights(tg, T.make_motif(W.MOTIFS["6chain"], 50)).close()
    assert tg.info()["bytes"] == alone


@pytest.mark.parametrize("m", [AT_ONCE - 1, AT_ONCE])
def test_large_graphs_have_them_at_once(T, m):
    rng = np.random.default_rng(45)
    u = rng.integers(0, 9000, m)
    v = (u + 1 + rng.integers(0, 8999, m)) % 9000
    g = T.Graph(u.astype(np.int32), v.astype(np.int32), rng.permutation(m).astype(np.int64), 9000)
    alone = g.info()["bytes"]
    ranks = 2 * ((16 * m + 255) // 256 * 256)
    T.Weights(g, T.make_motif(W.MOTIFS["4cycle"], 50)).close()  # two launches
    assert g.info()["bytes"] == alone
    T.Weights(g, T.make_motif(W.MOTIFS["scatter_gather"], 50)).close()  # three
    assert g.info()["bytes"] == alone + (ranks if m >= AT_ONCE else 0)


def make_ranks(T, g):
    path = T.make_motif(PATH2, 50)
    for _ in range(8):
        T.Weights(g, path).close()


@pytest.mark.parametrize("scale", [1, 1 << 20])
def test_every_motif_with_ranks_matches_oracle(T, scale):
    # a third of the edges answer or repeat an earlier one within seconds
    rng = np.random.default_rng(48)
    g = W.small_graph(M, 48, n=3000, span=M // 16)
    pick = rng.choice(M, M // 3, replace=False)
    rev = rng.random(pick.size) < 0.5
    e = np.stack([np.r_[g.src, np.where(rev, g.dst[pick], g.src[pick])],
                  np.r_[g.dst, np.where(rev, g.src[pick], g.dst[pick])],
                  np.r_[g.t, g.t[pick] + rng.integers(0, 8, pick.size)]], 1)
    e = np.unique(e, axis=0)
    e = e[rng.permutation(len(e))[:M]]
    u, v, t = e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2].astype(np.int64) * scale
    og, tg = O.Graph(u, v, t, 3000), T.Graph(u, v, t, 3000)
    alone = tg.info()["bytes"]
    make_ranks(T, tg)
    assert tg.info()["bytes"] == alone + RANKS
    motifs = [(x, W.MOTIFS[x], None) for x in W.MOTIFS] + [("po_diamond", *W.PO_MOTIFS["po_diamond"])]
    for name, edges, before in motifs:
        delta = 60 * scale
        P = O.Prep(og, O.make_motif(edges, delta, before=before))
        Wt = T.Weights(tg, T.make_motif(edges, delta, before=before))
        assert Wt.W == P.W and P.W > 0, name
        assert Wt.interval_weights() == P.interval_weights(), name
        ro, reco = P.sample(3, 66_000, records=True)
        rg, recg = Wt.sample(3, 66_000, records=True)
        assert (reco == recg).all() and rg.estimate == ro.estimate, name


def test_without_their_memory_the_build_goes_on(T, edges):
    A = T.TorchAllocator()
    g, h = T.Graph(*edges, allocator=A), T.Graph(*edges)
    alone = g.info()["bytes"]
    mo = T.make_motif(W.MOTIFS["6chain"], 50)
    T.Weights(g, mo).close()
    A.fail_next = 1  # the ranks' memory is the first that the second build asks for
    w = T.Weights(g, mo)
    assert A.failed == 1 and g.info()["bytes"] == alone
    assert fields(w.sample(5, 100_000)[0]) == fields(T.Weights(h, mo).sample(5, 100_000)[0])
    w.close()
    T.Weights(g, mo).close()  # not asked for again
    assert g.info()["bytes"] == alone
    g.close()
    assert A.live_bytes == 0


def test_threads_on_a_new_graph(T, edges):
    import torch
    mo = [T.make_motif(W.MOTIFS[x], 50) for x in ("6chain", "scatter_gather", "4cycle", "6chain")]
    h = T.Graph(*edges)
    want = [fields(T.Weights(h, x).sample(5, 100_000)[0]) for x in mo]
    g = T.Graph(*edges)
    got, gate = [None] * 4, threading.Barrier(4)

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            gate.wait()
            got[i] = [fields(T.Weights(g, mo[i]).sample(5, 100_000)[0]) for _ in range(2)]

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for x in threads:
        x.start()
    for x in threads:
        x.join()
    assert got == [[x, x] for x in want]


def test_recorded_plans_have_them(T, edges):
    mo = [T.make_motif(W.MOTIFS[x], 50) for x in ("6chain", "4cycle")]
    g = T.Graph(*edges)
    alone = g.info()["bytes"]
    plan = T.BatchPlan([g, g], mo, [100_000, 70_000], [5, 6])
    assert g.info()["bytes"] == alone + RANKS
    h = T.Graph(*edges)
    want = [fields(T.Weights(h, x).sample(s, k)[0]) for x, s, k in zip(mo, (5, 6), (100_000, 70_000))]
    for _ in range(3):
        assert [fields(r) for r in plan.run()] == want
    plan.close()
