"""List searches through the guides (one entry per slice of a list's time or
neighbour range), against the oracle: graphs on both sides of the rule that
builds them (as many vertices as edges, one more), lists whose times or
neighbours fall into one slice, times at the ends of the range, and spans on
both sides of 32-bit times."""
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


def unique(u, v, t, n):
    e = np.unique(np.stack([u, v, t], 1)[u != v], axis=0)
    return e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2].astype(np.int64), n


def make(kind):
    rng = np.random.default_rng(31)
    g = W.small_graph(3000, 32, n=60, span=20000)
    if kind == "as_many_vertices":
        return unique(g.src, g.dst, g.t, len(np.unique(np.stack([g.src, g.dst, g.t], 1), axis=0)))
    if kind == "one_vertex_more":
        return unique(g.src, g.dst, g.t, len(np.unique(np.stack([g.src, g.dst, g.t], 1), axis=0)) + 1)
    if kind == "many_idle_vertices":
        # long gaps between the vertices that have edges, ids at both ends
        ids = np.sort(rng.choice(2900, 60, replace=False))
        ids[0], ids[-1] = 0, 2899
        return unique(ids[g.src], ids[g.dst], g.t, 2900)
    if kind == "one_time":
        u, v = rng.integers(0, 50, 1500), rng.integers(0, 50, 1500)
        return unique(u, v, np.full(1500, 7), 50)
    if kind == "times_at_both_ends":
        # every list's times in the first and the last slice
        t = np.where(rng.random(3000) < 0.5, rng.integers(0, 40, 3000), 10**6 - rng.integers(0, 40, 3000))
        return unique(g.src, g.dst, t, 60)
    if kind == "near_ids":
        # every neighbour's id inside a list's first slice
        u, v, t = rng.integers(0, 9, 1500), rng.integers(0, 9, 1500), rng.integers(0, 4000, 1500)
        return unique(u, v, t, 1200)
    # spans around 32-bit times: the small graph's times stretched, the last
    # edge at the span's end
    span = {"span_31_bits": 2**31 - 1, "span_32_bits": 2**32 - 2, "span_33_bits": 2**32, "span_40_bits": 2**40 + 12345}[kind]
    t = g.t * (span // 20001)
    t[np.argmax(t)] = span
    t[np.argmin(t)] = 0
    return unique(g.src, g.dst, t, 60)


@pytest.mark.parametrize("kind", ["as_many_vertices", "one_vertex_more", "many_idle_vertices", "one_time",
                                  "times_at_both_ends", "near_ids", "span_31_bits", "span_32_bits", "span_33_bits",
                                  "span_40_bits"])
def test_weights_and_samples_match_oracle(T, kind):
    u, v, t, n = make(kind)
    print("[guides]", kind, len(u), n, flush=True)
    og, tg = O.Graph(u, v, t, n), T.Graph(u, v, t, n)
    delta = max(1, int(t.max() - t.min()) // 20)
    for name in ("3cycle", "scatter_gather", "6chain"):
        P = O.Prep(og, O.make_motif(W.MOTIFS[name], delta))
        Wt = T.Weights(tg, T.make_motif(W.MOTIFS[name], delta))
        assert Wt.W == P.W
        assert Wt.interval_weights() == P.interval_weights()
        for k in (500, 70_000):  # list searches per sample, then kept windows
            if P.W == 0 and k > 500:
                continue
            ro, reco = P.sample(3, k, records=True)
            rg, recg = Wt.sample(3, k, records=True)
            assert (reco == recg).all() and rg.estimate == ro.estimate


@pytest.mark.parametrize("kind", ["as_many_vertices", "one_vertex_more", "many_idle_vertices", "one_time",
                                  "times_at_both_ends", "near_ids", "span_31_bits", "span_32_bits", "span_33_bits",
                                  "span_40_bits"])
def test_served_samples_match_oracle(T, kind):
    """A server's sets keep no windows: each of their samples searches the
    lists, below and above the count that sorts roots."""
    u, v, t, n = make(kind)
    print("[guides] served", kind, len(u), n, flush=True)
    og, tg = O.Graph(u, v, t, n), T.Graph(u, v, t, n)
    delta = max(1, int(t.max() - t.min()) // 20)
    with T.Server(4 << 30) as server:
        gid = server.add_graph(tg)
        for name in ("3cycle", "scatter_gather", "6chain"):
            P = O.Prep(og, O.make_motif(W.MOTIFS[name], delta))
            for k in (500, 70_000):
                r, _ = server.wait(server.submit(gid, T.make_motif(W.MOTIFS[name], delta), k, 3))
                assert r.W.value == P.W
                if P.W == 0:
                    continue
                o, _ = P.sample(3, k)
                assert (r.acc2.value, r.acc2_sq.value, r.n_valid, r.n_bad_vertex, r.n_bad_delta, r.n_bad_order,
                        r.n_nonzero, r.estimate) == \
                       (o.acc2.value, o.acc2_sq.value, o.n_valid, o.n_bad_vertex, o.n_bad_delta, o.n_bad_order,
                        o.n_nonzero, o.estimate), (name, k)
