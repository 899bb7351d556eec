"""The radix sorts at the sizes where their tiles change (256 lanes of 4 or of
16 keys, the change at 2^18 keys) and with ragged last tiles: every array a
graph build sorts, against numpy's stable sorts, for graphs whose canonical
order takes one sort or two and lists with 32-bit or 64-bit times."""
import numpy as np
import pytest

from paper_2507_20441_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


@pytest.mark.parametrize("span,n", [(5000, 900), (2**34, 900), (2**29, 2**19 + 5)])
@pytest.mark.parametrize("m", [1023, 1024, 1025, 4097, 2**18, 2**18 + 1, 2**18 + 4096])
def test_graph_arrays(T, m, span, n):
    print("[sort tiles]", m, span, n, flush=True)
    g = W.small_graph(m, 61, n=n, span=span)
    tg = T.Graph(g.src, g.dst, g.t, g.n)
    order = np.lexsort((g.dst, g.src, g.t))
    s, d, t = g.src[order], g.dst[order], g.t[order] - g.t.min()
    assert (tg.export("src") == s).all() and (tg.export("dst") == d).all() and (tg.export("t") == t).all()
    bt = max(1, int(t.max()).bit_length())
    for name, own, nbr in (("out", s, d), ("in", d, s)):
        eid = np.argsort(own, kind="stable")
        assert (tg.export(f"{name}_eid") == eid).all(), name
        assert (tg.export(f"{name}_off") == np.searchsorted(own[eid], np.arange(n + 1))).all(), name
        assert (tg.export(f"{name}_t") == t[eid]).all() and (tg.export(f"{name}_nbr") == nbr[eid]).all(), name
        pos = np.empty(m, np.int64)
        pos[eid] = np.arange(m)
        assert (tg.export(f"{name}_pos") == pos).all(), name
        neid = np.lexsort((t, nbr, own))
        assert (tg.export(f"{name}n_eid") == neid).all(), name
        assert (tg.export(f"{name}n_pos") == pos[neid]).all(), name
        key = (nbr[neid].astype(np.uint64) << np.uint64(bt)) | t[neid].astype(np.uint64)
        assert (tg.export(f"{name}n_key") == key).all(), name


@pytest.mark.parametrize("k", [2**16, 2**18, 2**18 + 1])
def test_root_sort_changes_nothing(T, k):
    # a run equals the sum of its pieces below the size that sorts
    g = W.small_graph(5000, 62, n=200, span=30000)
    w = T.Weights(T.Graph(g.src, g.dst, g.t, g.n), T.make_motif(W.MOTIFS["4cycle"], 600))
    whole, _ = w.sample(9, k)
    parts = [w.sample(9, k, j0=j, count=min(50_000, k - j), k_total=k)[0] for j in range(0, k, 50_000)]
    for f in ("acc2", "acc2_sq"):
        assert getattr(whole, f).value == sum(getattr(p, f).value for p in parts), f
    for f in ("n_valid", "n_bad_vertex", "n_bad_delta", "n_bad_order", "n_nonzero"):
        assert getattr(whole, f) == sum(getattr(p, f) for p in parts), f
    assert whole.n_nonzero > 0
