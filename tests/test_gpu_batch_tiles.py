"""Batched passes take the tile that the caller chose, whatever the pass's size
(the default alone is fitted to it): the device memory of a pass holds its
tiles, so it shrinks as they grow; results equal each job's own run."""
import pytest

from paper_2507_20441_amd import workloads as W

pytestmark = pytest.mark.gpu

TILES = (256, 512, 1024, 2048, 4096, 16384, 32768)
KS = (300_001, 65_536, 700_000, 1)


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


def fields(r):
    return (r.W.value, r.acc2.value, r.acc2_sq.value, r.n_valid, r.n_bad_vertex, r.n_bad_delta, r.n_bad_order,
            r.n_nonzero, r.estimate)


def test_the_chosen_tile_is_used(T):
    g = W.small_graph(30_000, 47, n=900, span=500_000)
    A = T.TorchAllocator()
    tg = T.Graph(g.src, g.dst, g.t, g.n, allocator=A)
    ws = [T.Weights(tg, T.make_motif(W.MOTIFS[x], 3000)) for x in ("4cycle", "6chain", "scatter_gather", "3cycle")]
    want = [fields(w.sample(9 + i, k)[0]) for i, (w, k) in enumerate(zip(ws, KS))]

    def asked(tile):
        prev = T.batch_config(tile)
        try:
            before = A.live_bytes
            A.peak_bytes = before
            got = T.sample_batch(ws, KS, [9 + i for i in range(4)])
            print("[tiles]", tile, A.peak_bytes - before, flush=True)
            assert [fields(r) for r in got] == want, tile
            return A.peak_bytes - before
        finally:
            T.batch_config(*prev)

    sizes = [asked(x) for x in TILES]
    assert sizes == sorted(sizes, reverse=True) and len(set(sizes)) == len(sizes), sizes
    # the default: about 8192 tiles, of 512 samples in passes as small as this one
    assert asked(8192) == asked(512)
