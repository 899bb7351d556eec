"""Graph builds when memory is short: the second sort buffers and the search
guides are asked for last, and a build that gets none of them goes on without,
with the same arrays, weights and samples; one that cannot have what every
graph needs returns TM_ENOMEM and gives everything back."""
import numpy as np
import pytest

from paper_2507_20441_amd import workloads as W

pytestmark = pytest.mark.gpu

M, N = 60_001, 3000


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


def limited(T, limit):
    """An allocator that has `limit` bytes in all (its attribute `limit`)."""
    A = T.TorchAllocator()
    A.limit = limit
    serve = A._fa

    def alloc(ctx, nbytes, stream):
        if A.live_bytes + nbytes > A.limit:
            A.failed += 1
            return None
        return serve(ctx, nbytes, stream)

    A._limited = T.ALLOC_FN(alloc)
    A.struct = T.Allocator(A._limited, A._ff, None)
    return A


def whole_blocks(nbytes):
    return (nbytes + 255) // 256 * 256


ARRAYS = [f"{d}{x}" for d in ("out", "in") for x in ("_off", "_eid", "_t", "_nbr", "_pos", "n_eid", "n_pos", "n_key")]


def samples(w):
    return [(r.W.value, r.acc2.value, r.acc2_sq.value, r.n_valid, r.n_bad_vertex, r.n_bad_order)
            for r in (w.sample(4, k)[0] for k in (5000, 100_000))]


@pytest.mark.parametrize("span", [10**6, 2**36])
def test_builds_go_on_without_optional_memory(T, span):
    g = W.small_graph(M, 46, n=N, span=span)
    s, d, t = (np.ascontiguousarray(x) for x in (g.src, g.dst, g.t))
    free = limited(T, 1 << 40)
    whole = T.Graph(s, d, t, N, allocator=free)
    peak = free.peak_bytes
    second = whole_blocks(M * (24 + (4 if span < 2**32 else 8)))
    guides = whole_blocks(4 * 4 * ((M >> 3) + N + 1))
    mo = T.make_motif(W.MOTIFS["scatter_gather"], span // 100)
    want = samples(T.Weights(whole, mo))
    assert want[0][0] > 0
    for missing, lost in ((second, 0), (second + guides, guides)):
        A = limited(T, peak - missing)
        tg = T.Graph(s, d, t, N, allocator=A)
        assert A.failed == (2 if lost else 1)
        assert tg.info()["bytes"] == whole.info()["bytes"] - lost
        for name in ARRAYS:
            assert (tg.export(name) == whole.export(name)).all(), name
        A.limit = 1 << 40
        w = T.Weights(tg, mo)
        assert samples(w) == want
        w.close()
        tg.close()
        assert A.live_bytes == 0
    for missing in (second + guides + 256, peak // 2, peak - 512):
        A = limited(T, peak - missing)
        with pytest.raises(T.TimestError) as e:
            T.Graph(s, d, t, N, allocator=A)
        assert e.value.code == T.TM_ENOMEM and A.live_bytes == 0
