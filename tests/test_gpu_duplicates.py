"""Graphs with tuples given more than once, above the size from which graphs
keep pair ranks: refused with TM_EDUP however often a tuple is repeated,
through the order by time first (whose flags the host reads before any list is
built: nothing more is allocated then) and through the full sort."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

M = (1 << 19) + 3


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


def edges(n, span, times, copies):
    """M distinct edges at `times` distinct times, then more copies of one."""
    rng = np.random.default_rng(91)
    u, v = rng.integers(0, n, 2 * M), rng.integers(0, n - 1, 2 * M)
    v = np.where(v >= u, v + 1, v)
    t = rng.integers(0, times, 2 * M) * (span // times)
    e = np.unique(np.stack([u, v, t], 1), axis=0)
    e = e[rng.permutation(len(e))[:M]]
    assert len(e) == M
    e = np.concatenate([e, np.repeat(e[1000:1001], copies, 0)])
    e = e[rng.permutation(len(e))]
    return e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2].astype(np.int64)


# (2^19 edges at 4000 times: 130 at one time, more than the order by time takes)
@pytest.mark.parametrize("copies", [1, 2, 300])
@pytest.mark.parametrize("n,span,times,early", [(3000, 10**6, 10**6, True), (700_000, 2**30, 2**30, True),
                                                (3000, 10**6, 4000, False)])
def test_repeated_tuples_are_refused(T, n, span, times, early, copies):
    print("[duplicates]", n, span, times, copies, flush=True)
    u, v, t = edges(n, span, times, copies)
    A = T.TorchAllocator()
    with pytest.raises(T.TimestError) as e:
        T.Graph(u, v, t, n, allocator=A)
    assert e.value.code == T.TM_EDUP
    assert A.live_bytes == 0
    refused = A.peak_bytes
    keep = np.unique(np.stack([u, v, t], 1), axis=0, return_index=True)[1]
    g = T.Graph(u[keep], v[keep], t[keep], n, allocator=A)
    if early and copies < 300:
        # (300 copies of one tuple are a long run of one time)
        assert refused < A.peak_bytes // 2
    g.close()
    assert A.live_bytes == 0
