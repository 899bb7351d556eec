"""The canonical (t, u, v) order of graphs sorted by time first: runs of equal
times short and too long for that path (which then sorts in full), both sides
of its density rule, one packed key and two, and duplicates among equal
times."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

M, TIE = 1 << 18, 256  # TIE: the longest run the first path looks through on one side


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


def edges(m, n, span, seed, run=0):
    """m distinct edges with times uniform in [0, span]; the first `run` of them
    at one time."""
    rng = np.random.default_rng(seed)
    u, v = rng.integers(0, n, 2 * m), rng.integers(0, n - 1, 2 * m)
    v = np.where(v >= u, v + 1, v)
    t = rng.integers(0, span + 1, 2 * m)
    e = np.unique(np.stack([u, v, t], 1), axis=0)
    e = e[rng.permutation(len(e))[:m]]
    assert len(e) == m
    if run:
        # distinct pairs share the time span // 2
        k = np.arange(run)
        e[:run] = np.stack([k % n, (k % n + 1 + k // n) % n, np.full(run, span // 2)], 1)
        rest = e[run:]
        rest[rest[:, 2] == span // 2, 2] += 1
        e = np.unique(e, axis=0)
    e = e[rng.permutation(len(e))]
    e[0, 2], e[1, 2] = 0, span
    return e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2].astype(np.int64)


@pytest.mark.parametrize("m,n,span,run", [
    (40, 30, 5, 0), (40, 30, 4, 0), (M, 3000, 10**6, 0), (M + 3, 3000, M // 8, 0),
    (M + 3, 3000, (M + 3) // 8 - 1, 0), (M, 3000, 10**6, TIE), (M, 3000, 10**6, TIE + 1),
    (M, 3000, 10**6, 5000), (M, 700_000, 2**30, 0), (M, 700_000, 2**30, 2 * TIE),
    (M, 3000, 2**36, 100)])
def test_edge_order(T, m, n, span, run):
    print("[time order]", m, n, span, run, flush=True)
    u, v, t = edges(m, n, span, 81, run)
    assert len(np.unique(np.stack([u, v, t], 1), axis=0)) == len(u)
    tg = T.Graph(u, v, t, n)
    order = np.lexsort((v, u, t))
    assert (tg.export("t") == t[order] - t.min()).all()
    assert (tg.export("src") == u[order]).all() and (tg.export("dst") == v[order]).all()


@pytest.mark.parametrize("n,run", [(3000, 10), (3000, 5000), (700_000, 10)])
def test_duplicates_are_found(T, n, run):
    u, v, t = edges(M, n, 10**6 if n < 10**5 else 2**30, 82, run)
    at = np.flatnonzero(t == np.sort(t)[len(t) // 3])[0]
    u, v, t = np.r_[u, u[at]], np.r_[v, v[at]], np.r_[t, t[at]]
    with pytest.raises(T.TimestError) as e:
        T.Graph(u, v, t, n)
    assert e.value.code == T.TM_EDUP
