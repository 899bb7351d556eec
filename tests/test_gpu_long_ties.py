"""The canonical (t, u, v) order of graphs with times that many edges share:
their edges are listed and sorted apart from the rest, up to half of all edges
(then the full sort starts over), with one packed key and two, 32-bit and
64-bit times, runs at the first and the last time, of the longest length that
is placed without the list and one more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

M, TIE = 100_003, 256  # TIE: the most edges of one time that are placed without the list


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "no HIP device"
    from paper_2507_20441_amd import timest
    timest.lib()
    return timest


def edges(n, span, runs, seed):
    """M distinct edges: runs of the given lengths at times of their own (the
    first run at time 0, the last at the span), the rest at distinct times."""
    rng = np.random.default_rng(seed)
    at = np.linspace(0, span, len(runs)).astype(np.int64) if len(runs) > 1 else np.array([span // 3])
    parts = []
    for length, t in zip(runs, at):
        code = rng.choice(200 * 200, length, replace=False)
        u, v = code // 200, code % 200 + 200
        parts.append(np.stack([u * (n // 400), v * (n // 400) - 1, np.full(length, t)], 1))
    rest = M - sum(runs)
    t = rng.choice(min(span - 1, 40 * M), rest + len(runs), replace=False).astype(np.int64) + 1
    t = t[~np.isin(t, at)][:rest]
    u, v = rng.integers(0, n, rest), rng.integers(0, n - 1, rest)
    v = np.where(v >= u, v + 1, v)
    parts.append(np.stack([u, v, t], 1))
    # the edges whose times a build samples to see how many share one: here the
    # ones at times of their own, so that the list is tried whatever the runs
    shown = np.unique([(i * 0x9E3779B97F4A7C15 % 2**64) * M >> 64 for i in range(1, 1025)])
    e = np.empty((M, 3), np.int64)
    p = parts.pop()
    p = p[rng.permutation(rest)]
    e[shown] = p[:len(shown)]
    hidden = np.setdiff1d(np.arange(M), shown)
    e[hidden] = np.concatenate(parts + [p[len(shown):]])[rng.permutation(len(hidden))]
    assert (e[:, 0] != e[:, 1]).all()
    return e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), e[:, 2].astype(np.int64)


# vertices and span: one key of 64 bits or less, two keys; 64-bit list times, two ways
@pytest.mark.parametrize("n,span", [(3000, 10**7), (700_000, 2**30), (3000, 2**36), (700_000, 2**36)])
@pytest.mark.parametrize("runs", [[TIE] * 3, [TIE + 1], [TIE + 1, TIE, TIE + 1], [300, 257, 20_000, 259, 3000],
                                  [2500] * 20, [2500] * 20 + [3], [1] + [16_667] * 3 + [TIE],
                                  [1] + [16_667] * 3 + [TIE + 1]],
                         ids=lambda r: f"{len(r)}x{max(r)}")
def test_edge_order(T, n, span, runs):
    print("[long ties]", n, span, len(runs), sum(runs), flush=True)
    u, v, t = edges(n, span, runs, 95)
    tg = T.Graph(u, v, t, n)
    order = np.lexsort((v, u, t))
    assert (tg.export("t") == t[order] - t.min()).all()
    assert (tg.export("src") == u[order]).all() and (tg.export("dst") == v[order]).all()
    tg.close()


@pytest.mark.parametrize("n,span", [(3000, 10**7), (700_000, 2**30)])
@pytest.mark.parametrize("runs", [[300, 300], [1] + [16_667] * 3 + [TIE + 1]], ids=lambda r: f"{len(r)}x{max(r)}")
def test_duplicates_in_a_long_run_are_found(T, n, span, runs):
    u, v, t = edges(n, span, runs, 96)
    at = np.flatnonzero(t == t.max())
    u[at[17]], v[at[17]] = u[at[40]], v[at[40]]
    with pytest.raises(T.TimestError) as e:
        T.Graph(u, v, t, n)
    assert e.value.code == T.TM_EDUP
