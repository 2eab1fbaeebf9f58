"""GPU: the hub windows' row walk (4 lanes, then 16 lanes a row), hubs cut into
id ranges, and the 8-bit counters of hubs with at most 255 lower neighbours,
against the oracle: rows whose slices end at every remainder of the steps,
at the row's start and at its end, with and without entries in the batch."""
import numpy as np
import pytest

from oracle import native

pytestmark = pytest.mark.gpu


def counts(n, k):
    return native.static_counts(n, (k // n).astype(np.int32), (k % n).astype(np.int32))


@pytest.mark.parametrize("window", ["64", "512", None])
@pytest.mark.parametrize("hubs,lows", [(40, 255), (40, 256), (300, 700)])
def test_walk_remainders(monkeypatch, window, hubs, lows):
    """`lows` vertices of lengths 1 .. 150 and more over `hubs` hubs and fillers."""
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case walk", window, hubs, lows, flush=True)
    if window:
        monkeypatch.setenv("GC_C4_WINDOW", window)
        monkeypatch.setenv("GC_C4_DENSE_MIN", "0")
    rng = np.random.default_rng(hubs + lows)
    n = hubs + lows + 900
    u, v = [], []
    for j in range(lows):  # low vertex j: j % 150 + 1 hubs and fillers
        deg = j % 150 + 1
        nb = rng.choice(hubs + 900, min(deg, hubs + 900), replace=False)
        u += [hubs + 900 + j] * nb.size
        v += nb.tolist()
    for h in range(hubs):  # hubs: nearly every filler, each other
        nb = rng.choice(np.arange(hubs, hubs + 900), 850, replace=False)
        u += [h] * nb.size
        v += nb.tolist()
        u += [h] * (hubs - h - 1)
        v += list(range(h + 1, hubs))
    u, v = np.array(u), np.array(v)
    k = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
    e = lambda x: ((x // n).astype(np.int32), (x % n).astype(np.int32))  # noqa: E731
    z = np.zeros(0, np.int32)
    with Graph(n, *e(k), delta=-1, radius=0) as g:
        assert g.counts() == counts(n, k)
        for part in (3, 400):
            gone = rng.choice(k, k.size // part, replace=False)
            k2 = np.setdiff1d(k, gone)
            assert g.apply_batch(z, z, *e(gone)) == counts(n, k2)
            assert g.apply_batch(*e(gone), z, z) == counts(n, k)
        rows = g.apply_batch_seq([(z, z) + e(gone), e(gone) + (z, z), (z, z) + e(gone[::2])])
        assert rows[1][:6] == counts(n, k)[:6] and g.counts() == counts(n, np.setdiff1d(k, gone[::2]))


@pytest.mark.parametrize("pool", [False, True])
def test_hub_cut_into_ranges(pool):
    """Hubs with far more wedges than the smallest range (65,536)."""
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case cut", pool, flush=True)
    rng = np.random.default_rng(5)
    def one(n, hubs, deg):
        u = np.repeat(np.arange(hubs), deg)
        v = rng.integers(hubs, n, u.size)
        w = rng.integers(0, n, (2, 3 * n))
        u, v = np.concatenate([u, w[0]]), np.concatenate([v, w[1]])
        k = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
        return k[k // n != k % n]
    e = lambda n, x: ((x // n).astype(np.int32), (x % n).astype(np.int32))  # noqa: E731
    sets = [(6000, one(6000, 60, 3000)), (5000, one(5000, 30, 2500))] if pool else [(9000, one(9000, 80, 5000))]
    gone = [rng.choice(k, 500, replace=False) for _, k in sets]
    z = np.zeros(0, np.int32)
    if pool:
        g = Graph.pool([n for n, _ in sets], [e(n, k)[0] for n, k in sets], [e(n, k)[1] for n, k in sets], delta=-1)
        got = g.apply_batches([(z, z) + e(n, d) for (n, _), d in zip(sets, gone)])
    else:
        g = Graph(sets[0][0], *e(*sets[0]), delta=-1)
        got = [g.apply_batch(z, z, *e(sets[0][0], gone[0]))]
    with g:
        assert got == [counts(n, np.setdiff1d(k, d)) for (n, k), d in zip(sets, gone)]
