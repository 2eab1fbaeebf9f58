"""GPU: the edge-local 4-cycles' split between rows walked against a bitmap
and pairs searched, against the oracle after every batch.

The bitmap's window is shrunk (GC_DELTA_BITS) so that ids of N(o) fall below
it on small graphs; batches change many edges at the same ends, so that
N(o) holds edges of the batch; hubs far longer than the other end's row
(searched although the edge has a bitmap) meet ends on both sides of the
smallest total that earns a bitmap."""
import numpy as np
import pytest

from graphgen import rmat_batches, rmat_graph
from oracle import native
from oracle.semantics import apply_batch as oracle_apply

pytestmark = pytest.mark.gpu


def esorted(E):
    E = sorted(E)
    return (np.array([u for u, v in E], np.int32), np.array([v for u, v in E], np.int32))


def pairs(E):
    E = sorted(E)
    return np.array([u for u, _ in E], np.int32), np.array([v for _, v in E], np.int32)


@pytest.mark.parametrize("ids", [1, 33, 500, 0])
def test_bits_window_rmat(monkeypatch, ids):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case delta bits window", ids, flush=True)
    monkeypatch.setenv("GC_DELTA_BITS", str(ids))
    n, s, d, samp = rmat_graph(11, 24, 5)
    E = set(zip(s.tolist(), d.tolist()))
    hub = int(np.bincount(np.concatenate([s, d])).argmax())
    nb = [(min(hub, x), max(hub, x)) for x in range(n) if x != hub]
    with Graph(n, s, d, delta=1) as g:
        batches = rmat_batches(n, s, d, samp, [30, 400], 6)
        # many changed edges at one hub: half its edges go, then come back
        gone = [e for e in nb if e in E][::2]
        z = np.zeros(0, np.int32)
        for b in batches + [(z, z) + pairs(gone), pairs(gone) + (z, z)]:
            got, st = g.apply_batch(*b, stats=True)
            assert st["delta"] == 1
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *esorted(E))


@pytest.mark.parametrize("ids", [64, 0])
@pytest.mark.parametrize("ds", [20, 21, 22, 24, 26])
def test_bits_lopsided_pairs(monkeypatch, ids, ds):
    """Ends o with 3 hub neighbours (64 x 4 entries against hubs of about 3,000)
    and ends s with ds hub neighbours: totals around 4,096."""
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case delta bits lopsided", ids, ds, flush=True)
    monkeypatch.setenv("GC_DELTA_BITS", str(ids))
    rng = np.random.default_rng(ds)
    hubs, ends, n = 30, 12, 3600
    E = set()
    for h in range(hubs):
        E |= {(h, int(x)) for x in rng.choice(np.arange(100, n), 3000, replace=False)}
    o = list(range(hubs, hubs + ends))
    s = list(range(hubs + ends, hubs + 2 * ends))
    for k, x in enumerate(o):
        E |= {(int(h), x) for h in rng.choice(hubs, 3, replace=False)}
    for x in s:
        E |= {(int(h), x) for h in rng.choice(hubs, ds, replace=False)}
    z = np.zeros(0, np.int32)
    so = {(x, y) for x in o for y in s[::2]}
    flip = {e for e in E if e[1] in o[::3]} | {e for e in E if e[1] in s[::4]}
    one = {(o[0], s[0])}
    with Graph(n, *esorted(E), delta=1) as g:
        for b in [pairs(one) + (z, z), pairs(so - one) + pairs(flip), pairs(flip) + pairs(so)]:
            got = g.apply_batch(*b)
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *esorted(E))
