"""GPU: the triangle counts kept per edge and per vertex after passes that are
known to have taken the path: an allocation-free region pass that succeeds, and
one that outgrows the scratch and is undone, each between edge-local passes
that use the kept counts, against the oracle."""
import numpy as np
import pytest

from graphgen import rmat_batches, rmat_graph
from oracle import native
from oracle.semantics import apply_batch as oracle_apply

pytestmark = pytest.mark.gpu

Z = np.zeros(0, np.int32)


def pairs(E):
    E = sorted(E)
    return np.array([u for u, _ in E], np.int32), np.array([v for _, v in E], np.int32)


def dev(b):
    import torch
    return [torch.tensor(np.asarray(x, np.int32), device="cuda") for x in b]


def local(g, n, E, b):
    got, st = g.apply_batch(*b, stats=True)
    assert st["delta"] == 1
    oracle_apply(E, n, *b)
    assert got == native.static_counts(n, *pairs(E))


@pytest.mark.parametrize("radius", [0, 2])
def test_allocation_free_region_passes(radius):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case kept, allocation-free", radius, flush=True)
    n, s, d, samp = rmat_graph(11, 12, 77)
    E = set(zip(s.tolist(), d.tolist()))
    bs = rmat_batches(n, s, d, samp, [40, 60, 300, 50, 200, 30], 78)
    with Graph(n, s, d, delta=1, radius=radius) as g:
        # the first batches grow the buffers for the allocation-free ones
        for b in bs[:2]:
            local(g, n, E, b)
        grown = g.apply_batch_dev(*dev(bs[2]))
        oracle_apply(E, n, *bs[2])
        assert grown == native.static_counts(n, *pairs(E))
        for free, loc in ((bs[3], bs[4]), (bs[5], [x[::2] for x in (bs[4][2], bs[4][3], bs[4][0], bs[4][1])])):
            got, st = g.apply_batch_dev_noalloc(*dev(free), stats=True)
            assert st["delta"] == 0 and st["region_entries"] > 0
            oracle_apply(E, n, *free)
            assert got == native.static_counts(n, *pairs(E))
            local(g, n, E, loc)


def test_undone_batch():
    """0 and 401 joined to 1 .. 400; joining those to ten more vertices outgrows
    the hub cursors of the build, after the merge."""
    from paper_2308_14493_amd.graphlet4 import Graph, GraphletError
    print("case kept, undone", flush=True)
    n = 20412
    E = {(0, u) for u in range(1, 401)} | {(u, 401) for u in range(1, 401)} | {(0, 401)}
    E |= {(v, v + 1) for v in range(412, 20411)} | {(u, u + 1) for u in range(1, 400)}
    hub = (np.repeat(np.arange(1, 401, dtype=np.int32), 10), np.tile(np.arange(402, 412, dtype=np.int32), 400), Z, Z)
    rng = np.random.default_rng(5)
    with Graph(n, *pairs(E), delta=1) as g:
        before = g.counts()
        assert before == native.static_counts(n, *pairs(E))
        with pytest.raises(GraphletError) as e:
            g.apply_batch_dev_noalloc(*dev(hub))
        assert e.value.code == -2 and "undone" in str(e.value)
        assert g.counts() == before
        for _ in range(2):
            gone = rng.permutation(np.array(sorted(E)))[:30]
            add = rng.integers(0, 412, (2, 20)).astype(np.int32)
            local(g, n, E, (add[0], add[1], gone[:, 0].astype(np.int32), gone[:, 1].astype(np.int32)))
