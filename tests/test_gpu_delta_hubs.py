"""GPU: edge-local passes whose changed edges share an end with many other
changed edges, or with many neighbours below the bitmap's window: the members
that a bitmap leaves out are searched up to a number per edge (GC_DELTA_OUT
sets it) and walked in layers beyond, against the oracle on both sides of that
line; and the lists of such a pass do not grow as the square of its updates."""
import numpy as np
import pytest

from graphgen import rmat_graph
from oracle import native
from oracle.semantics import apply_batch as oracle_apply

pytestmark = pytest.mark.gpu

Z = np.zeros(0, np.int32)


def pairs(E):
    E = sorted(E)
    return np.array([u for u, _ in E], np.int32), np.array([v for _, v in E], np.int32)


def two_hubs(seed):
    """R-MAT of 2,048 vertices with two vertices joined to 700 others each, 600 of them common."""
    n, s, d, _ = rmat_graph(11, 20, seed)
    E = set(zip(s.tolist(), d.tolist()))
    rng = np.random.default_rng(seed)
    p = rng.permutation(n)
    h, k, common = int(p[0]), int(p[1]), [int(x) for x in p[2:602]]
    E = {e for e in E if not {h, k} & set(e)}
    key = lambda a, b: (min(a, b), max(a, b))  # noqa: E731
    for x in common:
        E |= {key(h, x), key(k, x)}
    E |= {key(h, int(x)) for x in p[602:702]} | {key(k, int(x)) for x in p[702:802]} | {key(h, k)}
    return n, E, h, k, common, key


# 127 .. 130 changed edges at one end: below, at and above 128 members left out
@pytest.mark.parametrize("changes,most", [(127, 128), (128, 128), (129, 128), (130, 128), (420, 128), (60, 1)])
@pytest.mark.parametrize("ids", [40, 1000, 0])
def test_layers_against_oracle(monkeypatch, ids, changes, most):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case layers", ids, changes, most, flush=True)
    monkeypatch.setenv("GC_DELTA_BITS", str(ids))
    monkeypatch.setenv("GC_DELTA_OUT", str(most))
    n, E, h, k, common, key = two_hubs(31)
    gone = {key(h, k)} | {key(h, x) for x in common[:changes - 1]}
    back = {key(k, x) for x in common[100:200]}  # both edges of some common neighbours
    with Graph(n, *pairs(E), delta=1) as g:
        for b in [(Z, Z) + pairs(gone), pairs(gone) + pairs(back), pairs(back) + pairs({key(h, k)}), pairs({key(h, k)}) + (Z, Z)]:
            got, st = g.apply_batch(*b, stats=True)
            assert st["delta"] == 1
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *pairs(E))


def test_layers_pool(monkeypatch):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case layers pool", flush=True)
    monkeypatch.setenv("GC_DELTA_BITS", "700")
    monkeypatch.setenv("GC_DELTA_OUT", "100")
    gs = [two_hubs(s) for s in (41, 42, 43)]
    Es = [set(q[1]) for q in gs]
    src, dst = zip(*[pairs(E) for E in Es])
    with Graph.pool([q[0] for q in gs], list(src), list(dst), delta=1) as g:
        gone = [{q[5](q[2], q[3])} | {q[5](q[2], x) for x in q[4][:150 + 60 * j]} for j, q in enumerate(gs)]
        for bs in ([(Z, Z) + pairs(x) for x in gone], [pairs(x) + (Z, Z) for x in gone]):
            got = g.apply_batches(bs)
            for j, b in enumerate(bs):
                oracle_apply(Es[j], gs[j][0], *b)
                assert got[j] == native.static_counts(gs[j][0], *pairs(Es[j]))


# lists of (16384 + 64) x 64 pairs take 72 MB and grow by half again; the
# pairs of every two changed edges of the hub would take more than 2 GB
@pytest.mark.parametrize("ids,updates", [(0, 10000), (4096, 100)])
@pytest.mark.parametrize("shared", [False, True])
def test_lists_do_not_square(monkeypatch, shared, ids, updates):
    import torch
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case lists do not square", shared, ids, updates, flush=True)
    monkeypatch.setenv("GC_DELTA_BITS", str(ids))
    n, leaves = 100002, 60000
    o = np.arange(2, 2 + leaves, dtype=np.int32)                  # leaves of vertex 0
    a = np.arange(2 + leaves // 2, 2 + leaves // 2 + leaves, dtype=np.int32)  # of vertex 1
    s = np.concatenate([np.zeros(leaves, np.int32), np.ones(leaves if shared else 0, np.int32)])
    d = np.concatenate([o, a]) if shared else o
    new = np.arange(2 + leaves, 2 + leaves + updates, dtype=np.int32)  # leaves of 1 that are none of 0
    hub = np.zeros(updates, np.int32)
    with Graph(n, s, d, delta=1) as g:
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        got, st = g.apply_batch(hub, new, Z, Z, stats=True)
        assert st["delta"] == 1
        assert free - torch.cuda.mem_get_info()[0] < (400 << 20 if updates > 1000 else 64 << 20)
        assert got == g.recount()
        before = g.apply_batch(Z, Z, hub, new)
        assert before == g.recount()
