"""GPU: the 4-cliques of the workgroup triangle tiers on dense graphs (checked
through the complement): no edge, few, many and too many edges with flags
among the slots of a vertex, out-degrees at the words of the slot masks and at
the tiers' edges, two and four versions, and wide words of the counts."""
import numpy as np
import pytest

from graphgen import erdos_renyi
from oracle import native

pytestmark = pytest.mark.gpu

COMP = [0, 6, 8, 7, 9, 10, 1, 3, 2, 4, 5]   # class of the complement


@pytest.mark.parametrize("n", [66, 127, 128, 129, 130, 194, 258, 300, 515])
@pytest.mark.parametrize("changes", [1, 12, 70, 400, 1500])
def test_flagged_edges_per_vertex(n, changes):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case tri", n, changes, flush=True)
    cs, cd = erdos_renyi(n, 0.04, n + changes)
    full = np.array([u * n + v for u in range(n) for v in range(u + 1, n)])
    k = np.setdiff1d(full, np.minimum(cs, cd).astype(np.int64) * n + np.maximum(cs, cd))
    rng = np.random.default_rng(n * changes)
    e = lambda x: ((x // n).astype(np.int32), (x % n).astype(np.int32))  # noqa: E731
    z = np.zeros(0, np.int32)

    def want(x):
        o = native.static_counts(n, *e(np.setdiff1d(full, x)))
        return [o[COMP[j]] for j in range(11)]

    gone = rng.choice(k, min(changes, k.size // 3), replace=False)
    k2, some = np.setdiff1d(k, gone), gone[::2]
    with Graph(n, *e(k), delta=-1, radius=0) as g:
        assert g.counts() == want(k)
        assert g.apply_batch(z, z, *e(gone)) == want(k2)
        assert g.apply_batch(*e(gone), z, z) == want(k)
        rows = g.apply_batch_seq([(z, z) + e(gone), e(some) + (z, z), (z, z) + e(some)])
        assert rows[0][:6] == want(k2)[:6] and rows[1][:6] == want(np.union1d(k2, some))[:6]
        assert rows[2][:6] == want(k2)[:6] and g.counts() == want(k2)
