"""GPU: the lists an edge-local pass grows to after finding them short."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

Z = np.zeros(0, np.int32)


def test_affected_edges_bounded_by_the_edges():
    """Deletions in a complete graph move t of its 1.1e6 edges 1.5e7 times.  The
    pairs (7.5e6, grown by a quarter, 68 bytes each) take 640 MB; a list and a
    table for every move would take 550 MB more, for every edge 35 MB."""
    import torch
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case affected edges bounded", flush=True)
    n, k = 1500, 5000
    s, d = (x.astype(np.int32) for x in np.triu_indices(n, 1))
    q = np.random.default_rng(3).permutation(s.size)[:k]
    with Graph(n, s, d, delta=1) as g:
        full = g.counts()
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        got, st = g.apply_batch(Z, Z, s[q], d[q], stats=True)
        assert st["delta"] == 1 and st["retries"] > 0
        assert free - torch.cuda.mem_get_info()[0] < (640 << 20) + (150 << 20)
        assert got == g.recount()
        assert g.apply_batch(s[q], d[q], Z, Z) == full
