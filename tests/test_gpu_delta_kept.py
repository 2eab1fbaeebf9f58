"""GPU: the triangle counts kept per edge and per vertex across passes, and
the edge-local 4-cliques' split between members walked against a bitmap and
pairs searched, against the oracle after every batch.

Region passes (the allocation-free entry point), edge-local passes and
multi-version sequences take turns on one graph whose rows move at every
growth (no slack), with one batch undone in between; cliques whose common
neighbours hold just below and just above the 4,096 row entries from which
they are walked, whole and with the window shrunk below them."""
import numpy as np
import pytest

from graphgen import raw_noise_batch, rmat_batches, rmat_graph
from oracle import native
from oracle.semantics import apply_batch as oracle_apply

pytestmark = pytest.mark.gpu


def esorted(E):
    E = sorted(E)
    return (np.array([u for u, v in E], np.int32), np.array([v for u, v in E], np.int32))


@pytest.mark.parametrize("slack", [0.0, 0.25])
def test_kept_counts_through_all_passes(slack):
    import torch
    from paper_2308_14493_amd.graphlet4 import Graph, GraphletError
    print("case kept counts slack", slack, flush=True)
    n, s, d, samp = rmat_graph(11, 12, 71)
    E = set(zip(s.tolist(), d.tolist()))
    dev = lambda b: [torch.tensor(np.asarray(x, np.int32), device="cuda") for x in b]  # noqa: E731
    batches = rmat_batches(n, s, d, samp, [60, 200, 40, 300, 150, 90, 120, 80, 500, 64, 32, 16], 72)
    with Graph(n, s, d, delta=1, slack=slack) as g:
        for j in range(0, 12, 4):
            # refused or undone: either way the graph stays as it is
            try:
                g.apply_batch_dev_noalloc(*dev(batches[j]))
            except GraphletError:
                g.apply_batch(*batches[j])
            oracle_apply(E, n, *batches[j])
            assert g.counts() == native.static_counts(n, *esorted(E))
            got, st = g.apply_batch(*batches[j + 1], stats=True)
            assert st["delta"] == 1
            oracle_apply(E, n, *batches[j + 1])
            assert got == native.static_counts(n, *esorted(E))
            b = raw_noise_batch(n, *esorted(E), 60, 80 + j)
            got = g.apply_batch(*b)
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *esorted(E))
            g.apply_batch_seq(batches[j + 2:j + 4])
            for q in (2, 3):
                oracle_apply(E, n, *batches[j + q])
            assert g.counts() == native.static_counts(n, *esorted(E))


def test_kept_counts_after_undo():
    """A batch whose counting outgrows the scratch is undone; the edge-local
    passes around it use the kept counts."""
    import torch
    from paper_2308_14493_amd.graphlet4 import Graph, GraphletError
    print("case kept counts undo", flush=True)
    n = 4000
    E = {(w, w + 1) for w in range(0, n - 1)} | {(w, w + 2) for w in range(0, n - 2)}
    hub = ([0] * 3500, list(range(400, 3900)), [], [])
    with Graph(n, *esorted(E), delta=1) as g:
        dev = [torch.tensor(np.asarray(x, np.int32), device="cuda") for x in hub]
        try:
            g.apply_batch_dev_noalloc(*dev)
            oracle_apply(E, n, *[np.array(x, np.int32) for x in hub])
        except GraphletError:
            pass
        for b in (([0, 5], [7, 9], [1, 400], [2, 401]), ([0, 3], [2000, 3000], [5], [9])):
            b = [np.array(x, np.int32) for x in b]
            got = g.apply_batch(*b)
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *esorted(E))


@pytest.mark.parametrize("ids", [8, 40, 0])
@pytest.mark.parametrize("k", [64, 65, 66, 90])
def test_k4_split_boundary(monkeypatch, k, ids):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case k4 split", k, ids, flush=True)
    monkeypatch.setenv("GC_DELTA_BITS", str(ids))
    n = k + 30
    E = {(u, v) for u in range(k) for v in range(u + 1, k)} | {(u, u + k) for u in range(30)}
    with Graph(n, *esorted(E), delta=1) as g:
        for b in (([], [], [0], [1]), ([0], [1], [], []), ([k, k + 1], [3, 4], [0, 0, 2], [2, 3, 9]),
                  ([0, 2], [2, 9], list(range(10, 20)), list(range(20, 30)))):
            b = [np.array(x, np.int32) for x in b]
            got = g.apply_batch(*b)
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *esorted(E))
