"""GPU: the triangle tiers above 512 out-neighbours on dense graphs (checked
through the complement), words of the bit matrix on both sides of the density
from which their edges are not packed, one version and several; and the global
tier's hash on both sides of the out-degree up to which it lies in LDS."""
import numpy as np
import pytest

from graphgen import erdos_renyi
from oracle import native

pytestmark = pytest.mark.gpu

COMP = [0, 6, 8, 7, 9, 10, 1, 3, 2, 4, 5]   # class of the complement
Z = np.zeros(0, np.int32)


# complements of 4% (61 of 64 bits set), 25% (48) and 45% (35); 514 to 1,024, 1,025
# to 1,280 and more out-neighbours at the largest
@pytest.mark.parametrize("n,p", [(516, 0.04), (600, 0.25), (600, 0.45), (1030, 0.04), (1300, 0.03), (1420, 0.03)])
@pytest.mark.parametrize("changes", [3, 300, 4000])
def test_dense_tiers(n, p, changes):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case dense tiers", n, p, changes, flush=True)
    cs, cd = erdos_renyi(n, p, n + changes)
    full = np.array([u * n + v for u in range(n) for v in range(u + 1, n)])
    k = np.setdiff1d(full, np.minimum(cs, cd).astype(np.int64) * n + np.maximum(cs, cd))
    rng = np.random.default_rng(n * changes)
    e = lambda x: ((x // n).astype(np.int32), (x % n).astype(np.int32))  # noqa: E731

    def want(x):
        o = native.static_counts(n, *e(np.setdiff1d(full, x)))
        return [o[COMP[j]] for j in range(11)]

    gone = rng.choice(k, changes, replace=False)
    k2, some = np.setdiff1d(k, gone), gone[::2]
    with Graph(n, *e(k), delta=-1, radius=0) as g:
        before, after = want(k), want(k2)
        assert g.counts() == before
        assert g.apply_batch(Z, Z, *e(gone)) == after
        assert g.apply_batch(*e(gone), Z, Z) == before
        rows = g.apply_batch_seq([(Z, Z) + e(gone), e(some) + (Z, Z), (Z, Z) + e(some)])
        assert rows[0][:6] == after[:6] and rows[1][:6] == want(np.union1d(k2, some))[:6]
        assert rows[2][:6] == after[:6] and g.counts() == after


@pytest.mark.parametrize("k", [1281, 4095, 4096, 4097, 5000])
def test_global_tier_hash(k):
    """A vertex isolated at the build, and so of the lowest rank, gets k edges."""
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case global tier hash", k, flush=True)
    n = 6001
    s, d = erdos_renyi(n - 1, 0.002, k)
    s, d = s + 1, d + 1
    star = np.arange(1, k + 1, dtype=np.int32)
    with Graph(n, s, d, delta=-1) as g:
        got = g.apply_batch(np.zeros(k, np.int32), star, s[::50], d[::50])
        keep = np.ones(s.size, bool)
        keep[::50] = False
        assert got == native.static_counts(n, np.concatenate([s[keep], np.zeros(k, np.int32)]),
                                           np.concatenate([d[keep], star]))


@pytest.mark.parametrize("k", [4094, 4097, 4230])
def test_dense_rows_of_many_words(k):
    """Rows of the bit matrix of 64 words and of more: 150 vertices of the lowest
    ranks (no edges at the build) joined to all, but for one pair in 50."""
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case dense rows of many words", k, flush=True)
    n, rng = k + 1, np.random.default_rng(k)
    s, d = np.nonzero(np.triu(rng.random((150, n)) < 0.98, 1))
    s, d = s.astype(np.int32), d.astype(np.int32)
    q = rng.permutation(s.size)[:3]
    some = np.isin(np.arange(s.size), q)
    with Graph(n, Z, Z, delta=-1, radius=0) as g:
        assert g.apply_batch(s, d, Z, Z) == native.static_counts(n, s, d)
        assert g.apply_batch(Z, Z, s[some], d[some]) == native.static_counts(n, s[~some], d[~some])
