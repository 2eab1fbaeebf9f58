"""GPU: sizes on both sides of the sorts' and scans' changes of path (one
workgroup's scan up to 32,768 entries; tile histograms summed by the scatter
up to 393,216 keys), through graphs and batches of those sizes, against the
oracle."""
import numpy as np
import pytest

from oracle import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [393216, 393217])
@pytest.mark.parametrize("half", [8192, 8193])
@pytest.mark.parametrize("delta", [-1, 1])
def test_sort_scan_sizes(n, half, delta):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case sort/scan", n, half, delta, flush=True)
    rng = np.random.default_rng(half + n)
    u = np.concatenate([np.arange(n), rng.integers(0, n, n // 4), rng.integers(0, 40, n // 8)])
    v = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, n // 4), rng.integers(40, n, n // 8)])
    k = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
    k = k[k // n != k % n]
    dele = rng.choice(k, half, replace=False)
    new = np.setdiff1d(np.unique(rng.integers(0, n - 1, 4 * half) * n + n - 1 - rng.integers(0, 3, 4 * half)), k)
    new = rng.permutation(new[new // n < new % n])[:half]
    after = np.union1d(np.setdiff1d(k, dele), new)
    e = lambda x: ((x // n).astype(np.int32), (x % n).astype(np.int32))  # noqa: E731
    with Graph(n, *e(k), delta=delta) as g:
        assert g.counts() == native.static_counts(n, *e(k))
        assert g.apply_batch(*e(new), *e(dele)) == native.static_counts(n, *e(after))
        assert g.apply_batch(*e(dele), *e(new)) == native.static_counts(n, *e(k))
