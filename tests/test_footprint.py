"""The admission estimate covers the parts of a handle by their own sizes (host
arithmetic), and what a handle that counts large batches edge-locally really
allocates (GPU)."""
import ctypes

import numpy as np
import pytest

from paper_2308_14493_amd import graphlet4


def estimate(n, s, d, delta):
    lib = graphlet4.load()
    opt = graphlet4._opts(None, None, 0, None, delta=delta)
    s, d = np.ascontiguousarray(s, np.int32), np.ascontiguousarray(d, np.int32)
    b = ctypes.c_int64()
    assert lib.gc_graph_footprint(n, s.ctypes.data, d.ctypes.data, s.size, ctypes.byref(opt), ctypes.byref(b)) == 0
    return b.value


@pytest.mark.parametrize("m", [1000, 1 << 18, 1 << 20])
def test_estimate_covers_the_parts(m):
    n = m + 1
    s = np.arange(m)
    rows = 2 * 4 * 4 * int(1.25 * 2 * m + 2 * n)       # entries and triangle counts, at least
    region = 40 * 3 * m                                # view of the union, scratch, versions
    hubs = 256 * 12 * n
    cap = min(1 << 18, 2 * m)
    lists = 68 * 64 * cap + 8 * 8 * cap + 12 * 12 * cap  # pairs, affected edges, their table
    compaction = rows
    region_only = rows + region + hubs + compaction
    assert estimate(n, s, s + 1, -1) >= region_only
    assert estimate(n, s, s + 1, 0) >= region_only + lists
    assert estimate(n, s, s + 1, 1) == estimate(n, s, s + 1, 0) > estimate(n, s, s + 1, -1)


@pytest.mark.gpu
def test_estimate_bounds_large_edge_local_batches():
    import torch
    print("case footprint edge-local", flush=True)
    n, m, k = 1 << 16, 1 << 20, 1 << 17
    rng = np.random.default_rng(11)
    u, v = rng.integers(n, size=(2, m + 2 * k))
    key = np.unique(np.minimum(u, v).astype(np.int64) * n + np.maximum(u, v))
    key = rng.permutation(key[key // n != key % n])
    e = lambda x: ((x // n).astype(np.int32), (x % n).astype(np.int32))  # noqa: E731
    old, new = key[:m], key[m:m + k]
    est = estimate(n, *e(old), 1)
    graphlet4.Graph(3, [0], [1], delta=1).close()  # the library's own memory (code, static staging)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    g = graphlet4.Graph(n, *e(old), delta=1)
    got, st = g.apply_batch(*e(new), *e(old[:k]), stats=True)
    assert st["delta"] == 1 and st["eff_ins"] == new.size and st["eff_del"] == k
    used = free - torch.cuda.mem_get_info()[0]
    print("  estimate %.1f MB, measured %.1f MB" % (est / 1e6, used / 1e6), flush=True)
    assert got == g.recount()
    g.close()
    assert 0 < used <= est
