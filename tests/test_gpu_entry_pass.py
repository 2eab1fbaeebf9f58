"""GPU: the entry pass and the per-vertex pass of a region count, against the
oracle: rows of 63 to 129 entries (sums of one row that end at, before and
after the 64 entries a wave takes), edges of the batch at both ends of rows,
vertex counts around the 256 a workgroup takes, two and four versions, the
whole graph and a region whose outermost rows are cut."""
import numpy as np
import pytest

from oracle import native
from oracle.semantics import apply_batch as oracle_apply

pytestmark = pytest.mark.gpu

Z = np.zeros(0, np.int32)


def pairs(E):
    E = sorted(E)
    return np.array([u for u, _ in E], np.int32), np.array([v for _, v in E], np.int32)


def circulant(n, r):
    """Every vertex has r neighbours: the r // 2 nearest on either side, and the opposite one."""
    E = {tuple(sorted((v, (v + k) % n))) for v in range(n) for k in range(1, r // 2 + 1)}
    return E | ({(v, v + n // 2) for v in range(n // 2)} if r % 2 else set())


@pytest.mark.parametrize("radius", [0, 2])
@pytest.mark.parametrize("n,r", [(254, 63), (256, 64), (257, 64), (258, 65), (255, 126), (512, 127), (513, 128), (514, 129)])
def test_rows_around_the_wave(n, r, radius):
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case entry pass", n, r, radius, flush=True)
    E = circulant(n, r)
    rows = {v: sorted({b if a == v else a for a, b in E if v in (a, b)}) for v in range(0, n, 7)}
    assert {len(x) for x in rows.values()} == {r}
    # the first and the last edge of every seventh row, and whole rows
    ends = {tuple(sorted((v, x[k]))) for v, x in rows.items() for k in (0, -1)}
    row = {tuple(sorted((7, x))) for x in rows[7]}
    some = set(sorted(ends)[::3])
    with Graph(n, *pairs(E), delta=-1, radius=radius) as g:
        assert g.counts() == native.static_counts(n, *pairs(E))
        for b in [(Z, Z) + pairs(ends), pairs(ends) + pairs(row - ends), pairs(row - ends) + (Z, Z)]:
            got, st = g.apply_batch(*b, stats=True)
            assert st["delta"] == 0
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *pairs(E))
        bs = [(Z, Z) + pairs(ends), pairs(some) + pairs(row - ends), pairs(row - ends) + (Z, Z)]
        got = g.apply_batch_seq(bs)
        for b, c in zip(bs, got):
            oracle_apply(E, n, *b)
            assert c == native.static_counts(n, *pairs(E))


@pytest.mark.parametrize("radius", [0, 2])
@pytest.mark.parametrize("tail", [191, 192, 193, 1000])
def test_region_inside_a_path(tail, radius):
    """Rows of one or two entries: a batch around one place of a path, whose
    region of radius 2 is a small part with cut outermost rows."""
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case region in a path", tail, radius, flush=True)
    n = 64 + tail
    E = {(v, v + 1) for v in range(n - 1)}
    with Graph(n, *pairs(E), delta=-1, radius=radius, autotune=0) as g:
        for b in [(np.array([10], np.int32), np.array([12], np.int32), np.array([30], np.int32), np.array([31], np.int32)),
                  (np.array([30], np.int32), np.array([32], np.int32), np.array([10], np.int32), np.array([12], np.int32))]:
            got = g.apply_batch(*b)
            oracle_apply(E, n, *b)
            assert got == native.static_counts(n, *pairs(E))


def test_region_view_filled_to_its_last_entry():
    """A region view of 11,034 entries (2 mod 4) at a capacity of as many, every
    hub in the windows: the rows are read 16 bytes at a time up to the end."""
    from paper_2308_14493_amd.graphlet4 import Graph
    print("case region view full", flush=True)
    n = 4004
    E = {(v, v + 1) for v in range(n - 1)} | {(0, n - 1)}
    ins = {(2 * i, 2 * i + 5) for i in range(1, 1514)}  # 8,008 + 2 x 1,513 entries
    assert not ins & E and len(ins) == 1513
    with Graph(n, *pairs(E), delta=-1, radius=0, tiers=(64, 1, 1)) as g:
        got, st = g.apply_batch(*(pairs(ins) + (Z, Z)), stats=True)
        assert st["region_entries"] == 2 * n + n // 2 + 1024 and st["tier_c4_large"] > 0
        assert got == native.static_counts(n, *pairs(E | ins))
