"""Edge support, vertex counts and the k-truss at the sizes of the support
kernel's staging: rows with entries on both sides of the lowest hub rank (8,192
from the top), rows at and above the LDS region's limits, and peeling rounds
of few and many edges."""
import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu


def check_all(n, s, d, ks=()):
    _, _, rank, row_off, col = oracle.oriented_csr(n, s, d)
    want = oracle.edge_support(n, row_off, col)
    with P.Graph(n, s, d) as g:
        got, tri = g.edge_support()
        assert np.array_equal(got, want)
        assert tri == int(want.sum()) // 3
        per, _ = g.vertex_counts()
        by_rank = np.zeros(n, np.uint64)
        np.add.at(by_rank, np.repeat(np.arange(n), np.diff(row_off)), want)
        np.add.at(by_rank, col, want)
        assert np.array_equal(per, (by_rank // 2)[rank])
        for k in ks:
            keep, left, _ = g.ktruss(k)
            ref = oracle.ktruss(n, row_off, col, k)
            ref = ref[0] if isinstance(ref, tuple) else ref
            assert np.array_equal(keep.astype(bool), np.asarray(ref).astype(bool))
            assert left == int(keep.sum())


@pytest.mark.parametrize("kind", ["rmat", "er", "rgg"])
def test_rows_across_the_lowest_hub(kind):
    if kind == "rmat":
        n, s, d = gen.rmat(15, 12, gen.seed(74, 0))
    elif kind == "er":
        n, s, d = gen.er(12001, 300000, gen.seed(74, 1))
    else:
        n, s, d = gen.rgg(20011, 40.0, gen.seed(74, 2))
    check_all(n, s, d, ks=(3, 5, 8))


@pytest.mark.parametrize("k", [63, 64, 65, 1024, 1025, 1026])
def test_long_rows(k):
    """K_k and a sparse rest: rows of up to k - 1 entries, all of them hubs;
    above 1,024 entries a row is searched in device memory."""
    a, b = np.triu_indices(k, 1)
    n, s, d = gen.er(9001, 20000, gen.seed(74, k))
    check_all(n, np.concatenate([s, a]).astype(np.int32), np.concatenate([d, b]).astype(np.int32))


@pytest.mark.parametrize("low", [341, 342, 600])
def test_rows_below_the_hubs(low):
    """K_low whose vertices rank below 8,192 others (a regular graph of a
    higher degree): rows of up to low - 1 entries below the hubs, at the
    limit of their table and above it."""
    a, b = np.triu_indices(low, 1)
    n, deg = 8300, low + 40
    ring = np.arange(n)
    s = np.concatenate([a] + [low + ring for j in range(1, deg // 2 + 1)])
    d = np.concatenate([b] + [low + (ring + j) % n for j in range(1, deg // 2 + 1)])
    check_all(low + n, s.astype(np.int32), d.astype(np.int32))
