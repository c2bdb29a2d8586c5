"""Staged lists that are searched in place: asked for, or too long for the LDS
table (over 2,730 entries), between items that stage bitmaps and tables in the
same region."""
import math

import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu


def clique(k, at=0):
    a, b = np.triu_indices(k, 1)
    return at + a, at + b


@pytest.mark.parametrize("by_rows", [True, False])
@pytest.mark.parametrize("kernel", [P.KERNEL_AUTO, P.KERNEL_HASH, P.KERNEL_BITMAP, P.KERNEL_SEARCH])
def test_long_rows_between_bitmaps(kernel, by_rows):
    """K_2800 in a stripe too wide for a bitmap (rows over 2,730 entries are
    searched), a random graph in the same stripe and in a narrow one."""
    k, wide, n = 2800, 150000, 156000
    rng = np.random.default_rng(5)
    a, b = clique(k)
    rs, rd = rng.integers(k, n, 300000), rng.integers(k, n, 300000)
    ns, nd = rng.integers(wide, n, 200000), rng.integers(wide, n, 200000)
    rest = (np.concatenate([rs, ns]).astype(np.int32), np.concatenate([rd, nd]).astype(np.int32))
    want = math.comb(k, 3) + oracle.tc(n, *rest)
    s, d = np.concatenate([a, rest[0]]).astype(np.int32), np.concatenate([b, rest[1]]).astype(np.int32)
    with P.Graph(n, s, d, order_by_id=True) as g:
        g.partition(2, cuts=np.array([0, wide, n], np.int32))
        for waves in (0, 2, 8):
            assert g.count(kernel=kernel, by_rows=by_rows, waves_per_block=waves) == want
            counts = {tuple(q): int(c) for q, c in zip(*g.task_counts())}
            assert sum(counts.values()) == want and counts[(0, 0, 0)] >= math.comb(k, 3)
        if kernel != P.KERNEL_BITMAP:
            return
        first = counts
        assert g.count(kernel=P.KERNEL_SEARCH, by_rows=by_rows) == want
        assert {tuple(q): int(c) for q, c in zip(*g.task_counts())} == first


@pytest.mark.parametrize("unroll", [1, 8])
@pytest.mark.parametrize("p", [1, 3])
@pytest.mark.parametrize("k", [2, 3, 5, 64, 65, 257, 700])
def test_searched_cliques(k, p, unroll):
    """Staged lists of every length below k, all of whose entries match."""
    a, b = clique(k)
    with P.Graph(k + 3, a.astype(np.int32), b.astype(np.int32)) as g:
        g.partition(p)
        for by_rows in (True, False):
            assert g.count(kernel=P.KERNEL_SEARCH, by_rows=by_rows, unroll=unroll) == math.comb(k, 3)


@pytest.mark.parametrize("p", [1, 4])
def test_searched_rmat(p):
    n, s, d = gen.rmat(13, 16, gen.seed(72, p))
    want = oracle.tc(n, s, d)
    with P.Graph(n, s, d) as g:
        g.partition(p)
        for by_rows in (True, False):
            for unroll in (0, 8):
                assert g.count(kernel=P.KERNEL_SEARCH, by_rows=by_rows, unroll=unroll) == want
