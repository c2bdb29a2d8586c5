"""Components and PageRank at the sizes where their segmented walks and
queued iterations can go wrong: rows of every length around a segment and
around a wave's rows, long chains, iteration limits around a queued round."""
import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen
from tests.test_gpu_bsp import check_cc, check_pr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 5, 6, 31, 32, 33, 64, 65, 66, 129, 300])
@pytest.mark.parametrize("p", [1, 3])
def test_complete_graphs(n, p):
    """K_n (one row of every length below n), twice, and n isolated vertices."""
    a, b = np.triu_indices(n, 1)
    s = np.concatenate([a, a + n]).astype(np.int32)
    d = np.concatenate([b, b + n]).astype(np.int32)
    check_cc(3 * n, s, d, p)
    check_pr(3 * n, s, d, p)


@pytest.mark.parametrize("order", ["up", "down", "shuffled"])
def test_long_paths(order):
    """Paths of 100,003 vertices: chains as long as the graph."""
    n = 100003
    ids = np.arange(n, dtype=np.int32)
    if order == "down":
        ids = ids[::-1].copy()
    elif order == "shuffled":
        ids = np.random.default_rng(5).permutation(n).astype(np.int32)
    check_cc(n, ids[:-1], ids[1:], 4)


@pytest.mark.parametrize("max_iter", [0, 1, 3, 4, 5, 8, 9])
def test_pagerank_iteration_limits(max_iter):
    n, s, d = gen.rmat(11, 8, gen.seed(73, 0))
    check_pr(n, s, d, 3, max_iter=max_iter, tol=0.0)
    check_pr(n, s, d, 3, max_iter=max_iter, tol=1e-2)


def test_many_trees_meet():
    """A sparse random graph: many local maxima hooked in the last pass."""
    n, s, d = gen.er(200003, 260000, gen.seed(73, 1))
    check_cc(n, s, d, 5)
