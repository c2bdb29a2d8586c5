"""4-cliques counted a vertex at a time from the CSR (rows of at most 1024
entries): the sizes at its edges -- a wave's and a workgroup's longest row,
whole and partial words of the bit matrix, grids whose counters sit in LDS
and in device memory, members inside and outside the hub bit matrix."""
import math

import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen
from tests.test_gpu_cliques import check_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 4, 64, 65, 66, 128, 257, 258, 1024, 1025, 1026])
@pytest.mark.parametrize("p", [1, 3])
def test_complete_graph_rows(n, p):
    """K_n has one row of every length below n."""
    a, b = np.triu_indices(n, 1)
    with P.Graph(n, a.astype(np.int32), b.astype(np.int32)) as g:
        g.partition(p)
        assert g.four_cliques() == math.comb(n, 4)
        assert int(g.four_clique_lists()[1].sum()) == math.comb(n, 4)


@pytest.mark.parametrize("p", [2, 12, 13])
@pytest.mark.parametrize("kind", ["rmat", "rgg"])
def test_lists_across_hubs_and_grids(kind, p):
    """More than 16,384 vertices, so that pairs fall on both sides of the
    lowest hub rank; 12 and 13 stripes: counters in LDS and not."""
    if kind == "rmat":
        n, s, d = gen.rmat(16, 6, gen.seed(71, p))
    else:
        n, s, d = gen.rgg(33001, 26.0, gen.seed(71, p))
    got, _ = check_lists(n, s, d, p)
    assert got == oracle.four_cliques(n, s, d)
