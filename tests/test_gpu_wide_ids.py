"""Builds whose ids are wide and sparse: more than 65,536 pairs, so the high ends
are sorted, with few of them per value of their high bits, and sizes on both
sides of where they are counted by their low bits."""
import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(1 << 18, 65537), (1 << 18, 800000), (1 << 18, 830000), (1 << 22, 70000),
                                 ((1 << 22) + 3, 1000000), (1 << 24, 70000)])
@pytest.mark.parametrize("kind", ["uniform", "hub"])
def test_degrees_of_wide_ids(n, m, kind):
    """Degrees order the ranks, and the CSR follows from them.  hub: a third of
    the pairs end in the last id."""
    rng = np.random.default_rng(n + m)
    s, d = rng.integers(0, n, m, dtype=np.int32), rng.integers(0, n, m, dtype=np.int32)
    if kind == "hub":
        d[: m // 3] = n - 1
    _, _, rank, row_off, col = oracle.oriented_csr(n, s, d)
    with P.Graph(n, s, d) as g:
        got_off, got_col, got_rank = g.export_csr()
        assert np.array_equal(got_rank, rank) and np.array_equal(got_off, row_off) and np.array_equal(got_col, col)
        assert g.count() == oracle.tc(n, s, d)
