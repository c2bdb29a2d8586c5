"""Triangles at the vertices of graphs with hubs: degrees at and around the parts
that a long vertex is cut into, long rows and long columns."""
import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu


def check(n, s, d, order_by_id):
    with P.Graph(n, s, d, order_by_id=order_by_id) as g:
        row_off, col, rank = g.export_csr()
        sup = oracle.edge_support(n, row_off, col)
        by_rank = np.zeros(n, np.uint64)
        np.add.at(by_rank, np.repeat(np.arange(n), np.diff(row_off)), sup)
        np.add.at(by_rank, col, sup)
        per, total = g.vertex_counts()
        assert total == oracle.tc(n, s, d)
        assert np.array_equal(per, (by_rank // 2)[rank])


@pytest.mark.parametrize("order_by_id", [False, True])
@pytest.mark.parametrize("degrees", [[1023], [1024], [1025], [2048, 2049], [1025] * 9, [5000, 1, 1100, 4097, 700]])
def test_hub_degrees(degrees, order_by_id):
    """Hubs of the given degrees over a cycle (a triangle for each two of their
    neighbours that follow each other), the hubs first: under the id order their
    edges are rows, under the degree order columns."""
    n, h = 6000, len(degrees)
    s, d = [h + np.arange(n)], [h + (np.arange(n) + 1) % n]
    for i, k in enumerate(degrees):
        s.append(np.full(k, i))
        d.append(h + (37 * i + np.arange(k)) % n)
    check(h + n, np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32), order_by_id)


@pytest.mark.parametrize("order_by_id", [False, True])
def test_rmat(order_by_id):
    check(*gen.rmat(15, 16, gen.seed(71, 5)), order_by_id)
