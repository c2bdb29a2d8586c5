"""k-trusses whose peeling rounds bring many edges below at once: a wave's buffer
for the next frontier fills up several times in a round, or stays almost empty."""
import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu


def check(n, s, d, ks):
    _, _, _, row_off, col = oracle.oriented_csr(n, s, d)
    with P.Graph(n, s, d) as g:
        for k in ks:
            keep, left, rounds = g.ktruss(k)
            want = oracle.ktruss(n, row_off, col, k)
            print("k-truss", n, k, left, rounds, flush=True)
            assert np.array_equal(keep, want)
            assert left == int(keep.sum())


@pytest.mark.parametrize("k,copies", [(12, 1), (40, 1), (40, 200), (130, 30)])
def test_cliques_short_of_an_edge(k, copies):
    """K_k less one edge, many times: the k-truss is empty, and the first round
    brings every other edge of each below."""
    a, b = np.triu_indices(k, 1)
    a, b = a[1:], b[1:]
    s = np.concatenate([a + c * k for c in range(copies)])
    d = np.concatenate([b + c * k for c in range(copies)])
    check(k * copies, s.astype(np.int32), d.astype(np.int32), (k - 1, k))


@pytest.mark.parametrize("kind", ["rmat", "rgg"])
def test_large_frontiers(kind):
    n, s, d = gen.rmat(15, 16, gen.seed(71, 6)) if kind == "rmat" else gen.rgg(30001, 30.0, gen.seed(71, 7))
    check(n, s, d, (6, 10, 14))
