"""The counting kernel's walk in 4-entry segments, at the sizes where it can
go wrong: lists of every length around a segment and around a batch, lists cut
to the entries above the staged list's vertex, packed items over stripes too
wide for a key's usual split."""
import math

import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 8, 9, 10, 33, 65, 131, 300])
@pytest.mark.parametrize("p", [1, 2, 5])
@pytest.mark.parametrize("kw", [{}, {"by_rows": True}, {"by_rows": False, "unroll": 8},
                                {"kernel": P.KERNEL_HASH}, {"kernel": P.KERNEL_SEARCH}])
def test_complete_graph(n, p, kw):
    """K_n has one row of every length below n."""
    a, b = np.triu_indices(n, 1)
    with P.Graph(n, a.astype(np.int32), b.astype(np.int32)) as g:
        g.partition(p)
        assert g.count(**kw) == math.comb(n, 3)


@pytest.mark.parametrize("width", [(1 << 26) - 1, 1 << 26, (1 << 28) + 3])
def test_wide_stripe(width):
    """Small cliques spread over a wide id range, ranks in id order so that
    the one stripe spans it: below 2^26 columns, at and above it."""
    rng = np.random.default_rng(width)
    s, d, want = [], [], 0
    for k in (3, 6, 12, 20, 40, 40, 64):
        ids = np.sort(rng.choice(width, k, replace=False)).astype(np.int32)
        a, b = np.triu_indices(k, 1)
        s.append(ids[a])
        d.append(ids[b])
        want += math.comb(k, 3)
    s, d = np.concatenate(s), np.concatenate(d)
    s, d = np.append(s, 0).astype(np.int32), np.append(d, width - 1).astype(np.int32)
    with P.Graph(width, s, d, order_by_id=True) as g:
        for rows in (True, False):
            assert g.partition(1).count(by_rows=rows) == want
    P.release_cached_memory()


@pytest.mark.parametrize("p", [1, 3, 16])
def test_short_lists(p):
    """Erdos-Renyi rows of a few entries: tiny and packed items."""
    n, s, d = gen.er(20011, 150000, gen.seed(72, p))
    with P.Graph(n, s, d) as g:
        g.partition(p)
        want = oracle.tc(n, s, d)
        assert g.count() == want
        assert g.count(by_rows=True) == want
        assert g.count(kernel=P.KERNEL_HASH) == want
