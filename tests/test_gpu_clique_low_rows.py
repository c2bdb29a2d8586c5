"""4-cliques of rows over 64 entries whose members rank below the 32,768 highest
(the hubs of a graph with such rows): their pairs are searched, not read from the
hubs' bit matrix.  Cliques beside a bipartite graph of higher degrees, which has
no triangles, so the counts have a closed form, per 4-list too."""
import math
from collections import Counter

import numpy as np
import pytest

import paper_2209_04541_amd as P

pytestmark = pytest.mark.gpu

HUBS = 32768


def graph(ks, above):
    """Cliques of the given sizes (ascending), then `above` vertices of a
    bipartite graph whose degrees exceed the cliques'."""
    s, d, at = [], [], 0
    for k in ks:
        a, b = np.triu_indices(k, 1)
        s.append(at + a)
        d.append(at + b)
        at += k
    left = above // 2
    right, deg = above - left, max(ks) + 60
    i = np.arange(left)[:, None]
    t = np.arange(deg)[None, :]
    s.append((at + i + 0 * t).ravel())
    d.append((at + left + (i + t * 17) % right).ravel())
    return at + above, np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32)


def in_list(stripes, q):
    """4-subsets of members with the given stripes that lie in stripes q."""
    have = Counter(stripes)
    out = 1
    for st, times in Counter(q).items():
        out *= math.comb(have[st], times)
    return out


@pytest.mark.parametrize("ks,inside", [
    ((70, 200), -300),        # every member below the hubs
    ((257, 600), -40),        # rows of whole workgroups among them
    ((70, 200), 37), ((70, 200), 122), ((200,), 150),  # the last clique lies across
    ((300, 600), 251), ((600,), 5),
])
@pytest.mark.parametrize("p", [1, 3, 13])
def test_cliques_below_the_hubs(ks, inside, p):
    """inside: members of the last clique among the hubs (negative: as many
    vertices of the bipartite graph below them too)."""
    n, s, d = graph(ks, HUBS - inside)
    with P.Graph(n, s, d) as g:
        row_off, col, rank = g.export_csr()
        lo, rows = n - HUBS, np.diff(row_off)
        assert np.array_equal(np.sort(rank[: sum(ks)]), np.arange(sum(ks)))  # the cliques rank lowest
        long_low = [v for v in range(sum(ks)) if 64 < rows[v] <= 1024 and col[row_off[v]] < lo]
        assert long_low and (max(ks) < 300 or any(rows[v] > 256 for v in long_low))
        first_hub = [int(np.sum(col[row_off[v]:row_off[v + 1]] < lo)) for v in long_low]
        if 0 < inside < max(ks) - 1:  # rows that change form inside a run of 4 and of 16
            assert any(x % 4 and x % 16 and x < rows[v] for x, v in zip(first_hub, long_low))
        g.partition(p)
        want = sum(math.comb(k, 4) for k in ks)
        assert g.four_cliques() == want
        ijkl, counts = g.four_clique_lists()
        stripe = np.searchsorted(g.cuts(), np.arange(n), side="right") - 1
        at, groups = 0, []
        for k in ks:
            groups.append(stripe[rank[at:at + k]].tolist())
            at += k
        for q, c in zip(ijkl, counts):
            assert int(c) == sum(in_list(st, q.tolist()) for st in groups), q
        assert int(counts.sum()) == want
