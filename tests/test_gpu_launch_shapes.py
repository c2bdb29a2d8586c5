"""Persistent launches at the edges of their work dealing: fewer units than
waves, fewer workgroups than queues, units beyond the first ones of each wave,
counts gathered per workgroup (up to 128 tasks) or added to their slots, and a
launch split by staged-list length."""
import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P

pytestmark = pytest.mark.gpu


def hubs(n, m, nhub, seed):
    """m random pairs plus nhub vertices joined to a third of all and to each other."""
    rng = np.random.default_rng(seed)
    s, d = [rng.integers(0, n, m)], [rng.integers(0, n, m)]
    for h in range(nhub):
        t = rng.choice(n, n // 3, replace=False)
        s.append(np.full(len(t), h)), d.append(t)
    a, b = np.triu_indices(nhub, 1)
    return np.concatenate(s + [a]).astype(np.int32), np.concatenate(d + [b]).astype(np.int32)


CASES = [(40, 120, 2), (3000, 20000, 0), (6000, 50000, 6), (20000, 400000, 30)]


@pytest.mark.parametrize("n,m,nhub", CASES)
@pytest.mark.parametrize("p", [1, 3, 8, 9])  # 1, 10, 120 and 165 tasks
def test_counts_by_grab(n, m, nhub, p):
    s, d = hubs(n, m, nhub, n + p)
    want = oracle.tc(n, s, d)
    with P.Graph(n, s, d) as g:
        g.partition(p)
        assert g.count() == want
        ijk, first = g.task_counts()
        assert int(first.sum()) == want
        for rows in (True, False):
            for grab in (0, 1, 64):
                assert g.count(by_rows=rows, rows_per_grab=grab) == want
                got_ijk, got = g.task_counts()
                assert np.array_equal(got_ijk, ijk) and np.array_equal(got, first)


@pytest.mark.parametrize("graphs", [1, 3, 40, 300])
def test_batches(graphs):
    """Launches of fewer and of more workgroups than ranges of rows; waves that
    pass several graphs between additions."""
    sizes = [8 + (37 * i) % 90 for i in range(graphs)]
    gl = [(n, *hubs(n, 6 * n, 3, i)) for i, n in enumerate(sizes)]
    want = [oracle.tc(*g) for g in gl]
    with P.Batch(gl) as b:
        for grab in (0, 1, 64):
            assert [int(x) for x in b.count(per_graph=True, rows_per_grab=grab)] == want


@pytest.mark.parametrize("n,m,nhub", CASES)
def test_other_persistent_launches(n, m, nhub):
    s, d = hubs(n, m, nhub, n)
    with P.Graph(n, s, d) as g:
        g.partition(2)
        row_off, col, _ = g.export_csr()
        support, total = g.edge_support()
        assert total == oracle.tc(n, s, d) and np.array_equal(support, oracle.edge_support(n, row_off, col))
        assert g.four_cliques() == oracle.four_cliques(n, s, d)
        label, nc, _ = g.components()
        want, wnc = oracle.components(n, s, d)
        assert nc == wnc and np.array_equal(label, want)
