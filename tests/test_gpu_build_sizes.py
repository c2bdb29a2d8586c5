"""Build and partition at the sizes where their passes change form: dedupe and
scan tiles, sorts of few and many tiles, the high ends counted or sorted, one
block partitioned from the build's statistics, rows around the long-row
bound."""
import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P

pytestmark = pytest.mark.gpu


def pairs(n, m, seed):
    """m pairs over n ids, skewed to low ids, with repeats, loops and reversed
    pairs among them."""
    rng = np.random.default_rng(seed)
    s = (n * rng.random(m) ** 2).astype(np.int32)
    d = rng.integers(0, n, m).astype(np.int32)
    if m > 8:
        s[m // 2:m // 2 + 3], d[m // 2:m // 2 + 3] = d[:3].copy(), s[:3].copy()
        s[-1], d[-1] = 1, 1
    return s, d


def check(n, s, d, ps, order_by_id=False):
    keys = oracle.clean(n, s, d)
    with P.Graph(n, s, d, order_by_id=order_by_id) as g:
        row_off, col, rank = g.export_csr()
        assert len(col) == len(keys)
        if order_by_id:
            assert np.array_equal(rank, np.arange(n))
            lo, hi = (keys >> np.uint64(32)).astype(np.int64), (keys & np.uint64(0xFFFFFFFF)).astype(np.int64)
            assert np.array_equal(row_off, np.concatenate([[0], np.cumsum(np.bincount(lo, minlength=n))]))
            assert np.array_equal(col, hi)
        else:
            _, _, rk, ro, cl = oracle.oriented_csr(n, s, d)
            assert np.array_equal(rank, rk) and np.array_equal(row_off, ro) and np.array_equal(col, cl)
        want = oracle.tc(n, s, d)
        for p in ps:
            g.partition(p)
            assert g.count(by_rows=True) == want
            assert g.count(by_rows=False) == want
            outs, ins = np.diff(row_off), np.bincount(col, minlength=n)
            inf = g.info()
            assert inf["m"] == len(col) and inf["max_out_degree"] == outs.max(initial=0)
            assert inf["isolated"] == int(np.sum((outs == 0) & (ins == 0)))
            if p == 1:
                assert inf["probe_work_col"] == int(np.sum(outs.astype(np.int64) ** 2))
                assert inf["row_items"] == int(np.sum((outs + 31) // 32))
                assert inf["col_items"] == int(np.sum((ins + 31) // 32))
            label, nc, _ = g.components()
            want_label, want_nc = oracle.components(n, s, d)
            assert nc == want_nc and np.array_equal(label, want_label)
        ranks, it, _ = g.pagerank()  # reads rows and columns of the last partition
        want_ranks, want_it, _ = oracle.pagerank(n, s, d)
        assert it == want_it
        np.testing.assert_allclose(ranks, want_ranks, rtol=1e-10, atol=1e-15)


@pytest.mark.parametrize("m", [1, 2, 255, 1024, 1025, 2047, 2048, 2049, 4097, 32768, 65535, 65536, 65537, 262144,
                               262145])
def test_pair_counts(m):
    n = max(4, m // 5)
    check(n, *pairs(n, m, m), ps=(1, 3))


@pytest.mark.parametrize("n", [2, 255, 256, 257, 65536, 65537, 70001])
@pytest.mark.parametrize("order_by_id", [False, True])
def test_vertex_counts(n, order_by_id):
    """Widths of the packed ids, isolated vertices before and between."""
    m = min(20000, 4 * n)
    s, d = pairs(n, m, 7 * n)
    keep = (s % 3 != 1) & (d % 3 != 1)
    check(n, s[keep], d[keep], ps=(1, 2), order_by_id=order_by_id)


@pytest.mark.parametrize("d", [63, 64, 65, 66, 2049])
def test_rows_around_the_long_bound(d):
    """Stars whose rows or columns have d entries, by degree and by id, beside
    a small clique."""
    a, b = np.triu_indices(12, 1)
    s = np.concatenate([np.zeros(d, np.int64), np.full(d, 3000), a + 4000]).astype(np.int32)
    t = np.concatenate([np.arange(1, d + 1), 5000 + np.arange(d), b + 4000]).astype(np.int32)
    for by_id in (False, True):
        check(9000, s, t, ps=(1, 4), order_by_id=by_id)


def test_endpoint_out_of_range_on_the_device():
    import torch
    s = torch.tensor([0, 1, 2], dtype=torch.int32, device="cuda")
    for bad in (-1, 5):
        d = torch.tensor([1, bad, 0], dtype=torch.int32, device="cuda")
        with pytest.raises(P.PgabbError) as e:
            P.Graph(5, s, d)
        assert e.value.status == P.EINVAL


def spread(kind):
    rng = np.random.default_rng(len(kind))
    if kind == "stretch":  # 2 dense groups, some 50,000 empty rows between them
        a, b = np.triu_indices(50, 1)
        return 60000, np.concatenate([a, a + 50000]), np.concatenate([b, b + 50000])
    if kind == "many":  # tiles of more rows than are marked: entries far apart
        a = np.sort(rng.choice(300000, 3000, replace=False))
        return 300100, np.concatenate([a, [3, 3, 7]]), np.concatenate([a + 1 + rng.integers(0, 90, 3000), [7, 9, 9]])
    if kind == "star":  # one row over several tiles, runs that begin in earlier ones
        t = rng.choice(np.arange(2, 30000), 9000, replace=False)
        return 30000, np.concatenate([np.full(9000, 1), t[:4000]]), np.concatenate([t, t[1:4001]])
    return 5000, rng.integers(0, 5000, 2048 * 6), rng.integers(0, 5000, 2048 * 6)


@pytest.mark.parametrize("kind", ["stretch", "many", "star", "plain"])
@pytest.mark.parametrize("order_by_id", [False, True])
@pytest.mark.parametrize("p", [1, 2, 7, 64])
def test_blocks_of_odd_rows(kind, order_by_id, p):
    """Every triple of stripes counted by rows and by columns, with equal and
    with nnz cuts."""
    n, s, d = spread(kind)
    s, d = s.astype(np.int32), d.astype(np.int32)
    with P.Graph(n, s, d, order_by_id=order_by_id) as g:
        row_off, col, _ = g.export_csr()
        for mode in (P.CUT_NNZ, P.CUT_UNIFORM):
            g.partition(p, cut_mode=mode)
            B = oracle.block_counts(n, row_off, col, g.cuts())
            for rows in (True, False):
                assert g.count(by_rows=rows) == int(B.sum())
                for (i, j, k), c in zip(*g.task_counts()):
                    assert c == B[i, j, k]
            want = oracle.probe_work_col(n, row_off, col, g.cuts())
            assert g.info()["probe_work_col"] == want


@pytest.mark.parametrize("pairs", [[(0, 0)], [(0, 0), (0, 0)], [(0, 1)], [(1, 0), (0, 1), (1, 1)], [(2, 1), (1, 0)]])
def test_fewest_pairs(pairs):
    """Sorts of one key (made, not sorted), of none left after the loops, and
    of one vertex."""
    s, d = np.array(pairs, np.int32).T.copy()
    check(int(max(s.max(), d.max())) + 1, s, d, ps=(1, 2))


@pytest.mark.parametrize("n", [2, 900, 8191, 8192, 8193, 300000])
def test_high_ends(n):
    """Counts of the high ends above 65,536 pairs: one value of the high bits,
    several in a tile, one over many tiles (a third of the pairs end at the
    last vertex)."""
    m = 90001
    s, d = pairs(n, m, n)
    d[:m // 3] = n - 1
    check(n, s, d, ps=(1,))
