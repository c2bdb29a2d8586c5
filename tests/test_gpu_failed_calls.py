"""Calls that run out of memory part way (an allocator hook that refuses):
the error is reported and what the graph holds afterwards is whole."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu

ALLOC = ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_void_p)
FREE = ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p)


class RefusingHook:
    """Device memory from torch, except for the requests that refuse(number,
    bytes) names."""

    def __init__(self, refuse):
        import torch
        self.calls = self.refused = 0
        live = {}

        def alloc(nbytes, stream, ctx):
            self.calls += 1
            if refuse(self.calls, int(nbytes)):
                self.refused += 1
                return None
            t = torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")
            live[t.data_ptr()] = t
            return t.data_ptr()

        def free(ptr, stream, ctx):
            torch.cuda.synchronize()
            live.pop(ptr, None)

        self._a, self._f = ALLOC(alloc), FREE(free)

    def __enter__(self):
        assert P.lib().pgabb_set_allocator(ctypes.cast(self._a, ctypes.c_void_p),
                                           ctypes.cast(self._f, ctypes.c_void_p), None) == P.OK
        return self

    def __exit__(self, *exc):
        assert P.lib().pgabb_set_allocator(None, None, None) == P.OK


@pytest.mark.parametrize("before", [0, 2])
@pytest.mark.parametrize("p", [1, 3])
def test_partition_that_runs_out_of_memory(p, before):
    """Whichever allocation of a partition fails, the graph is unpartitioned
    afterwards (or keeps its previous partition) and the next calls partition it
    themselves."""
    n, s, d = gen.rmat(11, 16, gen.seed(97, 6))
    want = oracle.tc(n, s, d)
    with P.Graph(n, s, d) as g:
        with RefusingHook(lambda k, b: False) as hook:
            g.partition(p)
        total = hook.calls
        assert total > 4
        ranks, _, _ = g.pagerank(max_iter=2)
        for k in range(1, total + 1):
            g.partition(before or 5)
            kept = g.info()["p"]
            with RefusingHook(lambda c, b: c == k):
                with pytest.raises(P.PgabbError) as e:
                    g.partition(p)
                assert e.value.status == P.ENOMEM, k
            left = g.info()["p"]
            print("refused", p, before, k, left, flush=True)
            assert left in (0, kept)
            if left == 0:
                assert g.info()["block_bytes"] == 0
                with pytest.raises(P.PgabbError) as e:
                    g.cuts()
                assert e.value.status == P.ESTATE
            assert g.count() == want
            assert int(g.task_counts()[1].sum()) == want
            # (sums of at most 2^16 terms in another order)
            assert np.allclose(g.pagerank(max_iter=2)[0], ranks, rtol=1e-10, atol=0)


@pytest.mark.parametrize("p", [1, 3])
@pytest.mark.parametrize("scale,most", [(13, 1 << 22), (13, 1 << 20), (13, 100 << 10), (11, 16 << 10), (11, 6 << 10)])
def test_four_cliques_with_little_memory(p, scale, most):
    """No request above `most` bytes is granted: the matrix of the highest ranks
    (8 MB at scale 13) shrinks, down to nothing at 16 KB, and at 6 KB the
    vertices' lists do not fit either; the 4-lists' counts stay the same."""
    n, s, d = gen.rmat(scale, 32, gen.seed(97, 7))
    want = oracle.four_cliques(n, s, d)
    with P.Graph(n, s, d) as g:
        g.partition(p)
        assert g.info()["max_out_degree"] > 64
        assert g.four_cliques() == want
        ijkl, counts = g.four_clique_lists()
        with RefusingHook(lambda k, b: b > most) as hook:
            assert g.four_cliques() == want
        assert hook.refused > 0
        got_ijkl, got = g.four_clique_lists()
        assert np.array_equal(got_ijkl, ijkl) and np.array_equal(got, counts)
