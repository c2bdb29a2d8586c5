"""Streams that end while the caches hold blocks freed on them: a caller's stream
after its graph and batch, a server's after the server.  Later calls on the
library's stream take those blocks."""
import ctypes

import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu


def _hip():
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(next(x.split()[-1] for x in f if "libamdhip64" in x))


@pytest.mark.parametrize("scale", [6, 11, 14])
def test_blocks_outlive_their_streams(scale):
    import torch

    torch.zeros(1, device="cuda")
    hip = _hip()
    n, s, d = gen.rmat(scale, 8, 5)
    want = oracle.tc(n, s, d)
    for _ in range(4):
        st = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(st), 1) == 0
        with P.Graph(n, s, d, stream=st.value) as g:
            g.partition(3)
            assert g.count() == want
        b = P.Batch([(n, s, d)], stream=st.value)
        assert b.count().tolist() == [want]
        b.close()
        assert hip.hipStreamDestroy(st) == 0
        srv = P.Server(1 << 30)
        t = [srv.submit(n, s, d) for _ in range(3)]
        srv.drain()
        assert [srv.poll(x)[1] for x in t] == [want] * 3
        srv.close()
        with P.Graph(n, s, d) as g:
            g.partition(3)
            assert g.count() == want
