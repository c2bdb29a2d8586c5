"""Launch shapes kept in the tuning cache by a library with other kernels are not
taken: the search runs again and its result is stored beside them."""
import os

import numpy as np
import pytest

import oracle
import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

pytestmark = pytest.mark.gpu


def keys_of(path, prefix):
    with open(path) as f:
        return {ln.split()[0] for ln in f if ln.startswith(prefix)}


@pytest.fixture
def cache(monkeypatch, tmp_path):
    import torch  # noqa: F401  (before the library: both load the HIP runtime)
    path = str(tmp_path / "tune.txt")
    before = os.environ.get("PGABB_TUNE_CACHE")
    monkeypatch.setenv("PGABB_TUNE_CACHE", path)
    assert P.lib().pgabb_tune_cache_reload() == P.OK
    yield path
    if before is None:
        monkeypatch.delenv("PGABB_TUNE_CACHE")
    else:
        monkeypatch.setenv("PGABB_TUNE_CACHE", before)
    assert P.lib().pgabb_tune_cache_reload() == P.OK


def shapes(which):
    if which == "batch":
        gl = [gen.batch_graph(g, (64, 900)) for g in range(24)]
        with P.Batch(gl) as b:
            assert np.array_equal(b.count(), np.array([oracle.tc(*x) for x in gl], np.uint64))
    else:
        gl = [gen.er(901, 9000, gen.seed(983, k)) for k in range(3)]
        objs = [P.Graph(*x) for x in gl]
        try:
            assert P.tc_count_batch(objs) == [oracle.tc(*x) for x in gl]
        finally:
            for g in objs:
                g.close()


@pytest.mark.parametrize("which,prefix", [("batch", "batch/"), ("graphs", "tc_graphs/")])
def test_unversioned_shapes_are_searched_again(cache, which, prefix):
    shapes(which)
    (key,) = keys_of(cache, prefix)
    parts = key.split("/")
    assert not parts[1].startswith(("G", "T"))  # a version, then the class
    old = "/".join(parts[:1] + parts[2:])
    with open(cache, "w") as f:
        f.write("%s 1 8 64\n" % old)  # as a library without versions wrote it
    assert P.lib().pgabb_tune_cache_reload() == P.OK
    shapes(which)
    assert keys_of(cache, prefix) == {old, key}
    # and a shape of this version is taken as it is
    with open(cache) as f:
        kept = f.read()
    assert P.lib().pgabb_tune_cache_reload() == P.OK
    shapes(which)
    with open(cache) as f:
        assert f.read() == kept
