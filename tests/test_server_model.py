"""CPU check of the server's streams: the request server and the memory caches
compiled for the host over a model of the runtime (tests/host_model), with the
address and undefined-behaviour sanitizers.  A server's streams end with it, while
blocks that were freed on them stay in the caches: no event that was recorded on
such a stream may be asked or waited for afterwards."""
import os
import subprocess

import pytest

from .test_streamer_model import CSRC, FLAGS, MODEL, sources


@pytest.fixture(scope="module")
def folder(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("server"))
    sources(d)
    with open(os.path.join(CSRC, "server.cpp")) as src, open(os.path.join(d, "request_server.cpp"), "w") as dst:
        dst.write(src.read())
    with open(os.path.join(MODEL, "server.cpp")) as src, open(os.path.join(d, "server.cpp"), "w") as dst:
        dst.write(src.read())
    for f in ("server", "memory", "request_server"):
        subprocess.check_call(["g++"] + FLAGS + ["-c", f + ".cpp", "-o", f + ".o"], cwd=d)
    return d


def link(d, name):
    subprocess.check_call(["g++"] + FLAGS + ["server.o", "memory.o", "request_server.o", "-o", name, "-lpthread"], cwd=d)
    return os.path.join(d, name)


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_blocks_of_an_ended_server_are_taken_without_its_streams(folder, seed):
    r = subprocess.run([link(folder, "model"), "30", str(seed)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["30"]
