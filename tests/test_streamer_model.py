"""CPU check of the streamed count's host side: the streamer and the memory caches
compiled for the host over a model of the runtime (tests/host_model), with the
address and undefined-behaviour sanitizers.  The model runs queued copies and
launches late and in any allowed order, so a wait that is missing, a range that
is reused too early and a copy past its allocation show."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2209_04541_amd", "csrc")
MODEL = os.path.join(ROOT, "tests", "host_model")


FLAGS = ["-std=c++17", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-I" + MODEL, "-I."]


def sources(d):
    for f in ("streamer.hip", "memory.cpp", "block_readers.hpp", "range_pool.hpp", "common.hpp", "count.hpp",
              "graph.hpp", "rules.hpp"):
        with open(os.path.join(CSRC, f)) as src:
            text = src.read().replace('"../../include/pgabb.h"', '"%s/include/pgabb.h"' % ROOT)
        with open(os.path.join(d, f.replace("streamer.hip", "count_streamed.cpp")), "w") as dst:
            dst.write(text)
    for f in ("tc_device.hpp", "streamer.cpp"):
        with open(os.path.join(MODEL, f)) as src, open(os.path.join(d, f), "w") as dst:
            dst.write(src.read())


def link(d, name):
    """The model with count_streamed.cpp as it is in d now."""
    subprocess.check_call(["g++"] + FLAGS + ["-c", "count_streamed.cpp", "-o", name + ".o"], cwd=d)
    subprocess.check_call(["g++"] + FLAGS + ["streamer.o", "memory.o", name + ".o", "-o", name, "-lpthread"], cwd=d)
    return os.path.join(d, name)


@pytest.fixture(scope="module")
def folder(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("streamer"))
    sources(d)
    for f in ("streamer", "memory"):
        subprocess.check_call(["g++"] + FLAGS + ["-c", f + ".cpp", "-o", f + ".o"], cwd=d)
    return d


@pytest.fixture(scope="module")
def model(folder):
    return link(folder, "model")


@pytest.mark.parametrize("seed", [0, 1000, 2000, 3000])
def test_blocks_are_there_when_they_are_read(model, seed):
    r = subprocess.run([model, "250", str(seed)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    ran, refused = map(int, r.stdout.split())
    assert ran > 500 and refused > 50


@pytest.mark.parametrize("line,instead", [
    ("readers.release(v, [&](int32_t w) { PGABB_HIP(hipEventSynchronize(done[w])); });", "readers.release(v, [](int32_t) {});"),
    ("PGABB_HIP(hipStreamWaitEvent(st, ce, 0));", ""),
    ("if (moving) PGABB_HIP(hipStreamWaitEvent(copy_s, moved[b], 0));", ""),
    ("static_cast<size_t>(cap) + kSeg * sizeof(int32_t), s);", "static_cast<size_t>(cap), s);"),
])
def test_the_model_sees_a_missing_wait(folder, model, line, instead):
    """Negative controls: the same without one of the waits, or without the room
    that the last segment reads."""
    path = os.path.join(folder, "count_streamed.cpp")
    with open(path) as f:
        text = f.read()
    assert text.count(line) == 1
    try:
        with open(path, "w") as f:
            f.write(text.replace(line, instead))
        r = subprocess.run([link(folder, "planted"), "400"], capture_output=True, text=True)
    finally:
        with open(path, "w") as f:
            f.write(text)
    assert r.returncode != 0 and "SIM:" in r.stderr, r.stderr[-500:]
