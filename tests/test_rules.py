"""CPU checks of the host-only arithmetic in csrc/rules.hpp: a g++-built driver
with overflow checks, against Python's whole numbers."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HDR = os.path.join(ROOT, "paper_2209_04541_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstring>
#include "rules.hpp"
using namespace pgabb;

int main() {
    char op[32];
    long long a, b;
    while (scanf("%31s %lld %lld", op, &a, &b) == 3) {
        if (!strcmp(op, "halfway")) printf("%lld\n", (long long)halfway((int32_t)a, (int32_t)b));
        if (!strcmp(op, "grab")) printf("%d\n", grab_items((int)a, (int)(b / 8), (int)(b % 8)));
        if (!strcmp(op, "low_bits")) printf("%d\n", degrees_by_low_bits(a, b, 13));
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src = d / "drv.cpp"
    src.write_text(DRIVER)
    exe = d / "drv"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover", "-I" + HDR,
                           str(src), "-o", str(exe)])

    def call(lines):
        text = "".join("%s %s\n" % (ln[0], " ".join(map(str, ln[1:]))) for ln in lines)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]

    return call


def test_halfway_of_positions_up_to_the_largest(run):
    top = 2**31 - 1
    pairs = [(0, 0), (0, 1), (6, 7), (2**30, 2**30 + 5), (2**30, top), (0, top), (top - 1, top), (top, top)]
    assert run([("halfway", a, b) for a, b in pairs]) == [(a + b) // 2 for a, b in pairs]


@pytest.mark.parametrize("length", [1, 2, 1000])
@pytest.mark.parametrize("at", [0, 2**30 - 500, 2**30 + 7, 2**31 - 1 - 1000])
def test_halving_stays_inside_the_list(run, at, length):
    """The search for the first entry above a bound, as the walk does it, on a
    list at positions [at, at + length): every probe lies inside."""
    for first in {0, 1, length // 2, length}:  # the answer, from the list's start
        lo, hi = at, at + length
        while lo < hi:
            (mid,) = run([("halfway", lo, hi)])
            assert lo <= mid < hi
            lo, hi = (mid + 1, hi) if mid - at < first else (lo, mid)
        assert lo == at + first


@pytest.mark.parametrize("ends,n", [(70000, 2**20), (70000, 2**24), (70000, 2**26), (100000, 2**28), (2**20, 2**22),
                                    (2**22, 2**24), (2**24, 2**26), (70000, 2**31 - 1), (2**32 - 1, 2**31 - 1)])
def test_sparse_wide_ids_are_counted_in_runs(run, ends, n):
    """Few ends share their high bits: no 8,192 counters per value."""
    assert run([("low_bits", ends, n)]) == [0]


@pytest.mark.parametrize("ends,n", [(70000, 8191), (15_700_000, 2**20), (64_000_000, 2**22), (2_000_000, 2**17)])
def test_dense_ids_are_counted_by_low_bits(run, ends, n):
    assert run([("low_bits", ends, n)]) == [1]


@pytest.mark.parametrize("parts", [1, 2, 3])
@pytest.mark.parametrize("chosen", [2, 16, 64])
def test_an_asked_for_grab_is_kept(run, parts, chosen):
    """rows_per_grab as the caller gave it, in split launches too; a chosen one
    grows with the parts."""
    assert run([("grab", a, 8 * chosen + parts) for a in (0, 1, 5, 64)]) == [chosen * parts, 1, 5, 64]
