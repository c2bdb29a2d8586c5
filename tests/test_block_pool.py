"""CPU check of the streamer's block placement (csrc/block_pool.hpp).

A g++-built driver places blocks of random sizes with random pinned sets and
costs and checks after every call, against a plain list of what is resident,
that ranges stay inside the pool and never overlap, that pinned blocks stay,
that only reported blocks leave, that a place is found whenever one exists,
that nothing leaves while a free gap holds the block, and that no other place
would have cost less."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HDR = os.path.join(ROOT, "paper_2209_04541_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <vector>
#include "block_pool.hpp"

int main(int argc, char **argv) {
    const uint64_t cap = std::strtoull(argv[1], nullptr, 10);
    const int largest = std::atoi(argv[2]);
    int bad = 0, placed = 0, full = 0;
    for (int trial = 0; trial < 300; ++trial) {
        std::mt19937 rng(trial);
        pgabb::BlockPool bp(cap);
        const int nb = 24;
        std::vector<uint64_t> size(nb), at(nb, UINT64_MAX);
        for (auto &x : size) x = 1 + rng() % largest;
        for (int step = 0; step < 200; ++step) {
            const int b = rng() % nb;
            if (at[b] != UINT64_MAX) continue;
            std::vector<char> pin(nb, 0);
            std::vector<double> cost(nb, 0);
            for (int v = 0; v < nb; ++v) pin[v] = rng() % 5 == 0, cost[v] = rng() % 4;
            // every byte offset tried
            double best = -1;
            for (uint64_t o = 0; o + size[b] <= cap; ++o) {
                double c = 0;
                bool ok = true;
                for (int v = 0; v < nb; ++v)
                    if (at[v] != UINT64_MAX && at[v] < o + size[b] && o < at[v] + size[v]) {
                        if (pin[v]) ok = false;
                        c += cost[v];
                    }
                if (ok && (best < 0 || c < best)) best = c;
            }
            bool gap = false;
            for (uint64_t o = 0; o + size[b] <= cap && !gap; ++o) {
                gap = true;
                for (int v = 0; v < nb; ++v)
                    if (at[v] != UINT64_MAX && at[v] < o + size[b] && o < at[v] + size[v]) gap = false;
            }
            double paid = 0;
            int left = 0;
            const uint64_t off = bp.place(b, size[b], [&](int32_t v) { return pin[v] != 0; },
                                          [&](int32_t v) { return cost[v]; },
                                          [&](int32_t v) {
                                              if (pin[v] || at[v] == UINT64_MAX) ++bad;
                                              paid += cost[v];
                                              ++left;
                                              at[v] = UINT64_MAX;
                                          });
            if (off == UINT64_MAX) {
                if (best >= 0 || left) ++bad;
                ++full;
                continue;
            }
            ++placed;
            if (off + size[b] > cap || paid != best || (gap && left)) ++bad;
            for (int v = 0; v < nb; ++v)
                if (at[v] != UINT64_MAX && at[v] < off + size[b] && off < at[v] + size[v]) ++bad;
            at[b] = off;
            if (rng() % 40 == 0) {
                bp.clear();
                at.assign(nb, UINT64_MAX);
            }
        }
    }
    printf("%d %d %d\n", bad, placed, full);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    src = d / "drv.cpp"
    src.write_text(DRIVER)
    exe = d / "drv"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + HDR, str(src), "-o", str(exe)])
    return str(exe)


@pytest.mark.parametrize("cap,largest", [(40, 12), (100, 30), (37, 40), (1, 2), (0, 1)])
def test_places(driver, cap, largest):
    bad, placed, full = map(int, subprocess.check_output([driver, str(cap), str(largest)]).split())
    assert bad == 0
    assert placed > 0 or cap == 0
    assert full > 0 or largest * 3 < cap
