"""How a launch's items are dealt out to its waves (queue.h) on the CPU: waves
draw in any order until each has been told that nothing is left, and every item
has to be taken exactly once -- also by fewer waves than cursors.  Two drivers
of the same loop: the header's arithmetic, and (to show that the check sees it)
one that always deals by eight cursors, which leaves items without a wave.
"""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_23037_amd", "csrc")

DRIVER = r"""
#include "queue.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
#ifdef ALWAYS_EIGHT
static uint32_t cursor(uint32_t w, uint32_t) { return w % 8u; }
static uint64_t nth(uint32_t id, uint64_t c, uint32_t waves) { return ((waves - id + 7u) / 8u + c) * 8u + id; }
#else
static uint32_t g_shift;
static uint32_t cursor(uint32_t w, uint32_t) { return soft::queue_cursor(w, g_shift); }
static uint64_t nth(uint32_t id, uint64_t c, uint32_t waves) { return soft::queue_item(id, c, waves, g_shift); }
#endif
// args: waves, items, seed, one (1: one cursor); prints the items taken, and those taken more than once
int main(int, char **argv) {
    const uint32_t waves = (uint32_t)atoi(argv[1]);
    const uint64_t n = (uint64_t)atoll(argv[2]);
    uint64_t x = 0x9E3779B97F4A7C15ull * (uint64_t)(atoi(argv[3]) + 1);
    std::vector<uint32_t> taken(n, 0u), live;
#ifndef ALWAYS_EIGHT
    g_shift = atoi(argv[4]) ? 0u : soft::queue_shift(waves);
#endif
    std::vector<char> started(waves, 0);
    unsigned long long cursors[soft::kQueueCursors] = {};
    for (uint32_t w = 0; w < waves; ++w) live.push_back(w);
    while (!live.empty()) {
        x ^= x << 13; x ^= x >> 7; x ^= x << 17;
        const size_t k = (size_t)(x % live.size());
        const uint32_t w = live[k];
        uint64_t item = w;
        bool more = true;
        if (!started[w]) started[w] = 1;
        else if (n <= waves) more = false;
        else item = nth(cursor(w, waves), cursors[cursor(w, waves)]++, waves);
        if (!more || item >= n) { live[k] = live.back(); live.pop_back(); continue; }
        ++taken[item];
    }
    size_t got = 0, twice = 0;
    for (uint32_t t : taken) { got += t > 0; twice += t > 1; }
    std::printf("%zu %zu\n", got, twice);
    return 0;
}
"""


@pytest.fixture(scope="module")
def drivers(tmp_path_factory):
    d = tmp_path_factory.mktemp("queue")
    src = d / "queue.cpp"
    src.write_text(DRIVER)
    exes = []
    for flags in ([], ["-DALWAYS_EIGHT"]):
        exes.append(str(d / ("queue%d" % len(exes))))
        subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", exes[-1]] + flags, check=True)
    return exes


def taken(exe, waves, n, seed, one=0):
    out = subprocess.run([exe, str(waves), str(n), str(seed), str(one)], capture_output=True, text=True, check=True)
    return tuple(int(v) for v in out.stdout.split())


@pytest.mark.parametrize("waves", list(range(1, 21)) + [63, 64, 255, 1030])
def test_every_item_once(drivers, waves):
    for n in (1, 2, 7, 8, 9, 63, 64, 1000, waves, waves + 1, 3 * waves + 5):
        for seed in range(3):
            assert taken(drivers[0], waves, n, seed) == (n, 0), (n, seed)
        assert taken(drivers[0], waves, n, 3, one=1) == (n, 0), n


@pytest.mark.parametrize("waves", [2, 4, 6])
def test_the_check_sees_items_without_a_wave(drivers, waves):
    got, twice = taken(drivers[1], waves, 63, 0)
    assert got < 63 and twice == 0
