"""Lifetime of a context's device buffers (devbuf.h) on the CPU, with an
allocator that logs: what a recording holds is neither freed nor handed out for
new contents before the end, everything else is freed when it is replaced, and
nothing is left at the end.
"""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_23037_amd", "csrc")

DRIVER = r"""
#include "devbuf.h"
#include <cstdio>
#include <cstdlib>
#include <set>
static std::set<void *> live;
static bool refuse = false;
struct Mem {
    static int alloc(void **p, size_t n) { if (refuse) return 2; *p = std::malloc(n); live.insert(*p); return 0; }
    static int free(void *p) { if (!live.erase(p)) std::abort(); std::free(p); return 0; }
};
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    soft::Buffers<Mem> m;
    soft::DevBuf<int> a, t;
    // not recorded: kept while it is large enough, freed when it grows
    CHECK(m.ensure(a, 0) == 0 && a.p && a.n == 1);
    CHECK(m.ensure(a, 10) == 0 && a.n == 10 && live.size() == 1);
    int *p0 = a.p;
    CHECK(m.ensure(a, 4) == 0 && a.p == p0 && m.renew(a, 9) == 0 && a.p == p0);
    // recorded: grows into a new buffer, the old one stays
    a.recorded = true;
    CHECK(m.ensure(a, 10) == 0 && a.p == p0 && a.recorded);
    CHECK(m.ensure(a, 11) == 0 && a.p != p0 && !a.recorded && live.count(p0));
    // the new one is in no recording: freed when it grows
    CHECK(m.ensure(a, 100) == 0 && live.size() == 2 && live.count(p0) && live.count(a.p));
    // recorded tables are not written again, also when they would fit
    CHECK(m.renew(t, 8) == 0);
    int *t0 = t.p;
    t.recorded = true;
    CHECK(m.renew(t, 8) == 0 && t.p != t0 && live.count(t0) && !t.recorded);
    CHECK(m.renew(t, 8) == 0 && live.size() == 4);
    // a refused allocation leaves an empty buffer and what was recorded
    t.recorded = true;
    int *t1 = t.p;
    refuse = true;
    CHECK(m.renew(t, 8) == 2 && !t.p && t.n == 0 && !t.recorded && live.count(t1));
    refuse = false;
    CHECK(m.renew(t, 8) == 0 && t.p);
    m.release(a);
    m.release(t);
    CHECK(live.size() == 3 && live.count(p0) && live.count(t0) && live.count(t1));
    m.release_aside();
    CHECK(live.empty());
    return 0;
}
"""


def test_lifetimes(tmp_path):
    src, exe = tmp_path / "devbuf.cpp", tmp_path / "devbuf"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-fsanitize=address", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
