"""Circuits past the sign program's limits (signs.cpp) on the CPU: what it does
before it gives up is bounded, however long the circuit.  The driver leaves
build_signs a little memory more than the compiled circuit takes.
"""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_23037_amd", "csrc")

DRIVER = r"""
#include "signs.h"
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <new>
#include <sstream>
#include <sys/resource.h>
using namespace soft;
// args: circuit, MB that build_signs may take; prints 1 / 0 (on) or "memory"
int main(int, char **argv) {
    std::ifstream f(argv[1]);
    std::stringstream ss;
    ss << f.rdbuf();
    NoiseModel nm;
    nm.p1 = nm.p2 = nm.p_meas = 1e-5;
    Program P;
    compile_circuit(ss.str(), nm, P, true);
    // the address space in use, and what is allowed on top
    std::ifstream st("/proc/self/statm");
    unsigned long pages = 0;
    st >> pages;
    const rlimit lim = {pages * 4096ul + ((rlim_t)atol(argv[2]) << 20), RLIM_INFINITY};
    if (setrlimit(RLIMIT_AS, &lim)) return 1;
    SignProgram S;
    try {
        build_signs(P, S);
    } catch (const std::bad_alloc &) {
        std::printf("memory\n");
        return 0;
    }
    std::printf("%d\n", (int)S.on);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("limits")
    src = d / "limits.cpp"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src),
                    os.path.join(CSRC, "signs.cpp"), os.path.join(CSRC, "compile.cpp"), "-o", str(d / "limits")], check=True)
    return d


def build(d, lines, mb):
    (d / "c.txt").write_text("\n".join(lines) + "\n")
    return subprocess.run([str(d / "limits"), str(d / "c.txt"), str(mb)], capture_output=True, text=True, check=True).stdout.strip()


def rounds(n):
    return ["CX 0 1\nMR 1\nDETECTOR 0 %d" % i for i in range(n)]


def test_many_tests_and_records(driver):
    # a mask of all record words for each test: 50 MB at 20 000 rounds if the
    # limits were looked at only afterwards
    assert build(driver, ["QUBITS 2"] + rounds(20_000), 24) == "0"
    # few records, many tests of them; many coins
    assert build(driver, ["QUBITS 2", "M 0"] + ["DETECTOR 0 0"] * 60_000, 24) == "0"
    assert build(driver, ["QUBITS 2"] + ["H 0\nR 0"] * 20_000, 24) == "0"


@pytest.mark.parametrize("gates,on", [(100_000, "1"), (220_000, "0")])
def test_signature_table(driver, gates, on):
    # vectors of 13 test words, 13 record words and one of observables, six a
    # slot: 65 and 143 MB of the 134 allowed
    lines = ["QUBITS 3"] + rounds(400) + ["H 2"] * gates + ["M 2"]
    assert build(driver, lines, 110 if on == "1" else 24) == on


def test_within_the_limits(driver):
    assert build(driver, ["QUBITS 2"] + rounds(400), 24) == "1"
