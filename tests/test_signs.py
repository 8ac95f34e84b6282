"""The sign program of a list (signs.cpp) on the CPU, no GPU: a driver built
with g++ draws each shot's noise from the oracle's Philox words, XORs the hits'
signatures and reads off what ends the shot, the way the kernel does one lane
at a time.  Every shot that the signs decide must have the oracle's status,
abort op, observables and record; the others are counted.  Whole numbers, so
the comparison is exact.
"""
from __future__ import annotations

import os
import subprocess

import numpy as np
import pytest

import oracle
import workloads
from tests.gen_small import random_circuit

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_23037_amd", "csrc")
KEYS = ("p1", "p2", "p_idle", "p_meas", "p_reset", "p_mpp")

DRIVER = r"""
#include "signs.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <sstream>
using namespace soft;
// args: circuit, words file (rows of noise + measurement words), rows, six noise rates
int main(int argc, char **argv) {
    std::ifstream f(argv[1]);
    std::stringstream ss;
    ss << f.rdbuf();
    const size_t rows = (size_t)atoll(argv[3]);
    NoiseModel nm;
    double *q[6] = {&nm.p1, &nm.p2, &nm.p_idle, &nm.p_meas, &nm.p_reset, &nm.p_mpp};
    for (int i = 0; i < 6; ++i) *q[i] = atof(argv[4 + i]);
    Program P;
    compile_circuit(ss.str(), nm, P, true);
    SignProgram S;
    build_signs(P, S);
    std::printf("%d %d %.17g\n", (int)S.on, (int)S.complete, S.ends);
    if (!S.on) return 0;
    const uint32_t nt = (uint32_t)S.tests.size() - 1u, tw = S.need.tests, rw = S.need.recs;
    size_t resolved = 0;
    std::vector<uint32_t> words((size_t)P.n_noise + P.n_meas);
    std::ifstream wf(argv[2], std::ios::binary);
    for (size_t i = 0; i < rows; ++i) {
        wf.read((char *)words.data(), words.size() * 4);
        std::vector<uint32_t> x = S.ref;
        auto add = [&](const uint32_t *v) { for (size_t w = 0; w < x.size(); ++w) x[w] ^= v[w]; };
        for (size_t c = 0; c < S.coin.size(); ++c)
            if (words[P.n_noise + S.coin_slot[c]] >> 31) add(S.coin[c].data());
        // Basis entries still possible: the XORs of subsets of `gen` (index
        // shift, vector) on top of the entry that x follows.
        struct Gen { uint64_t beta; std::vector<uint32_t> v; };
        std::vector<Gen> gen;
        uint32_t t = 0, m = 0, m_at = 0;  // first set test; measurements passed, and the next that reads
        bool hand = false;
        auto first = [&]() { for (t = 0; t < nt && !((x[t >> 5] >> (t & 31u)) & 1u); ++t) {} };
        auto apply = [&](uint32_t s) {
            const SignSlot &L = S.slots[s];
            if (L.kind == NZ_NONE || words[s] > L.thr1) return;
            const uint64_t d = (uint64_t)L.thr1 + 1, w = words[s];
            uint32_t a = 1, b = 0;
            if (L.kind == NZ_DEP1) a = (uint32_t)(3 * w / d) + 1;
            else if (L.kind == NZ_DEP2) { const uint32_t k = (uint32_t)(15 * w / d) + 1; a = k >> 2; b = k & 3; }
            else if (L.kind == NZ_ZERR) a = 3;
            if (a) add(&S.vecs[((size_t)s * kSignVecs + a - 1) * x.size()]);
            if (b) add(&S.vecs[((size_t)s * kSignVecs + 3 + b - 1) * x.size()]);
        };
        uint32_t s = 0;
        for (;;) {
            first();
            // the next thing that happens: a measurement that tells entries
            // apart, or the first set test
            uint32_t c = m;
            while (!gen.empty() && c < S.meas.size()) {
                bool reads = S.meas[c].gamma == ~0ull;
                for (const Gen &g : gen) reads = reads || __builtin_parityll(S.meas[c].gamma & g.beta);
                if (reads) break;
                ++c;
            }
            m_at = c;
            const bool at_meas = !gen.empty() && c < S.meas.size() && t >= S.meas[c].test;
            const uint32_t stop = at_meas ? S.meas[c].stop : S.tests[t].stop;
            if (s < stop) { apply(s++); continue; }
            if (at_meas) {
                const SignMeas &M = S.meas[c];
                if (M.rec == kNone) { hand = true; break; }
                const uint32_t bit = words[P.n_noise + M.slot] >> 31;
                const uint32_t o = (x[tw + (M.rec >> 5)] >> (M.rec & 31u)) & 1u;
                size_t p = gen.size();
                for (size_t j = 0; j < gen.size(); ++j) {
                    if (!__builtin_parityll(M.gamma & gen[j].beta)) continue;
                    if (p == gen.size()) { p = j; continue; }
                    gen[j].beta ^= gen[p].beta;
                    for (size_t w = 0; w < x.size(); ++w) gen[j].v[w] ^= gen[p].v[w];
                }
                if (o != bit) add(gen[p].v.data());
                gen.erase(gen.begin() + p);
                m = c + 1;
                ++resolved;
                continue;
            }
            if (S.tests[t].kind != SGT_PAIR) break;
            x[t >> 5] ^= 1u << (t & 31u);
            const SignPair &Q = S.pairs[S.tests[t].pair];
            for (uint32_t sub = 0; sub < (1u << gen.size()); ++sub) {
                uint64_t b = Q.beta;
                for (size_t j = 0; j < gen.size(); ++j) if ((sub >> j) & 1u) b ^= gen[j].beta;
                if (!b) hand = true;
            }
            if (hand || gen.size() == 4) { hand = true; break; }
            gen.push_back(Gen{Q.beta, S.pair_vecs[Q.vec]});
            m = gen.size() > 1 ? std::min(m_at, Q.meas) : Q.meas;
        }
        if (hand) { std::printf("-\n"); continue; }
        const SignTest &T = S.tests[t];
        if (T.kind == SGT_HAND) { std::printf("-\n"); continue; }
        std::printf("%u %u %u", T.kind == SGT_NONE ? 0u : 1u, T.src, x[tw + rw] & S.mask[t][rw]);
        for (uint32_t w = 0; w < rw; ++w) std::printf(" %u", x[tw + w] & S.mask[t][w]);
        std::printf("\n");
    }
    std::printf("resolved %zu\n", resolved);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("signs")
    src = d / "signs.cpp"
    src.write_text(DRIVER)
    exe = d / "signs"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src),
                    os.path.join(CSRC, "signs.cpp"), os.path.join(CSRC, "compile.cpp"), "-o", str(exe)], check=True)
    return d, exe


def check(driver, text, noise, seed, n, hit_rate=None):
    """(decided shots, on, complete) after comparing the decided ones."""
    d, exe = driver
    circ = oracle.Circuit(text, {k: noise.get(k, 0.0) for k in KEYS})
    rng = np.random.default_rng(seed)
    words = rng.integers(0, 2**32, size=(n, circ.words_per_shot), dtype=np.uint64).astype(np.uint32)
    if hit_rate is not None and circ.n_noise_slots:  # denser hits than the model's
        thr = int(max(noise.values()) * 2**32)
        hit = rng.random((n, circ.n_noise_slots)) < hit_rate
        words[:, :circ.n_noise_slots] = np.where(hit, rng.integers(0, max(1, thr), size=hit.shape),
                                                 rng.integers(thr, 2**32, size=hit.shape)).astype(np.uint32)
    (d / "c.txt").write_text(text)
    (d / "w.bin").write_bytes(np.ascontiguousarray(words).tobytes())
    out = subprocess.run([str(exe), str(d / "c.txt"), str(d / "w.bin"), str(n)] +
                         [repr(float(noise.get(k, 0.0))) for k in KEYS], capture_output=True, text=True, check=True)
    lines = out.stdout.splitlines()
    on, complete, ends = lines[0].split()
    if not int(on):
        return 0, False, False
    ref = circ.batch(0, 0, n, words=words)
    decided = 0
    assert lines[-1].startswith("resolved ")
    check.resolved = int(lines[-1].split()[1])
    for i, line in enumerate(lines[1:-1]):
        if line == "-":
            continue
        v = [int(x) for x in line.split()]
        decided += 1
        assert v[0] == ref["status"][i] and v[1] == ref["abort_op"][i] and v[2] == ref["obs"][i], i
        assert v[3:] == [int(x) for x in ref["outcomes"][:, i]], i
    return decided, True, bool(int(complete))


@pytest.mark.parametrize("name,rate", [("cultivation_15q", None), ("cultivation_15q", 0.01), ("cultivation_42q", None),
                                       ("cultivation_42q", 0.004), ("clifford_t_8q", None)])
def test_workloads(driver, name, rate):
    w = workloads.config(name, seed=1)
    n = 3000
    decided, on, complete = check(driver, w.text, w.noise, 1, n, rate)
    assert on and complete == name.startswith("cultivation")
    assert decided > (0.9 if name == "clifford_t_8q" else 0.99) * n
    if complete:
        assert check.resolved > 20  # broken pairs whose branch a measurement took


@pytest.mark.parametrize("order", ["shuffled", "shuffled_tick"])
@pytest.mark.parametrize("seed,shape", enumerate([(7, 8, 3, [7, 4], 4), (9, 6, 3, [9, 5], 6), (8, 6, 2, [8], 6),
                                                  (10, 6, 3, [10, 6, 3], 6)]))
def test_brackets(driver, seed, shape, order):
    nd, na, rz, br, wt = shape
    w = workloads.cultivation_shaped(100 + seed, nd, na, rz, br, check_weight=wt, inverse_order=order)
    decided, on, complete = check(driver, w.text, w.noise, seed, 1500, 0.01)
    assert on and complete and decided > 500


def with_checks(text):
    """Postselect every other recorded Z measurement and observe the last."""
    out, rec = [], -1
    for line in text.strip().split("\n"):
        out.append(line)
        if line.split()[0] in ("M", "MX", "MR", "MRX", "MPP"):
            rec += 1
            if rec % 2 == 0:
                out.append("DETECTOR %d %s" % (rec % 4 // 2, " ".join(str(r) for r in range(rec, -1, -3)[:2])))
    return "\n".join(out + (["OBSERVABLE 1 %d" % rec, "OBSERVABLE 0 0"] if rec >= 0 else [])) + "\n"


@pytest.mark.parametrize("seed", range(40))
def test_random_circuits(driver, seed):
    # every op family: coins (random measurements outside the span), resets,
    # feedback by XOR and AND, diagonal and controlled gates, record flips
    rng = np.random.default_rng(seed)
    n = int(rng.integers(2, 9))
    text, _ = random_circuit(51000 + seed, n, int(rng.integers(20, 140)), p_t=0.0 if seed % 3 == 0 else 0.05,
                             p_meas=0.1, p_mpp=0.05, p_reset=0.05, p_msc=0.15 if seed % 2 else 0.0,
                             p_diag=0.03 if seed % 5 == 1 else 0.0, p_if=0.05 if seed % 4 == 2 else 0.0)
    noise = {"p1": 0.02, "p2": 0.02, "p_meas": 0.02, "p_reset": 0.02, "p_mpp": 0.05}
    decided, on, _ = check(driver, with_checks(text), noise, seed, 600)
    if seed % 3 == 0:
        assert on


def test_no_noise_and_empty(driver):
    for text in ("QUBITS 1\n", "QUBITS 2\nH 0\nT 0\nTDG 0\n", "QUBITS 1\nM 0\nDETECTOR 1 0\n"):
        decided, on, complete = check(driver, text, {}, 1, 4)
        assert on and complete and decided == 4
