"""What the counters say of shots that the sign pass decides (soft.h): every
shot is in one support bin, a decided one in that of the checkpoint before its
first noise hit (and among prefix_shots if there is one), gap sampling counts
the pairs of words that the oracle draws from, and nothing else of the sampler's work.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_helpers import make_ctx, run_gpu
from tests.test_signs_gpu import NOISE, rounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,p,bits,mode", [("cultivation_15q", 4e-3, 64, 0), ("cultivation_42q", 1e-3, 32, 1),
                                              ("cultivation_42q", 5e-4, 64, 1), ("clifford_t_8q", 4e-3, 64, 0),
                                              ("cultivation_42q", 1e-2, 32, 0)])
@pytest.mark.parametrize("n", [100, 5000, 150_000])
def test_every_shot_is_in_a_bin(name, p, bits, mode, n):
    ctx = make_ctx(workloads.config(name, seed=1).text, {k: p for k in NOISE}, seed=5, bits=bits)
    ctx.set_noise_mode(mode)
    for run in (ctx.run, ctx.run_noalloc):
        import torch
        st = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        run(0, n, status=st)
        torch.cuda.synchronize()
        c = ctx.counters()
        assert sum(c["support_hist"]) == c["shots"] == n == c["passed"] + c["discarded"]
        assert c["prefix_shots"] <= n and c["restarts"] <= n


def brackets(hit):
    """Three Bell pairs, twice a T layer that meets its inverse around checks of
    the pairs' parities; a certain X on the check's ancilla before `hit`."""
    out = ["QUBITS 7"]
    for i in range(3):
        out += ["H %d" % (2 * i), "CX %d %d" % (2 * i, 2 * i + 1)]
    rec = 0
    for r in range(2):
        if hit == ("layer", r):
            out.append("XERR 1.0 6")
        out += ["T %d" % (2 * i) for i in range(3)]
        for i in range(3):
            out += ["CX %d 6" % (2 * i), "CX %d 6" % (2 * i + 1)]
            if hit == ("check", r, i):
                out.append("XERR 1.0 6")
            out += ["MR 6", "DETECTOR 0 %d" % rec]
            rec += 1
        out += ["TDG %d" % (2 * i) for i in range(3)]
    return "\n".join(out) + "\n"


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("hit,support", [(("layer", 0), 0), (("check", 0, 2), 3), (("layer", 1), 3), (("check", 1, 1), 3), (None, 3)])
def test_bins_of_decided_shots(hit, support, mode):
    # before the first T layer the state is one entry and no checkpoint has
    # been passed; from it on the largest support was 2^3
    n = 3000
    ctx = make_ctx(brackets(hit), {}, seed=5)
    ctx.set_noise_mode(mode)
    out = run_gpu(ctx, 0, n)
    c = ctx.counters()
    assert c["events"] == 0 and c["entries_t"] == 0  # all decided
    assert (out["status"] == (0 if hit is None else 1)).all()
    assert c["support_hist"] == [n if b == support else 0 for b in range(16)]
    assert c["prefix_shots"] == (0 if hit == ("layer", 0) else n)
    assert c["restarts"] == 0 and c["max_norm_dev"] == 0.0
    # the sampler's own walk ends the shots the same way
    ctx.set_shared_prefix(False)
    ref = run_gpu(ctx, 0, n)
    for k in ref:
        assert (ref[k] == out[k]).all()


@pytest.mark.parametrize("p", [1e-4, 3e-3, 5e-2])
@pytest.mark.parametrize("n_rounds", [1, 12, 40])
def test_gap_words(n_rounds, p):
    # without checks a shot looks at every candidate up to the last slot: a gap
    # word and an acceptance word each, also for the gap that passes the end (of
    # which the oracle counts the first alone)
    text = "\n".join(l for l in rounds(n_rounds).split("MPP")[0].split("\n") if not l.startswith(("DETECTOR", "T"))) + "\n"
    noise = {k: p / (1 + i % 3) for i, k in enumerate(NOISE)}
    n = 4000
    ctx = make_ctx(text, noise, seed=23)
    ctx.set_noise_mode(1)
    run_gpu(ctx, 7, n)
    c = ctx.counters()
    assert c["events"] == 0 and c["passed"] == n
    ref = oracle.Circuit(text, noise, noise_mode=1).batch(23, 7, n)
    assert c["noise_slots"] == ref["work"]["noise_words"] + n


def test_runs_are_counted():
    w = workloads.config("cultivation_15q", seed=1)
    ctx = make_ctx(w.text, w.noise, seed=5)
    for i in range(1, 5):
        run_gpu(ctx, 0, 1000 * i)
        assert ctx.graph_info() == {"instantiations": 0, "launches": i}
    ctx.set_precision(32)
    run_gpu(ctx, 0, 100)
    assert ctx.graph_info() == {"instantiations": 0, "launches": 5}
    import torch
    st = torch.zeros(100, dtype=torch.int32, device="cuda")
    ctx.run_noalloc(0, 100, status=st)
    torch.cuda.synchronize()
    assert ctx.graph_info() == {"instantiations": 0, "launches": 5}
