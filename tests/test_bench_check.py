"""The benchmark's comparison of the timed launch with the oracle: it runs the
launch that is timed (not one with kept states, which leaves the sign pass
out), and a mistake in any output is counted.
"""
from __future__ import annotations

import numpy as np
import pytest

import bench
import oracle
import workloads


@pytest.fixture(scope="module")
def reference():
    w = workloads.config("clifford_t_8q", seed=1)
    circ = oracle.Circuit(w.text, w.noise)
    return circ, circ.batch(bench.SEED_RNG, 0, 300)


def copy(ref, n):
    return {k: np.array(ref[k][..., :n]) for k in ("outcomes", "status", "abort_op", "obs")}


def test_identical(reference):
    circ, ref = reference
    for bits in (32, 64):
        got = bench.compare_timed(oracle, circ, ref, copy(ref, 200), bits)
        assert got["shots"] == got["shots_identical"] == 200 and got["outcome_flips_outside_guard_band"] == 0


@pytest.mark.parametrize("key", ["outcomes", "status", "abort_op", "obs"])
def test_a_mistake_is_counted(reference, key):
    circ, ref = reference
    sub = copy(ref, 200)
    sub[key].reshape(-1, 200)[-1, 17] ^= 1
    got = bench.compare_timed(oracle, circ, ref, sub, 64)
    assert got["shots_identical"] == 199 and got["outcome_flips_outside_guard_band"] == 1


@pytest.mark.gpu
def test_the_timed_launch_is_what_is_compared():
    import torch
    from paper_2512_23037_amd import soft
    w = workloads.config("cultivation_15q", seed=1)
    ctx = bench.make_ctx(soft, w, 32, 1)
    shots, n = 50_000, 4000
    bufs = soft.sample(ctx, 0, shots)
    sub = bench.timed_subset(torch, ctx, shots, bufs, n)
    decided = ctx.counters()
    kept = bench.sample_subset(torch, soft, ctx, n)
    walked = ctx.counters()
    # per shot, the timed launch computes next to nothing by coefficients
    assert decided["events"] * n < 0.1 * walked["events"] * shots
    assert decided["shots"] == shots and walked["shots"] == n
    circ = oracle.Circuit(w.text, w.noise, noise_mode=1)
    ref = circ.batch(bench.SEED_RNG, 0, n)
    assert bench.compare_timed(oracle, circ, ref, sub, 32)["outcome_flips_outside_guard_band"] == 0
    assert bench.compare_with_oracle(oracle, circ, ref, kept, 32, 8)["outcome_flips_outside_guard_band"] == 0
