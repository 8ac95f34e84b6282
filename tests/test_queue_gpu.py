"""Launches of fewer waves than the work queue has cursors: soft_run_noalloc
shrinks its grid to the slabs that its scratch holds (two waves at span 20 in
FP64), and a launch of a shot or two builds every variant's checkpoint states
on one block.  Whole numbers against soft_run, bit for bit, with every output
filled beforehand.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads
from paper_2512_23037_amd import soft
from tests.gpu_helpers import make_ctx

pytestmark = pytest.mark.gpu


def outputs(run, ctx, shot0, n):
    import torch
    nw = max(ctx.info()["record_words"], 1)
    outs = [torch.full((nw, n), -7, dtype=torch.int32, device="cuda")] + \
        [torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
    run(shot0, n, *outs)
    torch.cuda.synchronize()
    c = ctx.counters()
    return [o.cpu().numpy().view(np.uint32) for o in outs], [c[f] for f in ("shots", "passed", "discarded", "logical_errors")]


def wide(k):
    """A span of 2^k entries read by four measurements, after a check that a
    tenth of the shots fail (so that the sign pass runs)."""
    out = ["QUBITS %d" % (k + 1), "M %d" % k, "DETECTOR 0 0"]
    out += ["H %d\nT %d" % (q, q) for q in range(k)]
    out += ["H %d\nM %d" % (q, q) for q in range(4)]
    return "\n".join(out + ["OBSERVABLE 0 1 2"]) + "\n"


@pytest.mark.parametrize("k,bits,wpb,waves", [(18, 64, 3, 6), (19, 64, 2, 4), (20, 32, 2, 4), (20, 64, 2, 2),
                                              (20, 64, 1, 2), (18, 32, 2, 16)])
@pytest.mark.parametrize("mode", [0, 1])
def test_few_waves(k, bits, wpb, waves, mode):
    ctx = make_ctx(wide(k), {"p_meas": 0.1}, seed=3, bits=bits, shape=(wpb, 0, 0))
    ctx.set_noise_mode(mode)
    ctx.set_tile_memory(2)
    for n in (1, waves, waves + 1, 3 * waves + 5):
        ref = outputs(ctx.run, ctx, 11, n)
        got = outputs(ctx.run_noalloc, ctx, 11, n)
        assert ref[1][0] == got[1][0] == n
        for a, b in zip(ref[0], got[0]):
            assert (a == b).all()
        assert ref[1] == got[1]
        assert not (got[0][1] == 0xFFFFFFFF).any()


def test_states_of_every_variant_on_one_block():
    # another circuit's states are in the scratch before each call
    mix = workloads.mixture(seed=1, total_shots=27000)
    ends = mix["shot_ends"]
    m = soft.Context(0)
    m.load_mixture([w.text for w in mix["workloads"]], mix["models"], ends)
    m.set_rng(3)
    m.set_noise_mode(1)
    w = workloads.config("cultivation_42q", seed=1)
    other = make_ctx(w.text, w.noise, seed=9)
    for v, end in enumerate(ends):
        outputs(other.run_noalloc, other, 0, 64)
        for n in (1, 2):
            shot0 = int(end) - 3 * (v + 1)
            ref = outputs(m.run, m, shot0, n)
            got = outputs(m.run_noalloc, m, shot0, n)
            for a, b in zip(ref[0], got[0]):
                assert (a == b).all(), (v, n)
            assert ref[1] == got[1]


@pytest.mark.parametrize("grab", [0, 1, 7, 8, 64])
def test_one_cursor_and_eight(grab):
    # groups around the size from which one cursor serves all waves (256 or
    # 512 of them), without the sign pass
    w = workloads.config("cultivation_15q", seed=1)
    ref = make_ctx(w.text, w.noise, seed=5)
    ref.set_shared_prefix(False)
    for wpb in (1, 2):
        ctx = make_ctx(w.text, w.noise, seed=5, shape=(wpb, 1, grab))
        ctx.set_shared_prefix(False)
        for n in (256 * wpb * 31, 256 * wpb * 32 - 1, 256 * wpb * 32, 256 * wpb * 41 + 7):
            a, b = outputs(ref.run, ref, 3, n), outputs(ctx.run, ctx, 3, n)
            for x, y in zip(a[0], b[0]):
                assert (x == y).all(), n
            assert a[1] == b[1] and a[1][0] == n
