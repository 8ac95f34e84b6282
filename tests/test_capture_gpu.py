"""Recordings of soft_run and soft_run_noalloc by a stream capture, replayed
after everything that replaces the context's buffers: a run that needs larger
checkpoint slots or more device-memory tiles, and loads of other circuits.
Each replay is checked against the eager run of the same shots, with the
context's own runs and synchronizations between.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads
from paper_2512_23037_amd import soft
from tests.gpu_helpers import make_ctx, run_gpu

pytestmark = pytest.mark.gpu

NOISE = {k: 4e-3 for k in ("p1", "p2", "p_idle", "p_meas", "p_reset", "p_mpp")}


class Recording:
    def __init__(self, ctx, shot0, n, noalloc=False):
        import torch
        self.ref = run_gpu(ctx, shot0, n)
        self.outs = soft.sample(ctx, shot0, n)
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph, stream=torch.cuda.Stream()):
            (ctx.run_noalloc if noalloc else ctx.run)(shot0, n, *self.outs, stream=torch.cuda.current_stream().cuda_stream)

    def check(self):
        import torch
        for o in self.outs:
            o.fill_(-7)
        torch.cuda.synchronize()
        self.graph.replay()
        torch.cuda.synchronize()
        for o, k in zip(self.outs, ("outcomes", "status", "abort_op", "obs")):
            got = o.cpu().numpy().view(np.uint32)
            want = self.ref[k]
            assert (got[: want.shape[0]] == want).all(), k


@pytest.mark.parametrize("tiles", [0, 2, 3])
@pytest.mark.parametrize("noalloc", [False, True])
def test_replays_after_larger_runs_and_loads(tiles, noalloc):
    w42, w15 = (workloads.config(c, seed=1) for c in ("cultivation_42q", "cultivation_15q"))
    ctx = make_ctx(w42.text, w42.noise, seed=5, bits=32)
    ctx.set_noise_mode(1)
    ctx.set_tile_memory(tiles)
    a = Recording(ctx, 0, 3001, noalloc)
    a.check()
    # larger slots and slabs, more waves
    ctx.set_precision(64)
    big = run_gpu(ctx, 0, 200_000)
    a.check()
    assert (run_gpu(ctx, 0, 200_000)["status"] == big["status"]).all()
    # a second recording, with the larger ones
    b = Recording(ctx, 77, 2000, noalloc)
    b.check()
    a.check()
    # other tables, smaller and larger than the recorded ones
    for text, noise in ((w15.text, NOISE), (w42.text, {k: v / 2 for k, v in w42.noise.items()})):
        ctx.load_noise(**{k: noise.get(k, 0.0) for k in NOISE})
        ctx.load_circuit(text)
        fresh = make_ctx(text, noise, seed=5, bits=64)
        fresh.set_noise_mode(1)
        want = run_gpu(fresh, 0, 5000)
        for _ in range(2):
            got = run_gpu(ctx, 0, 5000)
            for k in want:
                assert (got[k] == want[k]).all(), k
            a.check()
            b.check()
    mix = workloads.mixture(seed=1, total_shots=27000)
    ctx.load_mixture([w.text for w in mix["workloads"]], mix["models"], mix["shot_ends"])
    run_gpu(ctx, 0, 27000)
    for _ in range(3):
        a.check()
        b.check()


def test_states_stay_for_eager_runs_after_a_capture():
    # the recording has slots of its own: a replay between two runs leaves the
    # kept states alone, and other states in the recording's slots are rebuilt
    w = workloads.config("cultivation_42q", seed=1)
    ctx = make_ctx(w.text, w.noise, seed=5, bits=64)
    ctx.set_noise_mode(1)
    rec = Recording(ctx, 0, 4000)
    rec32 = None
    for bits in (64, 32, 64):
        ctx.set_precision(bits)
        want = run_gpu(ctx, 9, 4000)
        hist = ctx.counters()["support_hist"]
        rec.check()
        if rec32 is None and bits == 32:
            rec32 = Recording(ctx, 9, 4000)
        if rec32 is not None:
            rec32.check()
            rec.check()
        got = run_gpu(ctx, 9, 4000)
        for k in want:
            assert (got[k] == want[k]).all()
        assert ctx.counters()["support_hist"] == hist


def test_traced_replays():
    # a recorded run marks the trace's steps unwritten in every replay: between
    # them another, longer shot is traced into the same buffer
    w = workloads.config("cultivation_15q", seed=1)
    ctx = make_ctx(w.text, NOISE, seed=5)
    n, steps = 200, 48
    ops = run_gpu(ctx, 0, n)["abort_op"]
    short, long = int(np.argmin(ops)), int(np.argmax(ops))

    def trace():
        got = [ctx.read_trace(s) for s in range(steps)]
        return [g is not None for g in got], str(got)

    ctx.set_trace(long, steps)
    run_gpu(ctx, 0, n)
    most = sum(trace()[0])
    ctx.set_trace(short, steps)
    run_gpu(ctx, 0, n)
    want = trace()
    assert 0 < sum(want[0]) < most
    rec = Recording(ctx, 0, n)
    for _ in range(3):
        ctx.set_trace(long, steps)
        run_gpu(ctx, 0, n)
        assert sum(trace()[0]) == most
        rec.check()
        assert trace() == want
