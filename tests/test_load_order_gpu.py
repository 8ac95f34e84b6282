"""A load while the context's last run is still executing on a stream of its
own: the load waits for it, so the run reads the tables it was launched with.
"""
from __future__ import annotations

import pytest

import workloads
from paper_2512_23037_amd import soft
from tests.gpu_helpers import make_ctx, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
def test_load_waits_for_the_last_run(noalloc):
    import numpy as np
    import torch
    w, other = (workloads.config(c, seed=1) for c in ("cultivation_42q", "cultivation_15q"))
    ctx = make_ctx(w.text, w.noise, seed=5)
    ctx.set_shared_prefix(False)  # the sampler's own walk: some 40 ms
    n = 1_500_000
    ref = run_gpu(ctx, 0, n)
    outs = soft.sample(ctx, 0, n)
    for o in outs:
        o.fill_(-7)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    (ctx.run_noalloc if noalloc else ctx.run)(0, n, *outs, stream=side.cuda_stream)
    ctx.load_circuit(other.text)
    assert side.query()  # nothing of the run is left
    torch.cuda.synchronize()
    for o, k in zip(outs, ("outcomes", "status", "abort_op", "obs")):
        assert (o.cpu().numpy().view(np.uint32)[: ref[k].shape[0]] == ref[k]).all(), k


@pytest.mark.parametrize("noalloc", [False, True])
def test_counters_after_a_load_are_the_last_runs(noalloc):
    # other numbers of variants, each with other counter rows a variant
    import torch
    w = workloads.config("cultivation_15q", seed=1)
    ctx = make_ctx(w.text, w.noise, seed=5)
    rates = [{**w.noise, "p1": 1e-4 * v} for v in range(64)]
    st = torch.zeros(64_000, dtype=torch.int32, device="cuda")

    def load(m):
        if m == 1:
            ctx.load_circuit(w.text)
        else:
            ctx.load_mixture([w.text] * m, rates[:m], [1000 * (v + 1) for v in range(m)])

    def run(m, n):
        load(m)
        (ctx.run_noalloc if noalloc else ctx.run)(0, n, status=st)

    for m, n in ((1, 3000), (64, 64_000), (27, 27_000), (3, 3000)):
        run(m, n)
        total, each = ctx.counters(), [ctx.counters(v) for v in range(m)]
        assert total["shots"] == n and [e["shots"] for e in each] == [n // m] * m
        for other in (64, 5, 1, m):
            load(other)
            assert ctx.counters() == total
            for v in range(other):
                got = ctx.counters(v)
                if v < m:
                    assert got == each[v]
                else:
                    assert not any(got["support_hist"]) and not any(x for f, x in got.items() if f != "support_hist")
            with pytest.raises(soft.SoftError, match="no such variant"):
                ctx.counters(other)
