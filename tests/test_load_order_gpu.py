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
