"""The sign pass on the GPU (signs.hip) against the sampler kernel's own walk
of the same shots (checkpoints off, which also leaves the sign pass out): whole
numbers, so equal bit for bit.  Sizes around a wave's lanes, its chunks and the
launch's waves, every vector size and one circuit past the largest, shot
offsets across 2^32, variants that meet inside a chunk (one of them left to the
sampler), null outputs and both noise draws.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads
from paper_2512_23037_amd import soft
from tests.gen_small import random_circuit
from tests.gpu_helpers import make_ctx, run_gpu
from tests.test_signs import with_checks

pytestmark = pytest.mark.gpu

NOISE = {k: 4e-3 for k in ("p1", "p2", "p_idle", "p_meas", "p_reset", "p_mpp")}


def rounds(n_rounds: int, checks: int = 2) -> str:
    """T layers that meet their inverses around parity checks, repeated:
    `checks` records and tests and three T pairs a round."""
    out = ["QUBITS 6", "H 0", "CX 0 1", "CX 0 2"]
    rec = 0
    for _ in range(n_rounds):
        out += ["T 0", "T 1", "TDG 2"]
        for c in range(checks):
            out += ["CX %d %d" % (c, 3 + c), "CX %d %d" % (c + 1, 3 + c), "M %d" % (3 + c), "DETECTOR 0 %d" % rec, "R %d" % (3 + c)]
            rec += 1
        out += ["TDG 0", "TDG 1", "T 2"]
    return "\n".join(out + ["MPP X0*X1*X2", "OBSERVABLE 0 %d" % rec]) + "\n"


def both(build, shot0, n):
    got = []
    for on in (True, False):
        ctx = build()
        ctx.set_shared_prefix(on)
        got.append((run_gpu(ctx, shot0, n), ctx.counters()))
        ctx.close()
    (a, ca), (b, cb) = got
    for k in ("status", "abort_op", "obs", "outcomes"):
        assert (a[k] == b[k]).all(), (k, np.nonzero((a[k] != b[k]).reshape(-1, n).any(axis=0))[0][:5])
    for f in ("shots", "passed", "discarded", "overflow", "numeric", "logical_errors", "restarts"):
        assert ca[f] == cb[f], f
    return a, ca, cb


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n,shot0", [(1, 0), (3, 7), (63, 0), (64, 1), (65, 2**32 - 30), (1023, 5), (4097, 0),
                                     (70001, 2**40 + 3), (400_001, 2**32 - 200_000)])
def test_sizes(n, shot0, mode):
    w = workloads.config("cultivation_15q", seed=1)

    def build():
        ctx = make_ctx(w.text, NOISE, seed=5)
        ctx.set_noise_mode(mode)
        return ctx

    a, ca, cb = both(build, shot0, n)
    if n > 4000:  # most shots need no coefficients
        assert ca["events"] < 0.5 * cb["events"]


@pytest.mark.parametrize("n", [2_000_001, 5_300_007])
def test_few_left_over(n):
    # groups of several reads of 256 statuses, the last one short, with and
    # without shots left in them
    w = workloads.config("cultivation_15q", seed=1)

    def build():
        ctx = make_ctx(w.text, {k: 2e-3 for k in NOISE}, seed=7)
        ctx.set_noise_mode(1)
        return ctx

    a, ca, cb = both(build, 11, n)
    assert 0 < ca["events"] < 0.01 * cb["events"]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n_rounds", [1, 8, 16, 60, 200, 300])
def test_vector_sizes(n_rounds, mode):
    # 3 to 601 records and up to 1500 tests: every vector size, then past the last
    def build():
        ctx = make_ctx(rounds(n_rounds), {k: v / n_rounds for k, v in NOISE.items()}, seed=11)
        ctx.set_noise_mode(mode)
        return ctx

    both(build, 0, 3000)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("p", [1e-6, 0.02, 0.3, 0.75])
def test_rare_and_dense_hits(p, mode):
    # gaps past the last slot and of no slot at all, several hits in a step of
    # one shot, and kinds whose rates differ (candidates that are not accepted)
    def build():
        ctx = make_ctx(rounds(40), {k: p / (1 + i % 3) for i, k in enumerate(NOISE)}, seed=23)
        ctx.set_noise_mode(mode)
        return ctx

    both(build, 9, 5000)


@pytest.mark.parametrize("mode", [0, 1])
def test_variants_meet_inside_a_chunk(mode):
    # a circuit without checks before its first random read of coefficients
    # (left to the sampler) between two that the signs decide
    texts = [rounds(4), "QUBITS 2\nH 0\nT 0\nMPP X0\nDETECTOR 0 0\nH 1\nT 1\nMPP X1\n", rounds(9),
             workloads.config("cultivation_15q", seed=1).text]
    ends = [37, 1500, 1501, 9000]

    def build():
        ctx = soft.Context(0)
        ctx.load_mixture(texts, [NOISE] * 4, ends)
        ctx.set_rng(3)
        ctx.set_noise_mode(mode)
        return ctx

    both(build, 0, 9000)
    both(build, 30, 1475)


@pytest.mark.parametrize("seed", range(24))
def test_random_circuits(seed):
    rng = np.random.default_rng(700 + seed)
    text, _ = random_circuit(61000 + seed, int(rng.integers(2, 9)), int(rng.integers(30, 140)),
                             p_t=0.0 if seed % 3 == 0 else 0.05, p_meas=0.1, p_mpp=0.05, p_reset=0.05,
                             p_msc=0.15 if seed % 2 else 0.0, p_diag=0.03 if seed % 5 == 1 else 0.0,
                             p_if=0.05 if seed % 4 == 2 else 0.0)

    def build():
        ctx = make_ctx(with_checks(text), {**NOISE, "p1": 0.02}, seed=seed, bits=64)
        ctx.set_noise_mode(seed % 2)
        return ctx

    both(build, 11 * seed, 2000)


def test_null_outputs_and_noalloc():
    import torch
    w = workloads.config("cultivation_42q", seed=1)
    ctx = make_ctx(w.text, w.noise, seed=9, bits=32)
    ctx.set_noise_mode(1)
    n = 30_000
    ref = run_gpu(ctx, 4, n)
    st = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    for f in (ctx.run, ctx.run_noalloc):
        st.fill_(-7)
        f(4, n, status=st)
        torch.cuda.synchronize()
        assert (st.cpu().numpy().view(np.uint32) == ref["status"]).all()


def test_states_kept_between_runs():
    # the checkpoint states of a context stay for the runs that follow, on
    # this stream or another; a new precision, pruning threshold, support cap
    # or circuit builds them again
    import torch
    w = workloads.config("cultivation_42q", seed=1)
    N = 20_000

    def fresh(bits, tau, cap, text=w.text):
        ctx = make_ctx(text, w.noise, seed=8, bits=bits, tau=tau, cap=cap, keep=(0, 16))
        out = run_gpu(ctx, 0, N)
        return out, [ctx.read_coeffs(s) for s in range(16)], ctx.counters()["support_hist"]

    ctx = make_ctx(w.text, w.noise, seed=8, bits=64, keep=(0, 16))
    other = workloads.config("cultivation_15q", seed=1).text
    side = torch.cuda.Stream()
    for bits, tau, cap, text in ((64, -1.0, 0, w.text), (64, -1.0, 0, w.text), (32, -1.0, 0, w.text), (32, 1e-3, 0, w.text),
                                 (64, -1.0, 512, w.text), (64, -1.0, 0, w.text), (64, -1.0, 0, other), (64, -1.0, 0, w.text)):
        if text is not w.text or bits == 64:
            ctx.load_circuit(text)
        ctx.set_precision(bits)
        ctx.set_prune(tau)
        ctx.set_caps(cap)
        ref, kept, hist = fresh(bits, tau, cap, text)
        for stream in (None, side, None):
            with torch.cuda.stream(stream or torch.cuda.current_stream()):
                got = run_gpu(ctx, 0, N)
            for k in ("status", "abort_op", "obs", "outcomes"):
                assert (got[k] == ref[k]).all(), (bits, tau, cap, k)
            assert [ctx.read_coeffs(s) for s in range(16)] == kept
            assert ctx.counters()["support_hist"] == hist


def test_captured_runs():
    # soft_run recorded by a stream capture: the replays build their own
    # checkpoint states, whatever other runs of the context left, and those
    # runs build theirs again
    import torch
    w = workloads.config("cultivation_15q", seed=1)
    ctx = make_ctx(w.text, NOISE, seed=5)
    ctx.set_noise_mode(1)
    n = 3001
    ref = run_gpu(ctx, 0, n)
    outs = soft.sample(ctx, 0, n)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        ctx.run(0, n, *outs, stream=torch.cuda.current_stream().cuda_stream)
    for rep in range(3):
        for o in outs:
            o.zero_()
        if rep:  # other states in the slots
            ctx.set_precision(32)
            other = run_gpu(ctx, 0, n)
            ctx.set_precision(64)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        nw = ref["outcomes"].shape[0]
        assert (outs[1].cpu().numpy().view(np.uint32) == ref["status"]).all()
        assert (outs[0].cpu().numpy().view(np.uint32)[:nw] == ref["outcomes"]).all()
        again = run_gpu(ctx, 0, n)
        assert (again["status"] == ref["status"]).all() and (again["outcomes"] == ref["outcomes"]).all()
        if rep:
            ctx.set_precision(32)
            assert (run_gpu(ctx, 0, n)["status"] == other["status"]).all()
            ctx.set_precision(64)


@pytest.mark.parametrize("mode", [0, 1])
def test_record_planes_of_a_longer_variant(mode):
    # a shot that the signs decide has a zero in every record word past its
    # circuit's own, also those that only a variant left to the sampler has
    long = "QUBITS 2\nH 0\nT 0\nMPP X0\n" + "R 1\nX 1\nM 1\n" * 200
    ctx = soft.Context(0)
    ctx.load_mixture([rounds(4), long], [NOISE] * 2, [300, 500])
    ctx.set_rng(3)
    ctx.set_noise_mode(mode)
    got = []
    for on in (True, False):
        ctx.set_shared_prefix(on)
        import torch
        outs = [torch.full((ctx.info()["record_words"], 500), -7, dtype=torch.int32, device="cuda")] + \
            [torch.full((500,), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
        ctx.run(0, 500, *outs)
        torch.cuda.synchronize()
        got.append([o.cpu().numpy() for o in outs] + [ctx.counters()["events"]])
    assert got[0][0].shape[0] > 4 and got[0][4] < got[1][4]
    for a, b in zip(got[0][:4], got[1][:4]):
        assert (a == b).all()


@pytest.mark.parametrize("mode", [0, 1])
def test_signature_tables_past_their_limit(mode):
    # three circuits of 60 000 slots with the largest vectors, 46 MB each of
    # the 134 allowed: the last one is left to the sampler
    # (few hits: the signs decide nearly every shot of the others)
    checks = rounds(100).split("MPP")[0]
    texts = [checks + "H 5\n" * (60_000 + 10 * v) for v in range(3)]

    def build():
        ctx = soft.Context(0)
        ctx.load_mixture(texts, [{k: 1e-5 if k == "p1" else 1e-7 for k in NOISE}] * 3, [700, 1400, 2000])
        ctx.set_rng(3)
        ctx.set_noise_mode(mode)
        return ctx

    both(build, 0, 2000)
    ctx = build()
    run_gpu(ctx, 0, 2000)
    a, b, c = (ctx.counters(v)["events"] for v in range(3))
    assert max(a, b) < 0.02 * c


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n", [4097, 20_481, 163_841, 700_001])
def test_lists_that_the_signs_do_not_decide(n, mode):
    # a share of the shots ends by signs and the sampler runs the rest: groups
    # from a wave's whole share to several for each, in one launch with a
    # variant that is decided to its end
    w = workloads.config("clifford_t_8q", seed=1)

    def build(texts):
        ctx = soft.Context(0)
        ctx.load_mixture(texts, [NOISE] * len(texts), [n * (v + 1) // len(texts) for v in range(len(texts))])
        ctx.set_rng(3)
        ctx.set_noise_mode(mode)
        return ctx

    a, ca, cb = both(lambda: build([w.text]), 0, n)
    assert 0 < ca["events"] < cb["events"]
    both(lambda: build([rounds(4), w.text, workloads.config("cultivation_15q", seed=1).text]), 0, n)
