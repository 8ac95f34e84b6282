"""The sampler's work as its users have it, in cases that can be timed.

A case is one call of a public entry point (Context.run, run_noalloc,
run_list, a launch and its counters) on one circuit, noise rate, coefficient
precision, way of drawing noise and number of shots.  The circuits are the
seeded generators of `workloads` (the configurations that the benchmark, the
scans and the tests run) and two more shapes for what those leave out: random
Clifford+T circuits past 8 qubits, and T gates injected by teleportation with
classically controlled corrections.

Every output is a whole number (records, statuses, abort ops, observables,
counts), so exact() has no value to give.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import workloads
from paper_2512_23037_amd import soft

NOISE = ("p1", "p2", "p_idle", "p_meas", "p_reset", "p_mpp")

# Per-shot work that the oracle counts at the noise rates P_AT: words drawn
# per noise location, words of gap sampling, words of measurements whose
# outcome is drawn.  A sampler that stops a shot at its first failed check
# draws no more than these, and none that gives the same results draws fewer.
P_AT = (2.5e-4, 1e-3, 2e-3)
SLOT_WORDS = {"clifford8": (121, 121, 121), "cult15": (510, 470, 426), "cult42": (3661, 1857, 1347),
              "cult42_k12": (3601, 1858, 1415), "random16": (226, 226, 226), "inject": (184, 184, 184),
              "mixture": (542, 542, 542)}
GAP_WORDS = {"clifford8": (1.1, 1.3, 1.6), "cult15": (1.3, 2.0, 2.9), "cult42": (3.2, 5.8, 7.5),
             "cult42_k12": (3.1, 5.8, 7.8), "random16": (1.1, 1.5, 2.1), "inject": (1.1, 1.3, 1.7),
             "mixture": (2.3, 2.3, 2.3)}
# Coefficients that T gates write and measurements read, where the outcomes
# depend on them: the cultivation circuits' T layers meet their inverses, and
# their records follow from the tableau signs unless noise breaks a pair, so
# they count nothing here.
ENTRIES = {"clifford8": (5, 8), "random16": (1494, 722), "inject": (4358, 6407)}
OPS_PER_WORD, OPS_PER_ENTRY, OPS_PER_T, OPS_PER_M = 25, 8, 8, 5


def inject(seed: int, n: int = 12, layers: int = 4, per_layer: int = 3) -> str:
    """T gates on n qubits by magic-state injection: |T> on an ancilla, CX onto
    it, its measurement and a conditional S, `per_layer` of them in each of
    `layers` random Clifford layers, a random three-qubit Pauli product
    measured after each layer and every qubit at the end."""
    rng = np.random.default_rng(seed)
    a = n
    out = ["QUBITS %d" % (n + 1)] + ["H %d" % q for q in range(n)]
    rec = 0
    for _ in range(layers):
        for q in rng.permutation(n)[:per_layer]:
            out += ["H %d" % a, "T %d" % a, "CX %d %d" % (q, a), "MR %d" % a, "IF %d S %d" % (rec, q)]
            rec += 1
        for _ in range(n):
            x, y = rng.choice(n, size=2, replace=False)
            out += ["CX %d %d" % (x, y), "%s %d" % (("H", "S")[int(rng.integers(2))], int(rng.integers(n)))]
        out.append("MPP " + "*".join("%s%d" % ("XYZ"[int(rng.integers(3))], int(t))
                                     for t in rng.choice(n, size=3, replace=False)))
        rec += 1
    return "\n".join(out + ["M %d" % q for q in range(n)]) + "\n"


def circuit(kind: str, p: float):
    """(text, noise) of one circuit: gate noise on the random ones, the uniform
    circuit-level model on the others."""
    if kind == "clifford8":
        w = workloads.config("clifford_t_8q", p=p)
        return w.text, w.noise
    if kind == "random16":
        w = workloads.random_clifford_t(1, n=16, n_cliff=320, n_t=16, n_meas=16, n_post=2, p=p)
        return w.text, w.noise
    if kind == "inject":
        return inject(1), {k: p for k in NOISE}
    w = workloads.config({"cult15": "cultivation_15q", "cult42": "cultivation_42q",
                          "cult42_k12": "cultivation_42q_k12"}[kind], p=p)
    return w.text, w.noise


def _case(name, kind, shots, bits, gaps, p=1e-3, call="run"):
    c = {"kind": kind, "shots": shots, "bits": bits, "gaps": gaps, "p": p, "call": call}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a program that asks for a few hundred shots at a time inside its own
        # loop, which must not allocate: all latency
        _case("serve_8q_256", "clifford8", 256, 64, False, call="noalloc"),
        # the 8-qubit configuration as it stands: 10^4 shots, FP64, a word per
        # noise location (both defaults)
        _case("run_8q_1e4", "clifford8", 10_000, 64, False),
        # the 15-qubit configuration as it stands (10^6 shots), an odd count
        _case("run_15q_1e6_f64", "cult15", 1_000_003, 64, False),
        # the smallest batch of the throughput sweep
        _case("run_42q_4k_f32", "cult42", 4096, 32, True),
        # a middle batch, FP64
        _case("run_42q_64k_f64", "cult42", 65_537, 64, True),
        # the benchmark's launch
        _case("run_42q_1e7_f32", "cult42", 10_000_000, 32, True),
        # its circuit in FP64, near a million shots
        _case("run_42q_1e6_f64", "cult42", 1_048_613, 64, True),
        # the default noise draw at the rate whose discard rate is the paper's
        _case("run_42q_slots_f32", "cult42", 500_009, 32, False, p=5e-4),
        # the logical-error scan: the span-12 circuit at three rates in one
        # launch, statuses only, each rate's counts read after it
        _case("scan_k12_3e6_f32", "cult42_k12", 3_000_000, 32, True, call="scan"),
        # 27 circuits and rates in one launch
        _case("mixture_2e6_f64", "mixture", 2_000_025, 64, True),
        # circuits without postselection brackets, whose every shot runs to
        # the end on its coefficients
        _case("run_random16_f64", "random16", 100_003, 64, False),
        # injected T gates with conditional corrections
        _case("run_inject_f32", "inject", 50_001, 32, True),
    ]


# Shots and rates of the ranges; the largest numbers keep a case within the
# cost of the largest listed one.
MOST = {"clifford8": 2_000_000, "cult15": 4_000_000, "cult42": 4_000_000, "cult42_k12": 2_000_000,
        "mixture": 4_000_000, "random16": 200_000, "inject": 100_000}


def draw(rng):
    kind = rng.choice(("clifford8", "cult15", "cult42", "cult42", "cult42_k12", "mixture", "random16", "inject"))
    lo, hi = (27 * 64 if kind == "mixture" else 200), MOST[kind]
    shots = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    call = "run"
    if kind == "cult42_k12" and rng.random() < 0.5:
        call = "scan"
    elif kind != "mixture":
        call = rng.choice(("run", "run", "noalloc", "rerun" if kind in ("cult15", "random16") else "run"))
    p = 1e-3 if kind == "mixture" else math.exp(rng.uniform(math.log(P_AT[0]), math.log(P_AT[-1])))
    return _case(None, kind, shots | rng.randrange(2), rng.choice((32, 64)), rng.random() < 0.5, p, call)


def prepare(case, seed):
    """The context with its circuit loaded, and the output tensors; the seed
    gives the random streams' key and, where the shots may start anywhere, the
    first shot's index."""
    n, kind, call = case["shots"], case["kind"], case["call"]
    ctx = soft.Context(0)
    shot0 = 0
    if kind == "mixture":
        m = workloads.mixture(total_shots=n)
        ctx.load_mixture([w.text for w in m["workloads"]], m["models"], m["shot_ends"])
    elif call == "scan":
        rates = [case["p"] / 4, case["p"] / 2, case["p"]]
        text, _ = circuit(kind, case["p"])
        ctx.load_mixture([text] * 3, [{k: r for k in NOISE} for r in rates], [n * (v + 1) // 3 for v in range(3)])
    else:
        text, noise = circuit(kind, case["p"])
        ctx.load_noise(**noise)
        ctx.load_circuit(text)
        shot0 = seed * 7_919 % 1_000_003
    ctx.set_rng(0x5EED0000 + seed)
    ctx.set_precision(case["bits"])
    ctx.set_noise_mode(1 if case["gaps"] else 0)
    if call == "rerun":
        # a cap below the largest support, so that some shots overflow
        ctx.set_caps(1 << max(1, ctx.info()["k_max"] - 1))
    dev = torch.device("cuda", 0)
    words = max(ctx.info()["record_words"], 1)
    state = {"case": case, "ctx": ctx, "shot0": shot0, "shots": n,
             "status": torch.zeros(n, dtype=torch.int32, device=dev)}
    if call != "scan":
        state["outcomes"] = torch.zeros((words, n), dtype=torch.int32, device=dev)
        state["abort_op"] = torch.zeros(n, dtype=torch.int32, device=dev)
        state["obs"] = torch.zeros(n, dtype=torch.int32, device=dev)
    return state


def run(state):
    ctx, n, shot0, call = state["ctx"], state["shots"], state["shot0"], state["case"]["call"]
    if call == "scan":
        # reading the counters waits for the launch, as the scan does per batch
        ctx.run(0, n, status=state["status"])
        out = {"status": state["status"]}
        for v in range(3):
            c = ctx.counters(v)
            out["counts%d" % v] = [int(c[k]) for k in ("shots", "passed", "discarded", "logical_errors")]
        return out
    outs = (state["outcomes"], state["status"], state["abort_op"], state["obs"])
    (ctx.run_noalloc if call == "noalloc" else ctx.run)(shot0, n, *outs)
    out = dict(zip(("outcomes", "status", "abort_op", "obs"), outs))
    if call == "rerun":
        # the shots that passed the cap run again without it
        again = torch.nonzero(state["status"] == soft.OVERFLOW).flatten()
        m = int(again.numel())
        cap = 1 << max(1, ctx.info()["k_max"] - 1)
        second = [torch.zeros((outs[0].shape[0], m), dtype=torch.int32, device="cuda")] + \
            [torch.zeros(m, dtype=torch.int32, device="cuda") for _ in range(3)]
        if m:
            ctx.set_caps(0)
            ctx.run_list(again + shot0, *second)
            ctx.set_caps(cap)
        out.update(zip(("again_outcomes", "again_status", "again_abort_op", "again_obs"), second))
    return out


def _at(table, p):
    """Linear in log p between the rates of P_AT, the ends' values outside."""
    return float(np.interp(math.log(p), [math.log(x) for x in P_AT], table))


def work(case):
    """Bytes: the outputs, each written once.  Operations: the words of the
    random streams that the draws take and, where outcomes depend on them,
    the coefficients that T gates write and measurements read."""
    kind, n = case["kind"], case["shots"]
    words = {"clifford8": 1, "cult15": 1, "cult42": 3, "cult42_k12": 3, "random16": 1, "inject": 1, "mixture": 1}[kind]
    per_shot = 4 if case["call"] == "scan" else 4 * (3 + words)
    rates = [case["p"] / 4, case["p"] / 2, case["p"]] if case["call"] == "scan" else [case["p"]]
    table = (GAP_WORDS if case["gaps"] else SLOT_WORDS)[kind]
    drawn = sum(_at(table, r) for r in rates) / len(rates)
    t, m = ENTRIES.get(kind, (0, 0))
    ops = OPS_PER_WORD * drawn + (OPS_PER_ENTRY + OPS_PER_T) * t + (OPS_PER_ENTRY + OPS_PER_M) * m
    return {"bytes": n * per_shot, "flops": int(n * ops)}


def exact(case, seed):
    """Whole numbers only: nothing that 64 bits would give more exactly."""
    return None
