"""The sketched-AMSGrad step as its users run it: the cases a change to the kernels has to be timed on.

Three kinds of case ("op"):

  step    one whole iteration: sketch_accumulate, sketch_reduce, unsketch_topk, gather_topk, topk_refine when more
          candidates than k are taken (P > 1), and the update, which also runs the dense head of the next iteration.
          "pa": parameter averaging (Alg. 1, per-worker second moments) instead of gradient averaging (Alg. 2).
          "fuse_head" and "stage_spread" are the library's tunables of those names: 0 is the library's default, 2 and 1
          are what the benchmark runs with.
  sketch  the sketch operators by themselves: accumulate, mean, and the estimate of every coordinate, with a table
          so small beside the vector that the library adds its rows up in LDS.
  refine  the context-free second-round selection of topk_refine_static.

A state is what a training program holds between two iterations: the context (hashes and plan), the caller's buffers and
two batches of gradients that take turns.  Gradients have the distributions of paper_2210_07454_amd.inputs.
"""
import dataclasses
import itertools
import math

import numpy as np
import torch

from paper_2210_07454_amd import inputs, sams

# the recipes of gradient values (noise, layer segments, heavy coordinates), by the workload that they come from
RECIPES = ("C1", "C2", "C3", "C4", "P1", "P2a")
# the sketch of a vector longer than this keeps the order of its additions only if the table exceeds one LDS window
ORDERED_ANY_TABLE_MAX_D = 1 << 22
LDS_WINDOW = 1 << 15


def _step(name, recipe, d, n, r, c, k, P=1, pa=False, fuse_head=0, stage_spread=0):
    return {"name": name, "op": "step", "recipe": recipe, "d": d, "n": n, "r": r, "c": c, "k": k, "P": P, "pa": pa,
            "fuse_head": fuse_head, "stage_spread": stage_spread}


def listed():
    return [
        # a model of tens of thousands of parameters: launches and latencies
        _step("step-tiny", "C1", 65_536, 4, 5, 2_048, 256),
        # the paper's federated experiment: a small network, many workers, a sketch of 400 columns
        _step("step-small-n50", "P2a", 60_000, 50, 5, 400, 500),
        # the same with 100 workers, by parameter averaging and with four candidates for every selected coordinate
        _step("pa-small-n100-p4", "P2a", 60_000, 100, 5, 400, 500, P=4, pa=True),
        # parameter counts as they come: odd, a table that is no power of two, an even number of rows
        _step("step-ragged-431k", "C2", 431_003, 5, 4, 9_001, 4_311),
        _step("step-ragged-3m", "C2", 2_999_999, 8, 5, 150_001, 30_001),
        # a convolutional network of 11 million parameters, as the benchmark runs it and as the library's defaults do
        _step("step-11m", "C2", 11_200_000, 8, 5, 262_144, 50_000, fuse_head=2, stage_spread=1),
        _step("pa-11m-p4", "C2", 11_200_000, 8, 5, 262_144, 50_000, P=4, pa=True),
        # 25 million parameters: many workers and a large table; the paper's own table (10 rows of 100,000, P = 8)
        _step("step-26m", "C3", 25_600_000, 16, 7, 1_048_576, 100_000, fuse_head=2, stage_spread=1),
        _step("step-25m-r10-p8", "P1", 25_000_000, 16, 10, 100_000, 50_000, P=8, fuse_head=2),
        # a language model of 124 million parameters: the benchmark's workload
        _step("step-124m", "C4", 124_000_000, 8, 5, 4_194_304, 1_240_000, fuse_head=2, stage_spread=1),
        # a strongly compressing sketch of a long vector
        {"name": "sketch-narrow", "op": "sketch", "recipe": "C3", "d": 25_600_000, "n": 4, "r": 5, "c": 10_000},
        # the candidates of a large model's second round
        {"name": "refine-5m", "op": "refine", "k_in": 4_960_000, "k_out": 1_240_000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.random()
    if kind < 0.1:
        k_in = _log(rng, 2_000, 4_960_000)
        return {"op": "refine", "k_in": k_in, "k_out": max(1, k_in // rng.choice((2, 4, 8)))}
    if kind < 0.2:
        d = _log(rng, ORDERED_ANY_TABLE_MAX_D + 1, 25_600_000)
        return {"op": "sketch", "recipe": rng.choice(RECIPES), "d": d, "n": rng.randint(1, 8), "r": rng.randint(3, 5),
                "c": _log(rng, 400, LDS_WINDOW)}
    d = _log(rng, 50_000, 124_000_000)
    r = rng.choice((3, 4, 5, 5, 5, 7, 10) if d < 60_000_000 else (3, 4, 5, 5, 5))
    pa = rng.random() < 0.25
    # workers: dozens for small models, fewer for large ones; n * d and n * r * d stay below the largest listed case's
    most = min(100, int(990_000_000 // (d * (2 if pa else 1))), int(4_900_000_000 // (r * d)))
    n = _log(rng, 2, most) if most > 2 else 2
    c = max(400, int(d / math.exp(rng.uniform(math.log(24), math.log(160)))))
    if d > ORDERED_ANY_TABLE_MAX_D:
        c = max(c, LDS_WINDOW + rng.randint(1, 1_000))
    k = max(16, int(d * math.exp(rng.uniform(math.log(0.002), math.log(0.01)))))
    if rng.random() < 0.5:                       # tensors whose sizes are multiples of eight, as most layers' are
        d = (d + 7) // 8 * 8
    case = _step("", rng.choice(RECIPES), d, n, r, c, k, P=rng.choice((1, 1, 1, 4)), pa=pa,
                 fuse_head=rng.choice((0, 2)))
    del case["name"]
    return case


def _workload(case):
    w = inputs.WORKLOADS[case["recipe"]]
    return dataclasses.replace(w.scaled(case["d"]), d=case["d"], n=case["n"], r=case["r"], c=case["c"],
                               k=case.get("k", 1))


def _context(w, hp, k, **tunables):
    for key, value in tunables.items():
        sams.sams_configure(key, value)
    try:
        return sams.Context(w.d, w.n, w.r, w.c, k, hp)
    finally:
        for key in tunables:
            sams.sams_configure(key, 0)


class _Step:
    """A training run between two iterations."""

    def __init__(self, case, seed):
        w = self.w = _workload(case)
        gs = inputs.GradientStream(w, device="cuda", seed=seed)
        candidates = case["P"] * w.k
        self.pa, self.P = case["pa"], case["P"]
        self.ctx = _context(w, inputs.hash_params(w.r, seed=seed), candidates, fuse_head=case["fuse_head"],
                            stage_spread=case["stage_spread"])
        self.b = sams.Buffers(w.d, w.n, w.r, w.c, candidates, w.eps, gs.x1())
        if self.pa:
            self.v_w = torch.full((w.n, w.d), w.eps, device="cuda")
            self.vhat_w = torch.full((w.n, w.d), w.eps, device="cuda")
        self.idx, self.delta = self.b.idx, self.b.delta
        if self.P > 1:
            self.idx = torch.empty(w.k, device="cuda", dtype=torch.int32)
            self.delta = torch.empty(w.k, device="cuda")
        self.batches = itertools.cycle([gs.step(t) for t in range(2)])
        self.update(None, None, 0)               # the head of the first iteration

    def update(self, idx, delta, k):
        w, b, g = self.w, self.b, next(self.batches)
        if self.pa:
            self.ctx.amsgrad_ef_update_pa(g, b.m, b.e_u, self.v_w, self.vhat_w, b.x, idx, delta, k, w.beta1, w.beta2, w.lr)
        else:
            self.ctx.amsgrad_ef_update(g, b.m, b.e_u, b.v, b.vhat, b.x, idx, delta, k, w.beta1, w.beta2, w.lr)

    def run(self):
        ctx, b = self.ctx, self.b
        vhat = None if self.pa else b.vhat
        ctx.sketch_accumulate(b.e_u, b.S_workers)
        ctx.sketch_reduce(b.S_workers, b.S_mean)
        ctx.unsketch_topk(b.S_mean, vhat, b.idx, None)
        ctx.gather_topk(b.e_u, vhat, b.idx, b.U_workers, b.delta)
        if self.P > 1:
            ctx.topk_refine(b.idx, b.delta, self.w.k, self.idx, self.delta)
        self.update(self.idx, self.delta, self.w.k)
        out = {"S_workers": b.S_workers, "S_mean": b.S_mean, "idx": self.idx, "delta": self.delta,
               "U_workers": b.U_workers, "m": b.m, "e_u": b.e_u, "x": b.x}
        if self.P > 1:
            out.update(candidates=b.idx, candidate_delta=b.delta)
        if self.pa:
            out.update(v=self.v_w, vhat=self.vhat_w)
        else:
            out.update(v=b.v, vhat=b.vhat)
        return out


class _Sketch:
    """Vectors to sketch, a table for every worker, and the second moments that scale the estimates."""

    def __init__(self, case, seed):
        w = _workload(case)
        gs = inputs.GradientStream(w, device="cuda", seed=seed)
        self.ctx = _context(w, inputs.hash_params(w.r, seed=seed), 1)
        self.u = gs.step(0)
        self.vhat = gs.worker(1, 0).square_().clamp_(min=w.eps)
        self.S_workers = torch.empty((w.n, w.r, w.c), device="cuda")
        self.S_mean = torch.empty((w.r, w.c), device="cuda")
        self.est = torch.empty(w.d, device="cuda")

    def run(self):
        self.ctx.sketch_accumulate(self.u, self.S_workers)
        self.ctx.sketch_reduce(self.S_workers, self.S_mean)
        self.ctx.unsketch_estimates(self.S_mean, self.vhat, self.est)
        return {"S_workers": self.S_workers, "S_mean": self.S_mean, "est": self.est}


class _Refine:
    """Candidates in ascending order with their exact averaged values, which are heavy-tailed."""

    def __init__(self, case, seed):
        k_in, self.k_out = case["k_in"], case["k_out"]
        gen = torch.Generator(device="cuda").manual_seed(seed)
        gaps = torch.randint(1, 50, (k_in,), generator=gen, device="cuda", dtype=torch.int32)
        self.idx_in = torch.cumsum(gaps, 0, dtype=torch.int32)
        z = torch.randn(k_in, generator=gen, device="cuda")
        self.delta_in = z / torch.rand(k_in, generator=gen, device="cuda").clamp_(min=1e-6).pow_(1 / 1.5)
        self.idx_out = torch.empty(self.k_out, device="cuda", dtype=torch.int32)
        self.delta_out = torch.empty(self.k_out, device="cuda")

    def run(self):
        sams.topk_refine_static(self.idx_in, self.delta_in, self.k_out, self.idx_out, self.delta_out)
        return {"idx": self.idx_out, "delta": self.delta_out}


def prepare(case, seed):
    return {"step": _Step, "sketch": _Sketch, "refine": _Refine}[case["op"]](case, int(np.uint32(seed)))


def run(state):
    return state.run()


def work(case):
    """Inputs read once and outputs written once; a flop is an addition, multiplication, division or square root."""
    if case["op"] == "refine":
        return {"bytes": 8 * case["k_in"] + 8 * case["k_out"], "flops": 0}
    d, n, r, c = case["d"], case["n"], case["r"], case["c"]
    tables = 4 * (n + 1) * r * c
    if case["op"] == "sketch":
        return {"bytes": 4 * n * d + tables + 8 * d, "flops": n * r * d + (n + 1) * r * c + 2 * d}
    k, P = case["k"], case["P"]
    # g read, m and e read and written; v read and written and vhat read (per worker, and vhat written, with pa)
    dense = 36 * n * d if case["pa"] else 20 * n * d + 12 * d
    sparse = P * k * (4 * n + 8) + (8 * k if P > 1 else 0) + 8 * k   # U_workers, idx, delta; the refined pair; x
    flops = n * r * d + (n + 1) * r * c + (12 if case["pa"] else 5) * n * d + (0 if case["pa"] else 6) * d + P * k * (n + 2)
    return {"bytes": dense + tables + sparse, "flops": flops}


def tolerance(case):
    # The rows that are added up in LDS come in no fixed order: 32-bit sums of some thousand terms.  Everything else is
    # defined to the bit (terms added in coordinate order, ties to the smaller coordinate), indices included.
    return {"rel": 1e-5} if case["op"] == "sketch" else "exact"
