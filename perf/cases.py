"""The work that a user of the lock-step sampler has it do, as cases that can be timed and compared.

A case is one call of a public entry point on data that is resident before the call: `nuts_sample` (the sampler, on
each target family, dtype, sampler form and schedule) or `pcvm_run` (the program-counter virtual machine).  What is
made in `prepare` is what a sampling program holds before it samples: the target (uploaded and re-laid-out once), the
starting points if it goes on from an earlier run, and the options of the call.

`listed()` are fixed cases over the range; `draw(rng)` gives further ones of the same ranges.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1910_11141_amd as nuts
from paper_1910_11141_amd import pcvm, pcvm_programs, workloads

DTYPES = {"f32": np.float32, "f64": np.float64}


def _logreg(name, dtype, n, d, chains, iters, *, eps=None, start="prior", depth=10, leaf_steps=1, sampler=0, schedule=0):
    """Bayesian logistic regression: n data rows, d - 1 features and an intercept, prior N(0, I).  The step size follows
    the posterior's width, which shrinks with the square root of the number of rows.  start = "posterior": the call
    goes on from points of an earlier run (a sampler that emits its samples block by block)."""
    return {"name": name, "path": "logreg", "dtype": dtype, "n": n, "d": d, "chains": chains, "iters": iters,
            "eps": eps if eps is not None else min(0.2, 1.5 / math.sqrt(n)), "start": start, "depth": depth,
            "leaf_steps": leaf_steps, "sampler": sampler, "schedule": schedule}


def _gauss(name, form, dtype, d, chains, iters, *, eps, depth=10, leaf_steps=1, sampler=0, schedule=0):
    """Gaussian targets.  form: "std" standard normal, "diag" independent scales over four decades, "ar1" correlation
    0.9^|i-j| (a tridiagonal precision matrix), "spd" a full, well-conditioned precision matrix."""
    return {"name": name, "path": "gauss", "form": form, "dtype": dtype, "d": d, "chains": chains, "iters": iters,
            "eps": eps, "start": "prior", "depth": depth, "leaf_steps": leaf_steps, "sampler": sampler,
            "schedule": schedule}


def _machine(name, program, batch, *, queued, policy, top):
    """A batch of executions of one program of the virtual machine; `top` bounds the inputs."""
    return {"name": name, "path": "machine", "program": program, "batch": batch, "queued": queued, "policy": policy,
            "top": top}


def listed():
    return [
        # the smallest call: four chains of a two-dimensional standard normal, where only latency counts
        _gauss("normal_d2_4ch", "std", "f64", 2, 4, 100, eps=0.5, depth=6),
        # one analyst's regression with the four chains that diagnostics want
        _logreg("logreg_1000x25_4ch", "f64", 1000, 25, 4, 100, eps=0.05),
        # the headline workload (200 of its 1000 iterations)
        _logreg("logreg_1000x25_4096ch", "f64", 1000, 25, 4096, 200, eps=0.05),
        # more features than the headline workload, sampled block by block
        _logreg("logreg_5000x60_512ch", "f64", 5000, 60, 512, 10, start="posterior"),
        # a small data set of odd size in binary32, with the published sampler and its four steps per leaf
        _logreg("logreg_700x17_f32_slice", "f32", 700, 17, 250, 50, start="posterior", leaf_steps=4, sampler=1),
        # many data rows, few chains (four of the workload's 200 iterations)
        _logreg("logreg_100000x100_256ch", "f32", 100000, 100, 256, 4, eps=0.005),
        # the shape and the settings of the published experiment: 10 000 x 100, slice sampler, four steps per leaf
        _logreg("logreg_10000x100_slice", "f32", 10000, 100, 1024, 4, eps=0.015, leaf_steps=4, sampler=1),
        # a correlated Gaussian with a banded precision matrix (100 of the workload's 1000 iterations)
        _gauss("ar1_d100_1024ch", "ar1", "f64", 100, 1024, 100, eps=0.1),
        # a correlated Gaussian with a full precision matrix and many chains
        _gauss("spd_d100_4096ch", "spd", "f64", 100, 4096, 100, eps=0.1),
        # the same family with more dimensions, fewer chains, and every iteration awaited by all chains
        _gauss("spd_d250_300ch_sync", "spd", "f64", 250, 300, 10, eps=0.1, schedule=1),
        # an ill-conditioned diagonal Gaussian, the most chains (8 of the workload's 500 iterations)
        _gauss("diag_d1000_16384ch", "diag", "f32", 1000, 16384, 8, eps=0.01),
        # the virtual machine on its worked example, members taken from a queue
        _machine("fibonacci_200000", "fibonacci", 200000, queued=True, policy=1, top=18),
    ]


def _between(rng, lo, hi):
    """A whole number whose logarithm is uniform."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


#: Leapfrog steps of an iteration, as measured; they only size the drawn cases and `work`.  (Longer leaves make
#: trees with fewer of them.)
def _leaps(case):
    if case["path"] == "logreg":
        return 10.0 if case["leaf_steps"] == 1 else 15.0
    if case["form"] == "std":
        return 3.0 / case["eps"]
    return {"diag": 500.0, "ar1": 90.0, "spd": 30.0}[case["form"]]


def _flops_per_step(case):
    """Of one leapfrog step of one chain: the target's gradient and the updates."""
    d = case["d"]
    if case["path"] == "logreg":
        return 4.0 * case["n"] * d
    if case["form"] == "spd":
        return 2.0 * d * d
    return 14.0 * d if case["form"] == "ar1" else 8.0 * d


def draw(rng):
    kind = rng.choice(["logreg", "logreg", "logreg", "gauss", "gauss", "machine"])
    if kind == "machine":
        program, top = rng.choice([("fibonacci", 18), ("collatz_steps", 5000), ("gcd", 10 ** 9), ("binomial", 10)])
        queued = rng.random() < 0.5
        c = _machine("", program, _between(rng, 500, 200000), queued=queued, policy=int(queued and rng.random() < 0.5),
                     top=top)
        c.pop("name")
        return c
    more = {"leaf_steps": rng.choice([1, 1, 4]), "sampler": rng.choice([0, 0, 1]), "schedule": rng.choice([0, 0, 0, 1])}
    if kind == "logreg":
        dtype = rng.choice(["f32", "f64"])
        d = _between(rng, 3, 128)
        n = _between(rng, 100, 100000 if dtype == "f32" else min(30000, 1500000 // d))
        chains = _between(rng, 4, 4096)
        c = _logreg("", dtype, n, d, chains, 1, start=rng.choice(["prior", "posterior"]), **more)
        budget, one_chain = 4e10, 6e7
    else:
        form = rng.choice(["std", "diag", "ar1", "spd", "spd"])
        dtype = rng.choice(["f32", "f64"])
        d = _between(rng, 2, 320) if form == "spd" else _between(rng, 2, 2000)
        eps = {"std": 0.3, "diag": 0.02, "ar1": 0.1, "spd": 0.1}[form]
        c = _gauss("", form, dtype, d, _between(rng, 4, 4096), 1, eps=eps, **more)
        budget, one_chain = 2e10, 2e7
    # a pass stays within a fraction of a second: a bound on what all chains do, and on what one does, which is serial
    per_iteration = _leaps(c) * _flops_per_step(c)
    c["chains"] = max(4, min(c["chains"], int(budget / per_iteration)))
    c["iters"] = max(1, min(40, int(one_chain / per_iteration), int(budget / (per_iteration * c["chains"]))))
    c.pop("name")
    return c


class _Sampling:
    """What a sampling program holds before a call."""

    def __init__(self, target, case, seed, init):
        self.target, self.case, self.seed, self.init = target, case, seed, init


class _Machine:
    def __init__(self, program, inputs, depth, case):
        self.program, self.inputs, self.depth, self.case = program, inputs, depth, case


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    if case["path"] == "machine":
        program, b, top = pcvm_programs.ALL[case["program"]](), case["batch"], case["top"]
        if case["program"] == "gcd":
            x = rng.integers(0, top, size=(2, b))
        elif case["program"] == "binomial":
            n = rng.integers(0, top + 1, size=b)
            x = np.stack([n, (rng.random(b) * (n + 1)).astype(np.int64)])
        else:
            x = rng.integers(1, top + 1, size=(1, b))
        return _Machine(program, torch.from_numpy(np.ascontiguousarray(x, dtype=np.int64)).cuda(), 64, case)
    dtype, d, init = DTYPES[case["dtype"]], case["d"], None
    if case["path"] == "logreg":
        n = case["n"]
        X, y, w = workloads.logreg_data(n, d, 1.0 if d <= 32 else 0.5, rng, standardize=n <= 5000)
        target = nuts.Target(nuts.NUTS_TARGET_LOGISTIC_REGRESSION, d, dtype, X=X, y=y)
        if case["start"] == "posterior":
            pts = w + case["eps"] * rng.standard_normal((case["chains"], d))
            init = torch.from_numpy(pts.astype(dtype)).cuda()
    elif case["form"] == "std":
        target = nuts.Target(nuts.NUTS_TARGET_STD_NORMAL, d, dtype)
    elif case["form"] == "diag":
        target = nuts.Target(nuts.NUTS_TARGET_GAUSS_DIAG, d, dtype, scales=10.0 ** (-2.0 + 4.0 * rng.random(d)))
    else:
        P = workloads.ar1_precision(d, 0.9) if case["form"] == "ar1" else workloads.random_spd_precision(d, seed)
        target = nuts.Target(nuts.NUTS_TARGET_GAUSS_DENSE_PRECISION, d, dtype, precision=P)
    return _Sampling(target, case, int(rng.integers(1 << 62)), init)


def run(state):
    c = state.case
    if c["path"] == "machine":
        out, _, _ = pcvm.pcvm_run(state.program, state.inputs, state.depth, queued=c["queued"], policy=c["policy"])
        return out
    return nuts.nuts_sample(state.target, c["chains"], c["iters"], c["eps"], c["depth"], state.seed,
                            init_states=state.init, leaf_steps=c["leaf_steps"], sampler=c["sampler"],
                            schedule=c["schedule"])


def work(case):
    """Bytes: the target's data and the starting points read once, the outputs written once.  Operations: those of the
    leapfrog steps that an iteration of such a target takes on average (the virtual machine has none in floating point)."""
    if case["path"] == "machine":
        inputs = 2 if case["program"] in ("gcd", "binomial") else 1
        return {"bytes": 8.0 * (inputs + 1) * case["batch"], "flops": 0.0}
    size, d, chains, iters = (4 if case["dtype"] == "f32" else 8), case["d"], case["chains"], case["iters"]
    data = {"logreg": (case.get("n", 0) * (d + 1)) * size}.get(case["path"])
    if data is None:
        data = {"std": 0, "diag": d, "ar1": d * d, "spd": d * d}[case["form"]] * size
    start = chains * d * size if case["start"] == "posterior" else 0
    return {"bytes": float(data + start + iters * chains * (d * size + 8)),
            "flops": float(chains) * iters * _leaps(case) * _flops_per_step(case)}


def tolerance(case):
    """What another correct order of the same sums shows, measured between this framework's kernels on the listed cases
    and on odd shapes (the general kernel sums in binary64 throughout).  Binary64: states within 4e-15 (largest 1.1e-14)
    of each other up to 1000 rows, more with more terms, and the same trees.  Binary32 Gaussians: every decision is taken
    on binary64 sums of the same binary32 values, so at most the last bit of a state moves.  Binary32 logistic
    regression: 1e-7 (largest 1.3e-5) as long as no decision falls within rounding of its threshold; in 3 runs of 25 one
    did, and that chain then goes another, equally valid way (0.1 % of the trees, 5e-3 of the norm, single
    components by their posterior width)."""
    if case["path"] == "machine":
        return "exact"
    if case["dtype"] == "f64":
        return {"rel": 1e-12}
    if case["path"] == "gauss":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 2e-2, "max": 0.99, "differ": 0.005}
