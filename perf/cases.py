"""The work that users of this framework have it do, as measurable cases.

A case is one call of a public entry point on one workload: `call` says which
(a training step, a run of several steps, several independent runs side by side, or
the evaluation on all the data), the other fields are the workload's shape and options.
Shapes come from the five workloads of cada_synth/configs.py, from the settings of the
paper's experiments that they stand for, and from the odd shapes of the tests.

prepare() makes seeded data on the GPU with the distributions of
cada_synth/generators.py (drawn with torch, so that gigabytes take milliseconds), the
engine that a training program keeps, and a schedule of sampled rows; it advances the
engine by a few steps, so that a pass works on a run that is under way: reference points
differ from the iterate, stored gradients are in use and the rule decides.
"""
from __future__ import annotations

import math

import torch

from paper_2012_15469_amd import binding
from paper_2012_15469_amd.binding import Cada

RULES = {"always": 0, "cada1": 1, "cada2": 2, "lag": 3}
WARM_STEPS = 4       # steps in prepare()
SCHEDULE = 16        # sampled minibatches per engine (times the steps of a pass); passes take them in turn


def _case(name, call, dims, M, rows, B, rule, **kw):
    case = {"name": name, "call": call, "model": "mlp" if dims.count("-") else "logreg", "dims": dims, "M": M, "rows": rows, "B": B,
            "rule": rule, "c": 0.5, "D": 100, "steps": 1, "runs": 1, "store": "f32"}
    case.update(kw)
    return case


def listed():
    return [
        # Small logistic workloads, one call per step: the smallest calls, bound by launches and latency.
        # Workload 1 (covtype's width).
        _case("step_p54", "step", "54", 10, 1000, 10, "cada2", D=50),
        # The stochastic LAG baseline on ijcnn1's shape: 1 % of 9170 samples per worker and step.
        _case("step_p22_lag", "step", "22", 10, 9170, 92, "lag"),
        # MNIST's shape, ten workers, 1 % of 6000 samples per worker and step.
        _case("step_p784_b60", "step", "784", 10, 6000, 60, "cada2"),
        # Workload 2, twenty steps per call.
        _case("run_p784", "run", "784", 20, 3000, 32, "cada1", c=1.0, steps=20),
        # Ten Monte-Carlo runs of workload 1 side by side, twenty steps per call (every figure of the paper averages ten runs).
        _case("replicas_p54", "replicas", "54", 10, 1000, 10, "cada2", D=50, steps=20, runs=10),
        # Workload 3: the memory-bound one (fewer rows per worker than its 4096, so that several states fit the card; a
        # step reads 256 of them whatever their number).
        _case("step_p65536", "step", "65536", 100, 1024, 256, "cada2", c=0.3),
        # A high-dimensional workload of odd sizes: rows that start on no 16-byte boundary.
        _case("step_p20001_odd", "step", "20001", 37, 512, 75, "cada1", c=0.3),
        # Networks.  The paper's fully connected layer sizes with its minibatch of 12: small and latency-bound.
        _case("step_mlp_784_b12", "step", "784-500-10", 10, 6000, 12, "cada2", D=50),
        # Workload 4.
        _case("step_mlp_784_b128", "step", "784-512-10", 64, 6000, 128, "cada2"),
        # The distributed Adam baseline (everybody uploads) with odd sizes and the stored gradients kept as bf16.
        _case("step_mlp_odd_always", "step", "617-301-150-26", 24, 1500, 100, "always", store="bf16"),
        # Workload 5.
        _case("step_mlp_3072_b256", "step", "3072-1024-1024-10", 16, 3125, 256, "cada1", D=200),
        # Objective and accuracy of workload 4 on all the data (the y-axes of the paper's figures).
        _case("evaluate_mlp_784", "evaluate", "784-512-10", 64, 6000, 128, "cada2"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges."""
    rule = rng.choice(["cada1", "cada2", "cada1", "cada2", "always", "lag"])
    kind = rng.choice(["small", "small", "wide", "mlp", "mlp", "evaluate"])
    kw = {"c": round(rng.uniform(0.2, 1.0), 2), "D": rng.choice([50, 100, 200])}
    if kind == "small":
        call = rng.choice(["step", "run", "replicas"])
        if call == "step":
            p, M, B = _log(rng, 16, 4000), _log(rng, 4, 100), _log(rng, 8, 256)
        else:        # (workloads that the whole-step kernel serves; replicas need that)
            p, M = _log(rng, 16, 1000), _log(rng, 4, 24)
            B = _log(rng, 8, max(8, min(64, 24000 // p)))
        runs = rng.randint(2, 10) if call == "replicas" else 1
        case = _case("", call, str(p), M, _log(rng, 500, 5000), B, rule, steps=1 if call == "step" else rng.randint(10, 30), runs=runs, **kw)
    elif kind == "wide":
        p = _log(rng, 8192, 131072)
        if rng.random() < 0.6:
            p = p // 4 * 4
        M, B = _log(rng, 8, 100), _log(rng, 24, 256)
        while M * B * p > 1.6e9:
            M, B = max(8, M // 2), max(24, B * 2 // 3)
        case = _case("", "step", str(p), M, B + rng.randint(100, 400), B, rule, **kw)
    else:
        d0, h = _log(rng, 50, 3072), [_log(rng, 32, 1024) for _ in range(rng.randint(1, 2))]
        dims = "-".join(str(d) for d in [d0] + h + [rng.randint(2, 32)])
        M, B = _log(rng, 4, 64), _log(rng, 8, 256)
        while _forward_flops(dims, M * B) > 3e10:
            M, B = max(4, M // 2), max(8, B * 3 // 4)
        rows = _log(rng, 500, 3000)
        if kind == "evaluate" and rng.random() < 0.5:      # the evaluation of a logistic workload
            dims, rule = str(_log(rng, 50, 20000)), rng.choice(["cada1", "cada2"])
        store = "bf16" if dims.count("-") and rule != "lag" and rng.random() < 0.3 else "f32"
        case = _case("", "evaluate" if kind == "evaluate" else "step", dims, M, max(rows, B), B, rule, store=store, **kw)
    del case["name"]
    return case


def _dims(case):
    return [int(d) for d in str(case["dims"]).split("-")]


def _parameters(case):
    d = _dims(case)
    return d[0] if len(d) == 1 else sum(a * b + b for a, b in zip(d, d[1:]))


def _forward_flops(dims, rows):
    d = [int(x) for x in str(dims).split("-")]
    return 2.0 * rows * (d[0] if len(d) == 1 else sum(a * b for a, b in zip(d, d[1:])))


def _data(case, gen):
    """Features [M rows, d0], labels and the initial iterate."""
    d, M, n, dev = _dims(case), case["M"], case["rows"], gen.device
    d0, total = d[0], case["M"] * case["rows"]
    if case["model"] == "mlp":
        X = torch.rand(total, d0, generator=gen, device=dev) if d0 < 1000 else torch.randn(total, d0, generator=gen, device=dev)
        # labels of a random teacher network, one in ten replaced by chance
        a = torch.relu((X - (0.5 if d0 < 1000 else 0.0)) @ (torch.randn(d0, 64, generator=gen, device=dev) / math.sqrt(d0)))
        y = (a @ (torch.randn(64, d[-1], generator=gen, device=dev) / 8.0)).argmax(dim=1)
        chance = torch.randint(d[-1], (total,), generator=gen, device=dev)
        y = torch.where(torch.rand(total, generator=gen, device=dev) < 0.1, chance, y).to(torch.int32)
        parts = []
        for a_, b_ in zip(d, d[1:]):
            parts.append((2 * torch.rand(a_ * b_ + b_, generator=gen, device=dev) - 1) / math.sqrt(a_))
        return X, y, torch.cat(parts)
    if d0 < 200:         # dense features around a mean of each worker's own
        X = torch.randn(M, n, d0, generator=gen, device=dev)
        X += 0.5 * torch.randn(M, 1, d0, generator=gen, device=dev)
    elif d0 < 8192:      # image-like: four of five entries are zero
        X = torch.rand(M, n, d0, generator=gen, device=dev)
        X *= torch.rand(M, n, d0, generator=gen, device=dev) < 0.2
    else:                # rows of norm about one
        X = torch.randn(M, n, d0, generator=gen, device=dev)
        X /= math.sqrt(d0)
        X += torch.randn(M, 1, d0, generator=gen, device=dev) * (0.5 / math.sqrt(d0))
    X = X.view(total, d0)
    score = X @ torch.randn(d0, generator=gen, device=dev)
    score -= score.median()
    y = torch.where(score >= 0, 1.0, -1.0)
    y = torch.where(torch.rand(total, generator=gen, device=dev) < 0.05, -y, y)
    return X, y, torch.zeros(d0, device=dev)


def _engine(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    X, y, theta0 = _data(case, gen)
    M, n, B, mlp = case["M"], case["rows"], case["B"], case["model"] == "mlp"
    engine = Cada(model=case["model"], layer_dims=_dims(case), M=M, B=B, n_samples=[n] * M, X=X, y=y, theta0=theta0,
                  rule=RULES[case["rule"]], D=case["D"], d_max=10, c=case["c"], alpha=0.0005 if mlp else 0.005, beta1=0.9, beta2=0.999,
                  eps=1e-8, lam=0.0 if mlp else 1e-5, gemm_dtype="bf16" if mlp else "fp32", server=1 if case["rule"] == "lag" else 0,
                  whole_steps=case["call"] == "replicas",
                  gradient_store=binding.STORE_BF16 if case["store"] == "bf16" else binding.STORE_F32)
    # distinct rows of every worker for each step
    steps = WARM_STEPS + SCHEDULE * case["steps"]
    sched = torch.stack([torch.rand(M, n, generator=gen, device=dev).argsort(dim=1)[:, :B].to(torch.int32) for _ in range(steps)])
    return engine, sched


def prepare(case, seed):
    engines, warm, schedules = [], [], []
    for r in range(case["runs"]):
        engine, sched = _engine(case, seed * 1000 + r)
        engines.append(engine)
        warm.append(sched[:WARM_STEPS].contiguous())
        steps = sched[WARM_STEPS:].view(SCHEDULE, case["steps"], case["M"], case["B"])
        schedules.append([s.contiguous() for s in (steps[:, 0] if case["call"] == "step" else steps)])
    if case["call"] == "replicas":
        Cada.run_replicas(engines, warm)
    else:
        engines[0].run(warm[0])
    views = [engine.state() for engine in engines]
    outputs = [{name: v[name] for name in ("theta", "h", "vhat", "nabla", "lhs", "tau")} for v in views]
    return {"call": case["call"], "engines": engines, "schedules": schedules, "outputs": outputs, "at": 0}


def run(state):
    """One call of the entry point on the next sampled rows; returns the state that it advanced (views), or the evaluation."""
    engines, call, at = state["engines"], state["call"], state["at"]
    state["at"] = (at + 1) % SCHEDULE
    if call == "evaluate":
        return engines[0].evaluate()
    if call == "step":
        engines[0].step(state["schedules"][0][at])
    elif call == "run":
        engines[0].run(state["schedules"][0][at])
    else:
        Cada.run_replicas(engines, [s[at] for s in state["schedules"]])
    return state["outputs"]


def work(case):
    """Bytes and operations that a pass cannot do without.

    A step: the sampled rows once; each worker's fresh gradient written, the M stored ones read by the aggregate (CADA1:
    the innovations too, bf16 for a network and float32 for the logistic model); the server's vectors.  Operations: two
    gradient evaluations (one where the rule asks for one), each a forward product, a weight gradient of the same size and,
    from the second layer on, an activation gradient.  An evaluation: all rows once through the forward products."""
    d, M, B, p = _dims(case), case["M"], case["B"], _parameters(case)
    mlp = case["model"] == "mlp"
    if case["call"] == "evaluate":
        total = M * case["rows"]
        return {"bytes": 4.0 * total * (d[0] + 1) + 8.0 * p, "flops": _forward_flops(case["dims"], total)}
    grad = 2.0 if case["store"] == "bf16" else 4.0
    byts = 4.0 * M * B * (d[0] + 2) + 2.0 * grad * M * p + 40.0 * p
    if case["rule"] == "cada1":
        byts += (4.0 if mlp else 8.0) * M * p
    evals = 2.0 if case["rule"] in ("cada1", "cada2") else 1.0
    flops = 2.0 * _forward_flops(case["dims"], M * B)
    if mlp:
        flops += 2.0 * M * B * sum(a * b for a, b in zip(d[1:], d[2:]))
    times = case["steps"] * case["runs"]
    return {"bytes": byts * times, "flops": evals * flops * times}


def tolerance(case):
    """About four times what the outputs of a first pass differ by from the algorithm in 64 bits on the same inputs: at most
    7e-7 (2-norm) for the logistic model; 3e-3 for a network (single elements 0.15 of the vector's root mean square: the
    update divides by the root of vhat, so a coordinate whose gradient is below the rounding of the bf16 products takes a
    whole step in either direction), 1.2e-2 and 0.37 with gradients stored as bf16.  An evaluation differs by 3e-7, but
    a sample at a tie between two classes may fall to either side."""
    if case["call"] == "evaluate":
        return {"rel": 2e-6 + 4.0 / (case["M"] * case["rows"])}
    if case["model"] == "logreg":
        return {"rel": 3e-6, "max": 2e-5, "differ": 0.01}
    if case["store"] == "bf16":
        return {"rel": 0.03, "max": 0.9, "differ": 0.01}
    return {"rel": 0.012, "max": 0.6, "differ": 0.01}
