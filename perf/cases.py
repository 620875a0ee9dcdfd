"""Performance cases: what a program built on this framework asks of it, through the public
entry points of paper_2501_03944_amd.mgfwa (MGFWA.step / evaluate / ask / tell, Batch.step).

A case is a dict of plain values; `kind` says which call it stands for:

* step      generations of one optimisation job whose sparks are an MLP's weights (the method's
            main loop: explosion, fitness, guiding, fitness, selection, loser-out)
* net       generations of one job whose sparks are the input of a fixed MLP (the paper's testbed)
* evaluate  the fitness of weight vectors that the caller holds
* ask_tell  one generation whose fitness the caller computes itself
* batch     one generation of many jobs of uneven shape advanced together

Network shapes, population sizes, sample counts and data distributions are those of the
workloads in paper_2501_03944_amd/inputs.py and of the tests, or random ones of the same kind.
"""
import math

import numpy as np
import torch

from paper_2501_03944_amd import inputs
from paper_2501_03944_amd import mgfwa

LB, UB = -5.0, 5.0
STATE = ("F", "A", "Y", "Yc", "best_x", "best_y")


def _step(name, net, act, loss, samples, precision, fireworks, sparks, guiding, generations=1,
          populations=1, map_range=False, lag_guiding=False, regen_sparks=False):
    return dict(name=name, kind="step", net=net, act=act, loss=loss, samples=samples,
                precision=precision, populations=populations, fireworks=fireworks, sparks=sparks,
                guiding=guiding, generations=generations, map_range=map_range,
                lag_guiding=lag_guiding, regen_sparks=regen_sparks)


def _net(name, widths, act, fireworks=8, sparks=512, guiding=8, generations=1):
    return dict(name=name, kind="net", net=widths, act=act, fireworks=fireworks, sparks=sparks,
                guiding=guiding, generations=generations)


def _evaluate(name, net, acts, loss, samples, precision, rows):
    return dict(name=name, kind="evaluate", net=net, act=acts, loss=loss, samples=samples,
                precision=precision, rows=rows)


def _testbed(net_id):
    _, act, d, h, k = inputs.TESTBED_NETS[net_id]
    return "-".join(str(w) for w in (d,) + (h,) * (k + 1) + (1,)), act


def listed():
    net6, act6 = _testbed(6)
    net12, act12 = _testbed(12)
    return [
        # a small regression: ten generations between two looks at the best
        _step("step 8-16-1", "8-16-1", "tanh", "mse", 256, "fp32", 4, 32, 4, generations=10),
        # an ordinary classifier on mixture data, in both fitness precisions
        _step("step 64-128-128-10 fp32", "64-128-128-10", "relu", "ce", 4096, "fp32", 8, 256, 4),
        _step("step 64-128-128-10 bf16", "64-128-128-10", "relu", "ce", 4096, "bf16", 8, 256, 4),
        # a first layer too wide for the LDS on sparse 28 x 28 inputs: the largest jobs
        _step("step 784-256-10 fp32", "784-256-10", "relu", "ce", 8192, "fp32", 16, 256, 4),
        _step("step 784-256-10 bf16", "784-256-10", "relu", "ce", 8192, "bf16", 16, 256, 4),
        # the paper's testbed: a medium and the largest network
        _net("net 100-128x8", net6, act6),
        _net("net 2000-512x11", net12, act12),
        # candidates scored outside the loop: many on an uneven deep network, a few on a wide one
        _evaluate("evaluate 17-40-33-20-3", "17-40-33-20-3", "relu,identity,tanh", "ce", 1029,
                  "fp32", 2500),
        _evaluate("evaluate 64-128-128-10", "64-128-128-10", "relu,relu", "ce", 4096, "fp32", 300),
        _evaluate("evaluate 784-256-10", "784-256-10", "relu", "ce", 8192, "fp32", 37),
        # the caller's own black box over spark positions
        dict(name="ask tell 26122", kind="ask_tell", dim=26122, fireworks=8, sparks=256, guiding=4),
        # many jobs of uneven shape, tuned, advanced by one launch per generation
        dict(name="batch of 32", kind="batch", jobs=32, mix=1004, precision="bf16", generations=1),
    ]


# ---- drawn cases ------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _population(rng, big):
    guiding = rng.choice((1, 2, 4, 8))
    group = _log_int(rng, 4, 64 if big else 32)
    return rng.randint(2, 16 if big else 8), guiding * group, guiding


def _options(rng):
    pick = rng.random()
    return dict(map_range=pick < 0.15, lag_guiding=0.15 <= pick < 0.25,
                regen_sparks=0.25 <= pick < 0.4)


def _draw_net(rng):
    """(widths, activations, loss, samples) of a weights problem."""
    what = rng.random()
    if what < 0.25:      # small regressions
        h = _log_int(rng, 8, 64)
        widths = (rng.randint(2, 24),) + (h,) * rng.randint(1, 2) + (rng.randint(1, 3),)
        return widths, rng.choice(("tanh", "relu", "gelu")), "mse", _log_int(rng, 33, 2048)
    if what < 0.75:      # classifiers, one to three hidden layers
        depth = rng.choice((1, 1, 2, 2, 2, 3))
        top = 256 if depth == 1 else 224 if depth == 2 else 128
        h = _log_int(rng, 32, top)
        widths = (rng.choice((16, 30, 32, 64, 96)),) + (h,) * depth + (rng.choice((2, 10, 10, 16)),)
        return widths, rng.choice(("relu", "relu", "relu", "tanh")), "ce", _log_int(rng, 256, 8192)
    widths = (_log_int(rng, 256, 1024), _log_int(rng, 128, 256), rng.choice((2, 10, 10, 16)))
    return widths, "relu", "ce", _log_int(rng, 512, 8192)


def draw(rng):
    """One more case of the same ranges, at most as costly as the largest listed one."""
    while True:
        what = rng.random()
        if what < 0.5:
            widths, act, loss, samples = _draw_net(rng)
            wide = widths[0] >= 256
            fireworks, sparks, guiding = _population(rng, wide)
            case = _step("", "-".join(map(str, widths)), act, loss, samples,
                         rng.choice(("fp32", "fp32", "bf16")), fireworks, sparks, guiding,
                         generations=1, populations=rng.choice((1, 1, 1, 2, 3)), **_options(rng))
            if _flops(case) < 1e8:
                case["generations"] = rng.choice((1, 5, 10))
        elif what < 0.65:
            h = rng.choice((16, 32, 64, 96, 128, 200, 256, 384, 512))
            d = _log_int(rng, 10, 2000)
            fireworks, sparks, guiding = _population(rng, True)
            case = _net("", "-".join(map(str, (d,) + (h,) * rng.randint(2, 11) + (1,))),
                        rng.choice(("relu", "gelu", "tanh")), fireworks, sparks, guiding)
        elif what < 0.85:
            widths, act, loss, samples = _draw_net(rng)
            case = _evaluate("", "-".join(map(str, widths)), ",".join([act] * (len(widths) - 2)),
                             loss, samples, rng.choice(("fp32", "fp32", "bf16")),
                             _log_int(rng, 1, 3000))
        elif what < 0.95:
            fireworks, sparks, guiding = _population(rng, True)
            case = dict(kind="ask_tell", dim=_log_int(rng, 100, 200000), fireworks=fireworks,
                        sparks=sparks, guiding=guiding)
        else:
            case = dict(kind="batch", jobs=rng.randint(8, 32), mix=rng.randint(1, 1000),
                        precision=rng.choice(("fp32", "bf16")), generations=1)
        case.pop("name", None)
        if _affordable(case):
            return case


def _affordable(case):
    if case["kind"] == "batch":
        return True
    if case["kind"] == "ask_tell":
        return case["fireworks"] * case["sparks"] * case["dim"] <= 2 ** 29
    if case["kind"] == "net":
        return _flops(case) <= 5e10
    widths = _widths(case)
    rows = case["rows"] if case["kind"] == "evaluate" else (
        case["populations"] * case["fireworks"] * case["sparks"])
    limit = 5e12 if widths[0] >= 256 else 5e11
    return _flops(case) <= limit and rows * _dim(widths) <= 2 ** 30


# ---- sizes ------------------------------------------------------------------------------------
def _widths(case):
    return tuple(int(w) for w in case["net"].split("-"))


def _acts(case):
    acts = case["act"].split(",")
    return tuple(acts * (len(_widths(case)) - 2) if len(acts) == 1 else acts)


def _dim(widths):
    return sum((i + 1) * o for i, o in zip(widths, widths[1:]))


def _products(widths):
    return sum(i * o for i, o in zip(widths, widths[1:]))


def _flops(case):
    """Multiplications and additions of the layers' products in one pass."""
    if case["kind"] == "ask_tell":
        return 0.0
    if case["kind"] == "batch":
        return float(sum(wl.flops_per_eval() * wl.n_fireworks * (wl.n_sparks + wl.n_guiding)
                         for wl in _mix(case))) * case["generations"]
    per = 2.0 * _products(_widths(case)) * case.get("samples", 1)
    if case["kind"] == "evaluate":
        return per * case["rows"]
    return (per * case.get("populations", 1) * case["fireworks"]
            * (case["sparks"] + case["guiding"]) * case["generations"])


def work(case):
    """Bytes: the samples (or the fixed network) and the fireworks read, the candidates'
    fitness and the new fireworks written; sparks need not leave the chip, except where the
    caller holds them (evaluate) or takes them (ask)."""
    kind = case["kind"]
    if kind == "ask_tell":
        candidates = case["fireworks"] * (case["sparks"] + case["guiding"])
        return {"bytes": 4.0 * (candidates * (case["dim"] + 1) + 2 * case["fireworks"] * case["dim"]),
                "flops": 0.0}
    if kind == "batch":
        data = sum(wl.n_samples * (wl.widths[0] + 1) + 2 * wl.n_fireworks * wl.dim
                   for wl in _mix(case))
        return {"bytes": 4.0 * data * case["generations"], "flops": _flops(case)}
    widths = _widths(case)
    if kind == "evaluate":
        return {"bytes": 4.0 * (case["samples"] * (widths[0] + 1) + case["rows"] * (_dim(widths) + 1)),
                "flops": _flops(case)}
    fireworks = case.get("populations", 1) * case["fireworks"]
    if kind == "net":
        data, dim = _dim(widths), widths[0]
    else:
        data, dim = case["samples"] * (widths[0] + 1), _dim(widths)
    candidates = fireworks * (case["sparks"] + case["guiding"])
    return {"bytes": 4.0 * (data + 2 * fireworks * dim + candidates) * case["generations"],
            "flops": _flops(case)}


# ---- inputs -----------------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda")


def _uniform(gen, lo, hi, *shape):
    return torch.rand(*shape, generator=gen, device="cuda") * (hi - lo) + lo


def _samples(widths, loss, n, seed):
    """(x, y, labels) on the GPU: a noisy random teacher's targets for MSE, a Gaussian mixture
    for cross-entropy, sparse noisy prototypes in [0, 1] for wide inputs (the distributions of
    inputs.teacher_regression, gaussian_mixture and sparse_prototypes)."""
    gen = _generator(seed)
    d, out = widths[0], widths[-1]
    if loss == "mse":
        x = _normal(gen, n, d)
        teacher = _normal(gen, d, out) / math.sqrt(d)
        return x, torch.tanh(x @ teacher) + 0.1 * _normal(gen, n, out), None
    labels = (torch.arange(n, device="cuda") % out)[torch.randperm(n, generator=gen, device="cuda")]
    if d < 256:
        x = 2.0 * _normal(gen, out, d)[labels] + _normal(gen, n, d)
    else:
        support = (torch.rand(out, d, generator=gen, device="cuda") < 0.2).float()
        prototypes = _uniform(gen, 0.5, 1.0, out, d)
        x = (prototypes[labels] + 0.1 * _normal(gen, n, d)).clamp(0.0, 1.0) * support[labels]
    return x, None, labels.to(torch.int32)


def _mix(case):
    """The shapes of a batch's jobs (their data comes from the seed)."""
    key = (case["jobs"], case["mix"])
    if key not in _mixes:
        _mixes[key] = inputs.mixed_jobs(n_jobs=case["jobs"], seed=case["mix"])
    return _mixes[key]


_mixes = {}


def _outputs(job, names=STATE):
    """The job's state arrays (views of its own buffers)."""
    state = job.state()
    return {name: state[name] for name in names}


def _rows(case, seed):
    """Candidate weight vectors, uniform in the search box (rows padded to 4 floats)."""
    dim = _dim(_widths(case))
    ld = (dim + 3) // 4 * 4
    rows = torch.zeros(case["rows"], ld, device="cuda")
    rows[:, :dim] = _uniform(_generator(seed + 1), LB, UB, case["rows"], dim)
    return rows


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind}
    if kind == "batch":
        jobs = []
        for i, wl in enumerate(_mix(case)):
            x, y, labels = _samples(wl.widths, wl.loss, wl.n_samples, seed * 1000 + i)
            jobs.append(mgfwa.MGFWA(wl.widths, wl.acts, wl.loss, x, y, labels,
                                    n_fireworks=wl.n_fireworks, n_sparks=wl.n_sparks,
                                    n_guiding=wl.n_guiding, lb=LB, ub=UB,
                                    max_generations=wl.generations, precision=case["precision"],
                                    seed=seed + i))
        for job in jobs:
            job.autotune(3)
        state.update(jobs=jobs, batch=mgfwa.Batch(jobs), generations=case["generations"],
                     out=[_outputs(job, ("F", "Y")) for job in jobs])
        return state
    common = dict(lb=LB, ub=UB, max_generations=300, seed=seed)
    if kind == "ask_tell":
        # one layer of dim - 1 inputs: as many weights as the black box has variables
        job = mgfwa.MGFWA((case["dim"] - 1, 1), (), "mse", external_fitness=True,
                          n_fireworks=case["fireworks"], n_sparks=case["sparks"],
                          n_guiding=case["guiding"], **common)
        job.tell(_black_box(job.ask()))
        state.update(job=job, out=_outputs(job))
        return state
    widths, acts = _widths(case), _acts(case)
    if kind == "evaluate":
        x, y, labels = _samples(widths, case["loss"], case["samples"], seed)
        state.update(job=mgfwa.MGFWA(widths, acts, case["loss"], x, y, labels, n_fireworks=2,
                                     n_sparks=8, n_guiding=2, precision=case["precision"], **common),
                     rows=_rows(case, seed))
        return state
    common.update(n_fireworks=case["fireworks"], n_sparks=case["sparks"], n_guiding=case["guiding"])
    if kind == "net":
        gen = _generator(seed)
        layers = []
        for i, o in zip(widths, widths[1:]):
            bound = 1.0 / math.sqrt(i)
            layers += [_uniform(gen, -bound, bound, o * i), _uniform(gen, -bound, bound, o)]
        job = mgfwa.MGFWA(widths, acts, net=torch.cat(layers), **common)
    else:
        x, y, labels = _samples(widths, case["loss"], case["samples"], seed)
        job = mgfwa.MGFWA(widths, acts, case["loss"], x, y, labels, precision=case["precision"],
                          n_populations=case["populations"], map_range=case["map_range"],
                          lag_guiding=case["lag_guiding"], regen_sparks=case["regen_sparks"],
                          **common)
    state.update(job=job, generations=case["generations"], out=_outputs(job))
    return state


def _black_box(x):
    """The caller's objective over spark positions: the distance from the origin."""
    return torch.linalg.vector_norm(x, dim=1)


def run(state):
    kind = state["kind"]
    if kind == "batch":
        state["batch"].step(state["generations"])
        return state["out"]
    job = state["job"]
    if kind == "evaluate":
        return job.evaluate(state["rows"])
    if kind == "ask_tell":
        job.tell(_black_box(job.ask()))   # explosion sparks
        job.tell(_black_box(job.ask()))   # guiding sparks, then the selection
    else:
        job.step(state["generations"])
    return state["out"]


_ACT64 = {"identity": lambda z: z, "relu": torch.relu, "tanh": torch.tanh,
          "gelu": torch.nn.functional.gelu}


def exact(case, seed):
    """Losses of the caller's weight vectors in 64 bits (evaluate); a generation's state follows
    from the generator's draws and has no value of its own here."""
    if case["kind"] != "evaluate":
        return None
    widths, acts = _widths(case), _acts(case)
    x, y, labels = _samples(widths, case["loss"], case["samples"], seed)
    x = x.double()
    losses = np.empty(case["rows"])
    for r, row in enumerate(_rows(case, seed)):
        h, at = x, 0
        row = row.double()
        for layer, (i, o) in enumerate(zip(widths, widths[1:])):
            w = row[at:at + i * o].view(o, i)
            b = row[at + i * o:at + i * o + o]
            at += i * o + o
            h = h @ w.t() + b
            if layer < len(acts):
                h = _ACT64[acts[layer]](h)
        if case["loss"] == "mse":
            losses[r] = ((h - y.double()) ** 2).mean().item()
        else:
            losses[r] = torch.nn.functional.cross_entropy(h, labels.long()).item()
    return losses
