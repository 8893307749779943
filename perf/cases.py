"""What this framework is timed on: the calls that its users make, over the sizes they make them at.

A case is a dict of plain values.  Its "call" says which public entry point it goes through:

  sum      Plan.compute() on a plan that is kept (one summation per call, the main use)
  step     Plan(...) and compute() together: particles that moved, a new tree for every summation
  batch    Batch.compute(): many independent problems in one launch
  direct   direct_sum(): the compensated reference sum on sampled targets, by which errors are checked
  grad     mlp_loss_grad(): forward and backward of the degree model on one mini-batch of training pairs
  forward  mlp_forward(): the degree model's predictions for a list of pairs

Distributions, theta, degree and leaf sizes are those of the package's own workloads, tests and
benchmark (uniform cube, Gaussian cloud, sphere surface, slab, Plummer; theta 0.6 .. 0.87, degree
4 .. 9, leaves of 500 .. 2000).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2012_06925_amd import _lib, api, inputs
from paper_2012_06925_amd.train_degree_model import load_model

PHYSICAL = ("coulomb", "yukawa", "oscillatory", "regcoulomb")
FLAGS = {"fp64": 0, "fp32": _lib.FP32_EVAL, "tuned": _lib.FP32_EVAL | _lib.LEARNED_DEGREE}
SCHEMES = {"dual": 0, "bltc": _lib.BLTC, "cp_bltc": _lib.CP_BLTC}
# flops of one kernel value (differences, squares, 1/r and the kernel's own function) without the
# multiplication by the charge and the addition
VALUE_FLOPS = {"coulomb": 9, "yukawa": 13, "oscillatory": 12, "regcoulomb": 11}


def _sum(n, dist="uniform", kernel="coulomb", theta=0.7, degree=8, leaf=2000, form="fp64", scheme="dual", m=0,
         tdist="", call="sum"):
    """m targets of distribution tdist, or targets = sources when m is 0."""
    return dict(call=call, n=n, dist=dist, kernel=kernel, theta=theta, degree=degree, leaf=leaf, form=form,
                scheme=scheme, m=m, tdist=tdist)


def listed():
    return [
        # a small problem in a time loop: launches and the host's walk count
        dict(_sum(10_000, degree=6, leaf=500), name="cube1e4"),
        # the smallest of the method's published sizes, an odd number of clustered particles
        dict(_sum(100_003, dist="gaussian"), name="gauss1e5"),
        # the ordinary size of one summation
        dict(_sum(1_000_000, theta=0.8), name="cube1e6"),
        # the throughput workload, FP64 at an error of 1e-6
        dict(_sum(10_000_000, theta=0.8, degree=7), name="cube1e7"),
        # FP32 evaluation with the learned per-pair degree, the form used when 1e-6 is enough
        dict(_sum(1_000_000, theta=0.8, form="tuned"), name="cube1e6_tuned"),
        # targets apart from the sources (field on a surface from a cloud), screened kernel
        dict(_sum(10_000_000, dist="gaussian", kernel="yukawa", m=2_000_000, tdist="sphere"),
             name="sphere2e6_gauss1e7"),
        # screened electrostatics, targets = sources, small leaves: every interaction type occurs
        dict(_sum(300_007, kernel="yukawa", degree=6, leaf=500), name="yukawa3e5"),
        # oscillatory kernel (the domain two wavelengths wide)
        dict(_sum(120_011, kernel="oscillatory", degree=8, leaf=1000), name="osc1e5"),
        # moving particles: plan and summation for every step
        dict(_sum(200_003, theta=0.7, degree=7, call="step"), name="step2e5"),
        # many independent uneven problems at once
        dict(call="batch", count=40, lo=1_000, hi=100_000, kernel="coulomb", theta=0.7, degree=6, leaf=500,
             form="fp64", name="batch40"),
        # the accuracy check of a run: 0.1 % of the targets summed directly
        dict(call="direct", n=1_000_000, nsel=1000, dist="uniform", kernel="coulomb", name="direct1e6"),
        # one training step of the degree model at its training script's batch size
        dict(call="grad", n=1024, name="grad1024"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["sum"] * 10 + ["tuned", "tuned", "step", "batch", "batch", "direct", "grad", "forward"])
    dist = rng.choice(["uniform", "gaussian", "sphere", "slab", "plummer"])
    theta, degree, leaf = rng.choice([0.6, 0.7, 0.8, 0.87]), rng.randint(4, 9), rng.choice([500, 1000, 2000])
    if call == "sum":
        kernel = rng.choice(["coulomb", "coulomb", "yukawa", "oscillatory", "regcoulomb"])
        if kernel == "oscillatory":             # a domain of many wavelengths needs more than degree 9
            dist = rng.choice(["uniform", "gaussian", "sphere"])
        c = _sum(_log(rng, 1000, 1_000_000 if kernel == "coulomb" else 300_000), dist, kernel, theta, degree, leaf,
                 form=rng.choice(["fp64", "fp64", "fp64", "fp32"]))
        if rng.random() < 0.35:                 # targets of their own
            c.update(m=_log(rng, 1000, 300_000), tdist=rng.choice(["uniform", "gaussian", "sphere"]),
                     n=min(c["n"], 300_000), scheme=rng.choice(["dual", "dual", "bltc", "cp_bltc"]))
        return c
    if call == "tuned":
        return _sum(_log(rng, 30_000, 1_000_000), rng.choice(["uniform", "gaussian"]), theta=rng.choice([0.8, 0.87]),
                    form="tuned")
    if call == "step":
        return _sum(_log(rng, 5_000, 300_000), dist, theta=theta, degree=degree, leaf=leaf, call="step")
    if call == "batch":
        lo = _log(rng, 500, 3_000)
        return dict(call="batch", count=rng.randint(4, 48), lo=lo, hi=_log(rng, 3 * lo, 60_000),
                    kernel=rng.choice(["coulomb", "coulomb", "yukawa"]), theta=rng.choice([0.6, 0.7, 0.8]),
                    degree=rng.randint(4, 8), leaf=rng.choice([300, 500, 1000]), form="fp64")
    if call == "direct":
        return dict(call="direct", n=_log(rng, 10_000, 1_000_000), nsel=_log(rng, 1, 3000), dist=dist,
                    kernel=rng.choice(PHYSICAL))
    if call == "grad":
        return dict(call="grad", n=_log(rng, 32, 8192))
    return dict(call="forward", n=_log(rng, 100, 300_000))


# ---- inputs -------------------------------------------------------------------------------------

def _generator(seed, stream=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + 7919 * stream) % (1 << 62))
    return g


def _points(n, dist, g):
    rand = lambda *s: torch.rand(*s, dtype=torch.float64, device="cuda", generator=g)       # noqa: E731
    normal = lambda *s: torch.randn(*s, dtype=torch.float64, device="cuda", generator=g)    # noqa: E731
    if dist == "uniform":
        return 2.0 * rand(3, n) - 1.0
    if dist == "gaussian":
        return 0.25 * normal(3, n)
    if dist == "slab":
        return rand(3, n) * torch.tensor([[1.0], [10.0], [10.0]], dtype=torch.float64, device="cuda")
    v = normal(3, n)
    v = v / v.norm(dim=0)
    if dist == "sphere":
        return v
    if dist == "plummer":                       # radius from the enclosed mass, cut at 100
        top = 1e6 / (1.0 + 1e4) ** 1.5
        u = rand(n) * top
        return v / torch.sqrt(u.clamp_min(1e-300) ** (-2.0 / 3.0) - 1.0)
    raise ValueError(dist)


def _charges(n, dist, g):
    if dist == "plummer":
        return torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    return 2.0 * torch.rand(n, dtype=torch.float64, device="cuda", generator=g) - 1.0


def _sets(case, seed):
    """(targets or None, sources) as contiguous float64 cuda vectors."""
    g = _generator(seed)
    p = _points(case["n"], case["dist"], g)
    src = [p[0].contiguous(), p[1].contiguous(), p[2].contiguous(), _charges(case["n"], case["dist"], g)]
    if not case.get("m"):
        return None, src
    t = _points(case["m"], case["tdist"], _generator(seed, 1))
    return [t[0].contiguous(), t[1].contiguous(), t[2].contiguous()], src


def _batch_sizes(case):
    """Sizes and distributions of a batch's problems: they do not move with the seed of the particles."""
    rng = np.random.default_rng([case["count"], case["lo"], case["hi"]])
    sizes = np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["count"]))).astype(int)
    return sizes, rng.integers(0, 3, case["count"])


def _batch(case, seed):
    sizes, kinds = _batch_sizes(case)
    return [_sets(dict(n=int(n), dist=("uniform", "gaussian", "sphere")[k]), int(seed) * 64 + i)
            for i, (n, k) in enumerate(zip(sizes, kinds))]


def _pair_features(n, seed):
    """Features of separated pairs as a traversal meets them: radius ratio, separation, counts."""
    g = _generator(seed, 2)
    u = torch.rand(n, 4, dtype=torch.float32, device="cuda", generator=g)
    lo = torch.tensor([-1.2, 0.15, 4.5, 4.5], device="cuda")
    hi = torch.tensor([1.2, 1.2, 10.0, 10.0], device="cuda")
    return (lo + u * (hi - lo)).contiguous()


def _pair_errors(n, feats, seed):
    """log10 errors that fall with the degree and the separation, some of them missing (NaN)."""
    g = _generator(seed, 3)
    d = torch.arange(2, 13, dtype=torch.float32, device="cuda")
    e = -0.4 - feats[:, 1:2] * d - 0.2 * d + 0.3 * torch.randn(n, 11, device="cuda", generator=g)
    gone = torch.rand(n, 1, device="cuda", generator=g) < 0.02
    return torch.where(gone, torch.nan, e).clamp_min(-14.0).contiguous()


def _model(seed):
    """The shipped model, its weights a little moved: another point of a training run."""
    m = load_model()
    rng = np.random.default_rng([int(seed), 23])
    k = m.size - 16
    m[:k] += 0.02 * rng.standard_normal(k).astype(np.float32)
    return m


def _plan(case, targets, sources):
    flags = FLAGS[case["form"]] | SCHEMES[case["scheme"]]
    if max(case["n"], case["m"]) >= 150_000:    # below, the host builds trees sooner
        flags |= _lib.DEVICE_TREE
    plan = api.Plan(targets, sources, kernel=case["kernel"], theta=case["theta"], degree=case["degree"],
                    leaf=case["leaf"], flags=flags)
    if case["form"] == "tuned":
        plan.set_degree_model(load_model(), fallback=8, tau=inputs.TAU)
    return plan


def prepare(case, seed):
    call = case["call"]
    if call == "sum":
        targets, sources = _sets(case, seed)
        return dict(call=call, plan=_plan(case, targets, sources))
    if call == "step":
        targets, sources = _sets(case, seed)
        return dict(call=call, case=case, targets=targets, sources=sources)
    if call == "batch":
        return dict(call=call, batch=api.Batch(_batch(case, seed), kernel=case["kernel"], theta=case["theta"],
                                               degree=case["degree"], leaf=case["leaf"], flags=FLAGS[case["form"]]))
    if call == "direct":
        _, sources = _sets(case, seed)
        pick = torch.randperm(case["n"], device="cuda", generator=_generator(seed, 4))[:case["nsel"]]
        return dict(call=call, kernel=case["kernel"], sources=sources, sel=pick.sort().values.contiguous())
    feats = _pair_features(case["n"], seed)
    model = torch.from_numpy(_model(seed)).cuda()
    if call == "forward":
        return dict(call=call, model=model, feats=feats)
    return dict(call=call, model=model, feats=feats, errors=_pair_errors(case["n"], feats, seed))


def run(state):
    call = state["call"]
    if call == "sum":
        return state["plan"].compute()
    if call == "step":
        with _plan(state["case"], state["targets"], state["sources"]) as plan:
            return plan.compute()
    if call == "batch":
        return state["batch"].compute()
    if call == "direct":
        s = state["sources"]
        return api.direct_sum(s[:3], s, kernel=state["kernel"], sel=state["sel"])
    if call == "forward":
        return api.mlp_forward(state["model"], state["feats"])
    loss, grad = api.mlp_loss_grad(state["model"], state["feats"], state["errors"])
    return dict(loss=loss, grad=grad)


# ---- what a pass cannot do without ---------------------------------------------------------------

_terms = {}


def _host_terms(case):
    """Kernel terms of the method's own interaction lists, counted on a set of the case's kind."""
    key = tuple(sorted((k, v) for k, v in case.items() if k != "name"))
    if key not in _terms:
        s = inputs.particles(case["n"], case["dist"], seed=1)
        t = inputs.particles(case["m"], case["tdist"], seed=2, charges=False) if case["m"] else None
        with api.HostPlan(None if t is None else (t.x, t.y, t.z), (s.x, s.y, s.z, s.q), kernel=case["kernel"],
                          theta=case["theta"], degree=case["degree"], leaf=case["leaf"],
                          flags=SCHEMES[case["scheme"]]) as plan:
            plan.traverse_host()
            _terms[key] = sum(plan.stats()["interactions"].values())
    return _terms[key]


def _sum_work(case):
    terms = _host_terms(case)
    m = case["m"] or case["n"]
    values = terms / 2 if not case["m"] else terms          # one kernel value serves both directions
    return {"bytes": 32.0 * case["n"] + (24.0 * m if case["m"] else 0.0) + 8.0 * m,
            "flops": VALUE_FLOPS[case["kernel"]] * values + 2.0 * terms}


def work(case):
    call = case["call"]
    if call in ("sum", "step"):
        return _sum_work(case)
    if call == "batch":
        sizes, _ = _batch_sizes(case)
        one = _sum(int(np.mean(sizes)), kernel=case["kernel"], theta=case["theta"], degree=case["degree"],
                   leaf=case["leaf"])
        w = _sum_work(one)
        return {k: v * case["count"] for k, v in w.items()}
    if call == "direct":
        return {"bytes": 32.0 * case["n"] + 16.0 * case["nsel"],
                "flops": (VALUE_FLOPS[case["kernel"]] + 8.0) * case["n"] * case["nsel"]}
    weights = 4 * 64 + 64 * 64 + 64 * 11
    if call == "forward":
        return {"bytes": 4.0 * (15 * case["n"] + weights), "flops": 2.0 * weights * case["n"]}
    return {"bytes": 4.0 * (15 * case["n"] + 2 * weights), "flops": 6.0 * weights * case["n"]}


# ---- the same results in 64 bits -----------------------------------------------------------------

EXACT_PAIRS = 4e10          # more than that takes too long by plain summation


def _value(r2, kernel):
    param = {"yukawa": 0.5, "regcoulomb": 0.005}.get(kernel, 0.0)
    zero = r2 == 0.0
    r = torch.sqrt(r2)
    if kernel == "coulomb":
        g = 1.0 / r
    elif kernel == "yukawa":
        g = torch.exp(-param * r) / r
    elif kernel == "oscillatory":
        g = torch.sin(math.pi * r) / r
    else:
        g = 1.0 / torch.sqrt(r2 + param * param)
    return g.masked_fill_(zero, 0.0)


def _direct(targets, sources, kernel):
    x, y, z, q = sources
    out = torch.empty_like(targets[0])
    rows = max(1, int(4e7 // x.numel()))
    for a in range(0, out.numel(), rows):
        tx, ty, tz = (t[a:a + rows, None] for t in targets)
        r2 = (tx - x) ** 2
        r2 += (ty - y) ** 2
        r2 += (tz - z) ** 2
        out[a:a + rows] = (_value(r2, kernel) * q).sum(dim=1)
    return out


def _net(model, feats):
    p = model.double()
    k = p.numel() - 16
    shapes = [(64, 4), (64,), (64, 64), (64,), (11, 64), (11,)]
    w, o = [], 0
    for s in shapes:
        w.append(p[o:o + math.prod(s)].reshape(s).clone().requires_grad_(True))
        o += math.prod(s)
    assert o == k
    x = (feats.double() - p[k:k + 4]) * p[k + 4:k + 8]
    h = torch.tanh(x @ w[0].T + w[1])
    h = torch.tanh(h @ w[2].T + w[3])
    return w, h @ w[4].T + w[5]


def exact(case, seed):
    call = case["call"]
    if call in ("sum", "step"):
        if float(case["n"]) * (case["m"] or case["n"]) > EXACT_PAIRS:
            return None
        targets, sources = _sets(case, seed)
        return _direct(targets or sources[:3], sources, case["kernel"])
    if call == "batch":
        problems = _batch(case, seed)
        if sum(float(s[0].numel()) ** 2 for _, s in problems) > 2 * EXACT_PAIRS:
            return None
        return [_direct(s[:3], s, case["kernel"]) for _, s in problems]
    if call == "direct":
        state = prepare(case, seed)
        s = state["sources"]
        return _direct([t[state["sel"]] for t in s[:3]], s, case["kernel"])
    state = prepare(case, seed)
    w, y = _net(state["model"], state["feats"])
    if call == "forward":
        return y.detach()
    ok = ~torch.isnan(state["errors"])
    loss = ((y - state["errors"].double())[ok] ** 2).mean()
    loss.backward()
    return dict(loss=float(loss.detach()), grad=torch.cat([t.grad.reshape(-1) for t in w]))
