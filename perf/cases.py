"""What a user of this library has it do, as cases to be timed.

A case is one call of a public entry point on a state a program would hold: steps of
the integrator (``md.md_step``, single systems and ensembles), one force evaluation
(``md.md_force``), the energies of a report (``md.md_energy``), a Hessian-vector
product (``md.md_hvp``) and the gradient of a trajectory (``autograd.trajectory`` and
its backward).  Initial states are those of ``inputs.py`` (waterbags of angles, the
unit disk), drawn on the GPU from the seed; softening and time steps are the
benchmark's.

``listed`` holds the workloads of ``bench.py`` and the sizes of the paper's tables
beside the smallest calls; ``draw`` gives others over the same ranges.  ``exact``
computes what ``run`` returns in plain FP64 torch from the definitions.
"""
from __future__ import annotations

import math
import random

import torch

from paper_1212_0262_amd import autograd, md

MODELS = {"grav2d": md.GRAV2D, "ring": md.RING, "hmf": md.HMF}
PRECS = {"fp64": md.FP64, "mixed": md.MIXED, "kahan": md.MIXED_KAHAN, "pairf64": md.MIXED_PAIRF64,
         "f32state": md.MIXED_F32STATE}
EPS = {"grav2d": 1e-3, "ring": 1e-2, "hmf": 0.0}
DT = {"grav2d": 0.01, "ring": 0.05, "hmf": 0.1}


def listed():
    return [
        # the headline run: 2D gravity at N = 262,144, mixed precision
        {"name": "grav2d_mixed_262144", "call": "step", "model": "grav2d", "prec": "mixed", "n": 262144, "steps": 1},
        # a size of the paper's 2D table in FP64, between two reports
        {"name": "grav2d_fp64_20480", "call": "step", "model": "grav2d", "prec": "fp64", "n": 20480, "steps": 5},
        # a few hundred bodies, where launches and latency count
        {"name": "grav2d_kahan_301", "call": "step", "model": "grav2d", "prec": "kahan", "n": 301, "steps": 10},
        # the Ring workload: N = 2048 in FP64, the whole run of 50 steps
        {"name": "ring_fp64_2048", "call": "step", "model": "ring", "prec": "fp64", "n": 2048, "steps": 50},
        # the paper's third Ring size, ragged
        {"name": "ring_mixed_102401", "call": "step", "model": "ring", "prec": "mixed", "n": 102401, "steps": 1},
        # the HMF workload: N = 1e7 in FP64, bound by memory
        {"name": "hmf_fp64_1e7", "call": "step", "model": "hmf", "prec": "fp64", "n": 10_000_000, "steps": 5},
        # the smallest N of the paper's HMF table with the FP32 state, ragged
        {"name": "hmf_f32state_100003", "call": "step", "model": "hmf", "prec": "f32state", "n": 100_003, "steps": 10},
        # finite-N studies of the HMF: a few thousand particles over many steps
        {"name": "hmf_fp64_2001", "call": "step", "model": "hmf", "prec": "fp64", "n": 2001, "steps": 50},
        # the ensemble workload: 256 Ring realizations, compensated sums
        {"name": "ensemble_kahan_256", "call": "step", "model": "ring", "prec": "kahan", "nb": 256, "nmin": 1000,
         "nmax": 16384, "steps": 1},
        # the energies of one report of the headline run
        {"name": "energy_grav2d_262144", "call": "energy", "model": "grav2d", "prec": "mixed", "n": 262144},
        # the energies of one report of the paper's Ring accuracy run
        {"name": "energy_ring_16384", "call": "energy", "model": "ring", "prec": "fp64", "n": 16384},
        # the adjoint workload's system: the gradient of K_T through two steps
        {"name": "gradient_grav2d_32768", "call": "gradient", "model": "grav2d", "prec": "fp64", "n": 32768,
         "steps": 2},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choices(["step", "ensemble", "force", "energy", "hvp", "gradient"], [40, 10, 8, 16, 10, 16])[0]
    if call == "ensemble":
        model = rng.choice(["ring", "ring", "grav2d"])
        nmin = _log_int(rng, 64, 2000)
        case = {"call": rng.choice(["step", "step", "energy"]), "model": model,
                "prec": rng.choice(["fp64", "mixed", "kahan"]), "nb": _log_int(rng, 8, 256), "nmin": nmin,
                "nmax": _log_int(rng, nmin + 1, 16384)}
        if case["call"] == "step":
            case["steps"] = rng.randint(1, 2)
        return case
    model = rng.choice(["grav2d", "ring", "hmf"])
    # derivatives are taken in FP64
    if call in ("hvp", "gradient"):
        n = _log_int(rng, 200, 3_000_000) if model == "hmf" else _log_int(rng, 200, 40_000)
        case = {"call": call, "model": model, "prec": "fp64", "n": n}
        if call == "gradient":
            case["steps"] = rng.randint(1, 4)
        return case
    if model == "hmf":
        prec = rng.choice(["fp64", "f32state"]) if call == "step" else "fp64"
        n = _log_int(rng, 200, 10_000_000)
    else:
        prec = rng.choice(["fp64", "mixed", "kahan", "pairf64"])
        n = _log_int(rng, 100, 131_072)
    case = {"call": call, "model": model, "prec": prec, "n": n}
    if call == "step":
        case["steps"] = rng.randint(1, 2) if n > 30_000 and model != "hmf" else rng.randint(1, 20)
    return case


# ------------------------------------------------------------------------ states --

def _sizes(case):
    """The realization sizes of an ensemble: log-uniform in [nmin, nmax], the same for every seed."""
    nb, lo, hi = case["nb"], case["nmin"], case["nmax"]
    sizes = [int(round(lo * (hi / lo) ** ((b + 0.5) / nb))) for b in range(nb)]
    random.Random(nb).shuffle(sizes)
    return sizes


def _total(case):
    return sum(_sizes(case)) if "nb" in case else case["n"]


def _state(case, seed):
    """(q, p) on the GPU, the distributions of inputs.py."""
    n, model = _total(case), case["model"]
    g = torch.Generator(device="cuda").manual_seed(seed)

    def uniform(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)

    if model == "ring":
        return uniform(-math.pi / 2, math.pi / 2, 1, n), uniform(-0.5, 0.5, 1, n)
    if model == "hmf":
        return uniform(-1.0, 1.0, 1, n), uniform(-1.2, 1.2, 1, n)
    r, phi = uniform(0.0, 1.0, n).sqrt(), uniform(0.0, 2 * math.pi, n)
    p = 0.5 * torch.randn(2, n, dtype=torch.float64, device="cuda", generator=g)
    return torch.stack([r * phi.cos(), r * phi.sin()]), p - p.mean(dim=1, keepdim=True)


def _vectors(case, seed, count):
    """Adjoint vectors of unit scale."""
    d = 2 if case["model"] == "grav2d" else 1
    g = torch.Generator(device="cuda").manual_seed(seed + 1_000_003)
    return [torch.randn(d, case["n"], dtype=torch.float64, device="cuda", generator=g) for _ in range(count)]


def prepare(case, seed):
    q, p = _state(case, seed)
    model, prec, eps = MODELS[case["model"]], PRECS[case["prec"]], EPS[case["model"]]
    if "nb" in case:
        offsets = [0]
        for s in _sizes(case):
            offsets.append(offsets[-1] + s)
        ctx = md.md_batch_init(model, prec, offsets, eps)
    else:
        ctx = md.md_init(model, prec, case["n"], eps)
    s = {"case": case, "ctx": ctx, "q": q, "p": p}
    if case["call"] in ("step", "force"):
        s["f"] = torch.empty_like(q)
    if case["call"] == "step":
        md.md_force(ctx, q, s["f"])
    elif case["call"] == "hvp":
        (s["w"],) = _vectors(case, seed, 1)
        s["out"] = torch.empty_like(q)
    elif case["call"] == "gradient":
        s["gq"], s["gp"] = _vectors(case, seed, 2)
        q.requires_grad_(True)
        p.requires_grad_(True)
    return s


def run(state):
    case, ctx, q, p = state["case"], state["ctx"], state["q"], state["p"]
    call = case["call"]
    if call == "step":
        md.md_step(ctx, q, p, state["f"], DT[case["model"]], case["steps"])
        return {"q": q, "p": p, "f": state["f"]}
    if call == "force":
        return {"f": md.md_force(ctx, q, state["f"])}
    if call == "energy":
        return {"energies": md.md_energy(ctx, q, p)}
    if call == "hvp":
        return {"hw": md.md_hvp(ctx, q, state["w"], state["out"])}
    qT, pT = autograd.trajectory(ctx, q, p, DT[case["model"]], case["steps"])
    gq, gp = torch.autograd.grad((qT, pT), (q, p), (state["gq"], state["gp"]))
    return {"q": qT.detach(), "p": pT.detach(), "grad_q": gq, "grad_p": gp}


def work(case):
    """Bytes: each array of the call read or written once per pass over the state.  Flops: each
    unordered pair once per force evaluation (2D 14, Ring 18, product 30; logarithm or root of a
    pair energy 10), HMF 60 a particle and stage."""
    d = 2 if case["model"] == "grav2d" else 1
    call, steps = case["call"], case.get("steps", 0)
    sizes = _sizes(case) if "nb" in case else [case["n"]]
    n = sum(sizes)
    hmf = case["model"] == "hmf"
    pairs = 0 if hmf else sum(s * (s - 1) // 2 for s in sizes)
    term = 14 if d == 2 else 18
    evals = {"step": 3 * steps, "force": 1, "energy": 0, "hvp": 0, "gradient": 6 * steps + 2}[call]
    products = {"hvp": 1, "gradient": 3 * steps + 1}.get(call, 0)
    flops = evals * (60 * n if hmf else term * pairs) + products * (60 * n if hmf else 30 * pairs)
    if call == "energy":
        flops += 40 * n if hmf else 10 * pairs + 2 * d * n
    arrays = {"step": 6, "force": 2, "energy": 2, "hvp": 3, "gradient": 8}[call]
    byte = 8 * d * n * arrays
    if hmf:  # the mean field joins every particle at each stage: the state is read and written there
        width = 4 if case["prec"] == "f32state" else 8
        byte += 4 * width * n * max(0, evals - 1) + 5 * 8 * n * max(0, products - 1)
    return {"bytes": byte, "flops": flops}


# ------------------------------------------------------------------------- exact --

_CHUNK = 1 << 28  # pair-matrix elements held at a time


def _rows(n):
    step = max(1, _CHUNK // n)
    return [slice(a, min(n, a + step)) for a in range(0, n, step)]


def _force(model, q, eps):
    n = q.shape[1]
    f = torch.empty_like(q)
    if model == "hmf":
        c, s = q.cos(), q.sin()
        return c * s.mean() - s * c.mean()
    for r in _rows(n):
        if model == "grav2d":
            dx = q[0, r, None] - q[0]
            dy = q[1, r, None] - q[1]
            w = (dx * dx).addcmul_(dy, dy).add_(eps).reciprocal_()
            f[0, r] = dx.mul_(w).sum(1) * (-2.0 / n)
            f[1, r] = dy.mul_(w).sum(1) * (-2.0 / n)
        else:
            d = q[0, r, None] - q[0]
            h = (0.5 * d).sin_()
            u = h.mul_(h).mul_(2.0).add_(eps)
            f[0, r] = d.sin_().div_(u * u.sqrt()).sum(1) * (-1.0 / (2 * math.sqrt(2.0) * n))
    return f


def _product(model, q, w, eps):
    n = q.shape[1]
    out = torch.empty_like(q)
    if model == "hmf":
        c, s = q.cos(), q.sin()
        return w * (c * c.mean() + s * s.mean()) - (c * (c * w).mean() + s * (s * w).mean())
    for r in _rows(n):
        if model == "grav2d":
            dx, dy = q[0, r, None] - q[0], q[1, r, None] - q[1]
            ux, uy = w[0, r, None] - w[0], w[1, r, None] - w[1]
            inv = (dx * dx).addcmul_(dy, dy).add_(eps).reciprocal_()
            t = (dx * ux).addcmul_(dy, uy).mul_(inv).mul_(inv).mul_(2.0)
            out[0, r] = (ux.mul_(inv) - t * dx).sum(1) * (2.0 / n)
            out[1, r] = (uy.mul_(inv) - t * dy).sum(1) * (2.0 / n)
        else:
            d = q[0, r, None] - q[0]
            h = (0.5 * d).sin_()
            u = h.mul_(h).mul_(2.0).add_(eps)
            t = (d.cos() - 1.5 * d.sin().square_() / u) / (u * u.sqrt())
            out[0, r] = (t * (w[0, r, None] - w[0])).sum(1) * (1.0 / (2 * math.sqrt(2.0) * n))
    return out


def _potential(model, q, eps):
    n = q.shape[1]
    if model == "hmf":
        return 0.5 * n * (1.0 - q.cos().mean() ** 2 - q.sin().mean() ** 2)
    total = torch.zeros((), dtype=torch.float64, device=q.device)
    for r in _rows(n):
        if model == "grav2d":
            dx, dy = q[0, r, None] - q[0], q[1, r, None] - q[1]
            total += (dx * dx).addcmul_(dy, dy).add_(eps).log_().sum()
        else:
            h = (0.5 * (q[0, r, None] - q[0])).sin_()
            total += h.mul_(h).mul_(2.0).add_(eps).rsqrt_().sum()
    if model == "grav2d":  # every ordered pair and the n self terms were added
        return (total - n * math.log(eps)) / (2 * n)
    return -(total - n / math.sqrt(eps)) / (2 * math.sqrt(2.0) * n)


def _stages(dt, steps):
    """(kick, drift) of each stage in order (eq. 4); the last kick has no drift."""
    w1 = 1.0 / (2.0 - 2.0 ** (1.0 / 3.0))
    w0 = 1.0 - 2.0 * w1
    b0, b1 = 0.5 * w1, 0.5 * (w0 + w1)
    out = []
    for _ in range(steps):
        out += [(b0 * dt, w1 * dt), (b1 * dt, w0 * dt), (b1 * dt, w1 * dt), (b0 * dt, None)]
    return out


def _trajectory(model, q, p, eps, dt, steps):
    """(q, p, f, kick positions) after `steps` steps."""
    q, p, f, kicks = q.clone(), p.clone(), _force(model, q, eps), []
    for kick, drift in _stages(dt, steps):
        p += kick * f
        kicks.append(q.clone())
        if drift is not None:
            q += drift * p
            f = _force(model, q, eps)
    return q, p, f, kicks


def exact(case, seed):
    model, call, steps = case["model"], case["call"], case.get("steps", 0)
    eps, dt = EPS[model], DT[model]
    q, p = _state(case, seed)
    if "nb" in case:
        parts = [(a.contiguous(), b.contiguous())
                 for a, b in zip(q.split(_sizes(case), dim=1), p.split(_sizes(case), dim=1))]
        if call == "energy":
            rows = []
            for a, b in parts:
                k, v = 0.5 * (b * b).sum(), _potential(model, a, eps)
                rows.append(torch.stack([k, v, k + v]))
            return {"energies": torch.stack(rows)}
        done = [_trajectory(model, a, b, eps, dt, steps)[:3] for a, b in parts]
        return {k: torch.cat([x[i] for x in done], dim=1) for i, k in enumerate(("q", "p", "f"))}
    if call == "step":
        q, p, f, _ = _trajectory(model, q, p, eps, dt, steps)
        return {"q": q, "p": p, "f": f}
    if call == "force":
        return {"f": _force(model, q, eps)}
    if call == "energy":
        k, v = 0.5 * (p * p).sum(), _potential(model, q, eps)
        return {"energies": torch.stack([k, v, k + v])}
    if call == "hvp":
        (w,) = _vectors(case, seed, 1)
        return {"hw": _product(model, q, w, eps)}
    lq, lp = _vectors(case, seed, 2)
    qT, pT, _, kicks = _trajectory(model, q, p, eps, dt, steps)
    for (kick, drift), at in zip(reversed(_stages(dt, steps)), reversed(kicks)):
        if drift is not None:
            lp = lp + drift * lq
        lq = lq - kick * _product(model, at, lp, eps)
    return {"q": qT, "p": pT, "grad_q": lq, "grad_p": lp}
