"""The measured cases: evaluation and tracking calls as a user's program makes them.

A case is a dict of plain values.  ``kind`` is one of

* ``eval``  -- one ``eval_jac`` call on ``npts`` points that are already on the
  GPU, into output arrays the caller keeps (``jac`` false: values only; ``t``
  false: the target system alone, t = 1);
* ``track`` -- one ``track`` call on ``paths`` paths of one homotopy;
* ``batch`` -- one ``track_batch`` call over ``systems`` random systems.

``system`` names the recipe: the seeded generators of ``synth`` (dense,
quadratic, cubic, small, the stand-ins shaped like cyclic10, nash8 and
pieri44, the heterogeneous batch), drawn anew from the seed.
Precisions are the number of FP64 limbs: 1, 2 or 4.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1505_00383_amd as ph
from paper_1505_00383_amd import synth


def listed():
    return [
        # one launch on a handful of points: the call's own latency, as in a
        # program that evaluates the start points of a small system
        dict(name="eval_small_d", kind="eval", system="small", n=3, terms=4, k=2, e=2, npts=8, prec=1,
             jac=True, t=True),
        # the evaluation benchmark in complex double: 32 equations of 64
        # terms of 8 factors each
        dict(name="eval_dense_d", kind="eval", system="dense", n=32, terms=64, k=8, e=3, npts=65536, prec=1,
             jac=True, t=True),
        # few terms, very many points: the Jacobians of 2^20 points leave the chip
        dict(name="eval_quadratic16_d", kind="eval", system="quadratic", n=16, terms=16, k=2, e=2,
             npts=1 << 20, prec=1, jac=True, t=True),
        # the benchmark in double double
        dict(name="eval_dense_dd", kind="eval", system="dense", n=32, terms=64, k=8, e=3, npts=65536, prec=2,
             jac=True, t=True),
        # quad double on a modest odd number of points: the refinement of the
        # endpoints of one run
        dict(name="eval_dense_qd", kind="eval", system="dense", n=32, terms=64, k=8, e=3, npts=4999, prec=4,
             jac=True, t=True),
        # two shapes of the paper's evaluation tables at the paper's numbers of
        # paths: few long terms, and many terms in few unknowns
        dict(name="eval_cyclic10_dd", kind="eval", system="cyclic10", n=10, terms=10, k=10, e=1, npts=34940,
             prec=2, jac=True, t=True),
        dict(name="eval_nash8_qd", kind="eval", system="nash8", n=8, terms=130, k=7, e=1, npts=14833, prec=4,
             jac=True, t=True),
        # residuals alone (values, no Jacobian) of the target system at a set
        # of found endpoints
        dict(name="eval_values_dd", kind="eval", system="dense", n=32, terms=64, k=8, e=3, npts=6561, prec=2,
             jac=False, t=False),
        # the smallest tracking call: 8 paths of three quadrics
        dict(name="track_small_d", kind="track", system="small", n=3, terms=4, k=2, e=2, paths=8, prec=1,
             mixed=False, order=1),
        # every path of eight cubics, double-double residuals, FP64 solves
        dict(name="track_cubic8_dd", kind="track", system="cubic", n=8, terms=20, k=3, e=3, paths=6561, prec=2,
             mixed=True, order=1),
        # paths of sixteen quadrics with quad-double residuals, FP64 solves
        dict(name="track_quadratic16_qd", kind="track", system="quadratic", n=16, terms=16, k=2, e=2, paths=4096,
             prec=4, mixed=True, order=1),
        # a batch of systems of different sizes in one launch
        dict(name="track_batch_dd", kind="batch", system="batch", systems=16, paths=20000, prec=2, mixed=True,
             order=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every recipe at sizes spread over its range."""
    kind = rng.choice(["eval", "eval", "eval", "eval", "track", "batch"])
    if kind == "eval":
        prec = rng.choice([1, 2, 4])
        system = rng.choice(["dense", "dense", "quadratic", "small", "cyclic10", "nash8", "pieri44"])
        c = dict(kind="eval", system=system, prec=prec, jac=rng.random() < 0.8, t=rng.random() < 0.7)
        if system == "dense":
            n = rng.randint(5, 32)
            c.update(n=n, terms=_log_int(rng, 8, 64), k=rng.randint(2, min(n, 8)), e=rng.randint(1, 3))
        elif system == "quadratic":
            c.update(n=rng.randint(6, 16), terms=rng.randint(8, 20), k=2, e=2)
        elif system == "small":
            c.update(n=3, terms=4, k=2, e=2)
        else:
            c.update({"cyclic10": dict(n=10, terms=10, k=10, e=1), "nash8": dict(n=8, terms=130, k=7, e=1),
                      "pieri44": dict(n=16, terms=246, k=4, e=1)}[system])
        # points: from one up to the listed sizes, bounded by the work of the
        # largest listed evaluations (about 350 GFLOP) and by 5 GB of outputs
        probe = dict(c, npts=1)
        w = work(probe)
        most = min(1 << 20, int(3.5e11 / max(w["flops"], 1)), int(5e9 / w["bytes"]))
        c["npts"] = max(1, _log_int(rng, 1, max(2, most)))
        return c
    if kind == "track":
        system = rng.choice(["small", "cubic", "quadratic"])
        prec = rng.choice([1, 2, 2, 4])
        mixed = prec > 1 and rng.random() < 0.8
        order = rng.choice([1, 4])
        if system == "small":
            n, d, terms = 3, 2, 4
        elif system == "cubic":
            n, d = rng.randint(4, 8), 3
            terms = rng.randint(8, 20)
        else:
            n, d = rng.randint(6, 16), 2
            terms = rng.randint(8, 20)
        most = min(d ** n, 6561 if prec < 4 else 2048)
        if prec > 1 and not mixed:
            most = min(most, 1024 if prec == 2 else 128)
        return dict(kind="track", system=system, n=n, terms=terms, k=min(d, n), e=d, paths=_log_int(rng, 4, most),
                    prec=prec, mixed=mixed, order=order)
    systems = rng.randint(3, 24)
    return dict(kind="batch", system="batch", systems=systems, paths=_log_int(rng, 20 * systems, 20000),
                prec=rng.choice([1, 2]), mixed=True, order=rng.choice([1, 4]))


# ---------------------------------------------------------------------------
# systems
# ---------------------------------------------------------------------------
def _system(case, seed):
    s = synth.SEED_BASE + 1000 + 64 * int(seed)
    name = case["system"]
    if name == "small":
        return synth.tracking_small(seed=s)
    if name == "dense":
        return synth.eval_dense(seed=s + 1, n=case["n"], terms_per_eq=case["terms"], k=case["k"],
                                max_exp=case["e"])
    if name in synth.SHAPED:
        return synth.SHAPED[name](seed=s + 10)
    # quadratic: x_i^2, 1 and others of degree <= 2 in x_i and five other
    # unknowns; cubic: x_i^3, 1 and others of degree <= 3 in all unknowns
    rng = np.random.Generator(np.random.PCG64(s + 2))
    n, d = case["n"], case["e"]
    eqs = []
    for i in range(n):
        variables = list(range(n))
        if name == "quadratic":
            others = rng.choice([v for v in range(n) if v != i], size=5, replace=False)
            variables = sorted([i] + [int(v) for v in others])
        eqs.append(synth._equation_with_anchor(rng, variables, i, d, case["terms"]))
    return synth.system_from_terms(n, eqs, name=name, meta={"gamma": synth.unit_complex(rng)})


def _points(case, seed):
    """Points near the unit circle in every coordinate (torus points with
    random lower limbs) and t in [0, 1), as device arrays, point fastest."""
    g = torch.Generator(device="cuda")
    g.manual_seed(977 + int(seed))
    n, npts, L = case["n"], case["npts"], case["prec"]
    phi = torch.rand((n, npts), generator=g, device="cuda", dtype=torch.float64) * (2.0 * math.pi)
    x = torch.empty((n, 2, L, npts), device="cuda", dtype=torch.float64)
    x[:, 0, 0] = torch.cos(phi)
    x[:, 1, 0] = torch.sin(phi)
    for l in range(1, L):  # a random fraction of half an ulp of the limb above
        up = x[:, :, l - 1].abs()
        ulp = torch.nextafter(up, torch.full_like(up, math.inf)) - up
        x[:, :, l] = (torch.rand((n, 2, npts), generator=g, device="cuda", dtype=torch.float64) - 0.5) * ulp
    t = torch.rand((npts,), generator=g, device="cuda", dtype=torch.float64) if case["t"] else None
    return x.reshape(n * 2 * L, npts), t


def prepare(case, seed):
    kind = case["kind"]
    if kind == "eval":
        sysm = _system(case, seed)
        x, t = _points(case, seed)
        rows = sysm.n_eq * 2 * case["prec"]
        val = torch.empty((rows, case["npts"]), dtype=torch.float64, device="cuda")
        jac = None
        if case["jac"]:
            jac = torch.empty((rows * sysm.n_var, case["npts"]), dtype=torch.float64, device="cuda")
        return dict(case=case, sys=ph.System(sysm), gamma=synth.gamma_of(sysm), x=x, t=t, val=val, jac=jac)
    opts = ph.track_opts(prec=case["prec"], mixed=int(case["mixed"]), predictor_order=case["order"])
    if kind == "track":
        sysm = _system(case, seed)
        return dict(case=case, sys=ph.System(sysm), gamma=synth.gamma_of(sysm), opts=opts)
    # the supports and path subsets of the case are fixed; every coefficient
    # and gamma comes from the seed
    systems, gammas, paths, _ = synth.batch_heterogeneous(nsys=case["systems"], target_paths=case["paths"])
    rng = np.random.Generator(np.random.PCG64(synth.SEED_BASE + 5000 + int(seed)))
    for s in systems:
        th = rng.uniform(0.0, 2.0 * math.pi, size=len(s.coef))
        s.coef[:, 0], s.coef[:, 1] = np.cos(th), np.sin(th)
    gammas = [synth.unit_complex(rng) for _ in gammas]
    return dict(case=case, sys=[ph.System(s) for s in systems], gammas=gammas, paths=paths, opts=opts)


def run(state):
    c = state["case"]
    if c["kind"] == "eval":
        val, jac = ph.eval_jac(state["sys"], state["x"], c["npts"], c["prec"], t=state["t"], gamma=state["gamma"],
                               val=state["val"], jac=state["jac"], want_jac=c["jac"])
        return {"val": val, "jac": jac} if c["jac"] else {"val": val}
    if c["kind"] == "track":
        r = ph.track(state["sys"], state["gamma"], c["paths"], state["opts"])
    else:
        r = ph.track_batch(state["sys"], state["gammas"], state["paths"], state["opts"])
    return {k: r[k] for k in ("x_end", "status", "reason", "steps")}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
# FP64 flops of one complex product, addition and real scaling per precision
_FLOPS = {1: (6, 2, 2), 2: (80, 40, 16), 4: (660, 212, 124)}


def _term_flops(prec, k, m, jac):
    """One term of k factors, m of them with an exponent of 2 or more: 3k - 3
    products by reverse mode (k without derivatives) and one per power, the
    additions into H and J, the scalings by exponents and by c(t)."""
    mul, add, scale = _FLOPS[prec]
    if not jac:
        return (k + m) * mul + add + scale
    return (max(3 * k - 3, k) + m) * mul + (k + 1) * add + (m + 1) * scale


def _shape(case):
    """(terms, mean factors per term, mean factors with an exponent >= 2)."""
    s = case["system"]
    if s == "dense":
        return case["n"] * case["terms"], case["k"], case["k"] * (1 - 1 / case["e"])
    if s == "cyclic10":
        return 92, 5.0, 0.0
    if s in ("nash8", "pieri44"):
        return case["n"] * case["terms"], 3.7, 0.0
    # the anchored random equations: mostly monomials of full degree
    return case["n"] * case["terms"], 1.7 if case["e"] == 2 else 2.3, 0.3


def work(case):
    L = case["prec"]
    if case["kind"] == "eval":
        n, p = case["n"], case["npts"]
        rows = 2 * n + 2 * n + (2 * n * n if case["jac"] else 0)
        terms, k, m = _shape(case)
        return {"bytes": 8.0 * p * (rows * L + (1 if case["t"] else 0)),
                "flops": float(p) * terms * _term_flops(L, k, m, case["jac"])}
    if case["kind"] == "track":
        n, paths = case["n"], case["paths"]
        terms, k, m = _shape(case)
        terms += 2 * n
    else:
        n, paths, terms, k, m = 10, case["paths"], 220, 2.0, 0.3
    # Newton iterations per path, from runs of these recipes: about 450 with
    # the secant, 280 with the predictor of order four, fewer for quadrics
    its = (450 if case["order"] == 1 else 280) * (0.4 if case.get("e") == 2 else 1.0)
    solve = 4 * n ** 3 * (1 if case["mixed"] or L == 1 else _FLOPS[L][0] / 6)
    per = terms * _term_flops(L, k, m, True) + solve * 2
    return {"bytes": 8.0 * paths * (2 * n * L * 2 + 1), "flops": float(paths) * its * per}


# ---------------------------------------------------------------------------
# 64-bit reference of the evaluation, term by term from the definition
# ---------------------------------------------------------------------------
def exact(case, seed):
    if case["kind"] != "eval":
        return None  # following the paths again takes minutes
    sysm = _system(case, seed)
    x, t = _points(case, seed)
    n, L, npts = case["n"], case["prec"], case["npts"]
    gamma = synth.gamma_of(sysm)
    xv = x.reshape(n, 2, L, npts).sum(dim=2)
    z = torch.complex(xv[:, 0].contiguous(), xv[:, 1].contiguous())
    deg = sysm.degrees()
    val = torch.zeros((sysm.n_eq, 2, L, npts), dtype=torch.float64, device="cuda")
    jac = torch.zeros((sysm.n_eq, n, 2, L, npts), dtype=torch.float64, device="cuda") if case["jac"] else None
    for i in range(sysm.n_eq):
        h = torch.zeros(npts, dtype=torch.complex128, device="cuda")
        row = torch.zeros((n, npts), dtype=torch.complex128, device="cuda") if case["jac"] else None
        for c, mono in sysm.terms(i):
            pw = [z[v] ** e for v, e in mono]
            whole = torch.full((npts,), c, dtype=torch.complex128, device="cuda")
            before = []
            for f in pw:
                before.append(whole)
                whole = whole * f
            h += whole
            if row is not None:
                after = None
                for q in range(len(mono) - 1, -1, -1):
                    v, e = mono[q]
                    d = before[q] if after is None else before[q] * after
                    row[v] += d * (e * z[v] ** (e - 1)) if e > 1 else d
                    after = pw[q] if after is None else after * pw[q]
        if t is not None:
            d = int(deg[i])
            s = gamma * (1.0 - t)
            h = t * h + s * (z[i] ** d - 1.0)
            if row is not None:
                row *= t
                row[i] += s * (d * z[i] ** (d - 1))
        val[i, 0, 0], val[i, 1, 0] = h.real, h.imag
        if row is not None:
            jac[i, :, 0, 0], jac[i, :, 1, 0] = row.real, row.imag
    val = val.reshape(sysm.n_eq * 2 * L, npts)
    if jac is None:
        return {"val": val}
    return {"val": val, "jac": jac.reshape(sysm.n_eq * n * 2 * L, npts)}
