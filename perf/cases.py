"""Workloads of the VV10 engine whose run time is tracked.

Each case is one call sequence that a program built on the library makes,
through the public binding (``paper_2208_14639_amd.vv10``), on seeded water
clusters of the sizes that the package's own workloads, tests and benchmark
use.  ``kind`` names the sequence:

  scf       a new density on a grid: plan, energy and potential (one SCF cycle)
  gradient  a new geometry: plan, energy and potential, nuclear gradient
  hessian   a new geometry: plan, then energy, potential, Hessian terms and
            gradient from one nuclear-terms call (the benchmark's step)
  fock      the same with the Fock nuclear-derivative coefficients (what a
            coupled-perturbed SCF solver asks for besides the Hessian)
  becke     the hessian step with weights that move with the nuclei
  response  trial densities on a grid whose plan is kept (one CPSCF iteration)
  batch     many small clusters, one launch of a kept batch

``n_water`` and ``n_pa`` (points per atom) size the grid: N = 3 n_water n_pa
points, P = 9 n_water perturbations.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2208_14639_amd import inputs, vv10

F64 = torch.float64
PRECS = ("fp64", "fp32", "bf16x3")


def listed():
    c = lambda name, kind, n_water, n_pa, prec, **k: dict(name=name, kind=kind, n_water=n_water,
                                                          n_pa=n_pa, prec=prec, **k)
    return [
        # the smallest call in use: one molecule on a coarse grid, where launches and waits count
        c("scf_monomer_fp64", "scf", 1, 500, "fp64"),
        # an SCF cycle in full precision at the paper's timing system, (H2O)6
        c("scf_hexamer_fp64", "scf", 6, 1500, "fp64"),
        # an SCF cycle of a large cluster in the mixed arithmetic; odd points per atom
        c("scf_17mer_fp32", "scf", 17, 1999, "fp32"),
        # a geometry-optimisation step
        c("gradient_hexamer_bf16x3", "gradient", 6, 1500, "bf16x3"),
        # a small frequency job in full precision (two column blocks)
        c("hessian_dimer_fp64", "hessian", 2, 700, "fp64"),
        # the paper's timing system, mixed and full precision
        c("hessian_hexamer_bf16x3", "hessian", 6, 1500, "bf16x3", tiles="auto"),
        c("hessian_hexamer_fp64", "hessian", 6, 1500, "fp64", tiles="auto"),
        # ragged sizes: P = 81, and 777 points per atom leave part tiles everywhere
        c("fock_9mer_fp32", "fock", 9, 777, "fp32"),
        # the headline workload: N = 120000, P = 180
        c("hessian_20mer_bf16x3", "hessian", 20, 2000, "bf16x3", tiles="auto"),
        # atom-partitioned grids: every weight-derivative term
        c("becke_hexamer_bf16x3", "becke", 6, 1500, "bf16x3", tiles="auto"),
        # a CPSCF iteration: 54 trial densities on a kept plan, full precision
        c("response_hexamer_fp64", "response", 6, 1500, "fp64", n_t=54),
        # throughput: two dozen small clusters of uneven size in one launch
        c("batch_small_bf16x3", "batch", 6, 600, "bf16x3", n_mol=24),
    ]


def _relative_cost(case):
    """Pair work of a case relative to one FP32-rate multiply-add, for capping draws."""
    n = 3 * case["n_water"] * case["n_pa"]
    rate = {"fp64": 5.7, "fp32": 2.8, "bf16x3": 1.0}[case["prec"]]
    cols = 16 * math.ceil((case.get("n_t") or 9 * case["n_water"]) / 16)
    per_pair = {"scf": 20.0, "gradient": 50.0, "hessian": 60.0 + cols * rate,
                "fock": 60.0 + cols * rate, "becke": 60.0 + 2.5 * cols * rate,
                "response": 30.0 + cols * rate, "batch": 60.0 + cols * rate}[case["kind"]]
    return n * n * per_pair * case.get("n_mol", 1)


def draw(rng):
    """One more case: sizes spread over their logarithms, every kind and precision."""
    cap = max(_relative_cost(c) for c in listed()) / 2
    while True:
        kind = rng.choice(["scf", "scf", "gradient", "hessian", "hessian", "hessian", "fock",
                           "becke", "response", "batch"])
        case = dict(kind=kind, prec=rng.choice(PRECS),
                    n_water=round(math.exp(rng.uniform(0.0, math.log(20.4)))),
                    n_pa=round(math.exp(rng.uniform(math.log(200), math.log(2000)))))
        if kind == "response":
            case["n_t"] = round(math.exp(rng.uniform(0.0, math.log(96))))
        if kind == "becke":
            case["n_water"] = min(case["n_water"], 8)
        if kind == "batch":
            case["n_mol"] = rng.randint(3, 32)
            case["n_water"] = min(case["n_water"], 8)
            case["n_pa"] = min(case["n_pa"], 900)
        if rng.random() < 0.5:
            case["tiles"] = "auto"
        if _relative_cost(case) <= cap:
            return case


def _batch_sizes(case):
    """Waters per molecule of a batch: 1 .. n_water in turn."""
    return [1 + (5 * m) % case["n_water"] if case["n_water"] > 1 else 1
            for m in range(case["n_mol"])]


def _problem(case, seed):
    """The seeded cluster, grid, density and perturbations, on the GPU."""
    kind, dev = case["kind"], torch.device("cuda")
    d = lambda a: torch.as_tensor(a, dtype=F64).to(dev).contiguous()
    if kind in ("hessian", "fock", "gradient"):
        p = inputs.make_problem_on_device(case["n_water"], case["n_pa"], seed, torch, dev)
    else:
        p = inputs.make_problem(case["n_water"], case["n_pa"], seed,
                                with_derivatives=kind == "becke",
                                weights="becke" if kind == "becke" else "atomic")
    trial = inputs.trial_densities(p, case["n_t"], seed + 1) if kind == "response" else None
    p = dataclasses.replace(
        p, coords=d(p.coords), weights=d(p.weights), rho=d(p.rho), grad_rho=d(p.grad_rho),
        atom_of=torch.as_tensor(p.atom_of).to(dev),
        rho_x=None if p.rho_x is None else d(p.rho_x),
        grad_rho_x=None if p.grad_rho_x is None else d(p.grad_rho_x),
        w_x=None if p.w_x is None else d(p.w_x))
    return p, None if trial is None else tuple(d(t) for t in trial)


def prepare(case, seed):
    if case["kind"] == "batch":
        probs = [inputs.make_problem(k, case["n_pa"], seed + 97 * m)
                 for m, k in enumerate(_batch_sizes(case))]
        return dict(case=case, batch=vv10.Batch(probs, prec=case["prec"], tiles=case.get("tiles")))
    p, trial = _problem(case, seed)
    state = dict(case=case, problem=p, trial=trial)
    if case["kind"] == "response":
        # the plan a CPSCF solver keeps over its iterations
        state["plan"] = vv10.Plan(p, prec=case["prec"], tiles=case.get("tiles"))
    return state


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "batch":
        energy, blocks = state["batch"].run()
        return {"energy": energy, "hess": blocks}
    if kind == "response":
        f_rho, f_gamma = state["plan"].trial_response(*state["trial"])
        return {"f_rho_t": f_rho, "f_gamma_t": f_gamma}
    p = state["problem"]
    with vv10.Plan(p, prec=case["prec"], tiles=case.get("tiles")) as plan:
        if kind == "scf" or kind == "gradient":
            energy, f_rho, f_gamma = plan.energy_potential()
            out = {"energy": energy, "f_rho": f_rho, "f_gamma": f_gamma}
            if kind == "gradient":
                out["grad"] = plan.gradient(p.rho_x, p.grad_rho_x)
            return out
        return plan.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True, energy=True,
                                  potential=True, fock=kind == "fock", w_x=p.w_x)


def _one_work(kind, n, P):
    """Bytes (each input and output once) and flops of one cluster of a case:
    26 flops per pair for E, U, W; about 79 with A, B, C and the grid sums; 8
    per pair and column for the contraction, 6 more with moving weights."""
    data, pot = n * (8 * 8 + 4), 8 * (2 * n + 1)
    if kind == "scf":
        return data + pot, 26.0 * n * n
    if kind == "gradient":
        return data + pot + 32 * n * P + 8 * P, 36.0 * n * n
    if kind == "response":
        return data + 48 * n * P, 8.0 * n * n * P
    b, f = data + pot + 32 * n * P + 8 * P * (P + 1), n * n * (79.0 + 8.0 * P)
    if kind == "fock":
        b += 16 * n * P
    if kind == "becke":
        b, f = b + 8 * n * P, f + 6.0 * n * n * P
    return b, f


def work(case):
    if case["kind"] == "batch":
        one = [_one_work("hessian", 3 * k * case["n_pa"], 9 * k) for k in _batch_sizes(case)]
    else:
        n, P = 3 * case["n_water"] * case["n_pa"], case.get("n_t") or 9 * case["n_water"]
        one = [_one_work(case["kind"], n, P)]
    return {"bytes": sum(b for b, _ in one), "flops": sum(f for _, f in one)}


# ---------------------------------------------------------------------------
# The same quantities in plain 64-bit torch, from the equations of
# arXiv 2208.14639, Section II.
# ---------------------------------------------------------------------------
def _points(p):
    """omega, kappa and their partials, and the derived per-point factors."""
    r, G = p.rho, p.grad_rho
    gam = (G * G).sum(1)
    pi = math.pi
    S = p.C * gam ** 2 / r ** 4 + 4 * pi / 3 * r
    Sr = 4 * pi / 3 - 4 * p.C * gam ** 2 / r ** 5
    Sg = 2 * p.C * gam / r ** 4
    Srr, Srg, Sgg = 20 * p.C * gam ** 2 / r ** 6, -8 * p.C * gam / r ** 5, 2 * p.C / r ** 4
    om = S.sqrt()
    ka = p.b * 1.5 * pi * (r / (9 * pi)) ** (1 / 6)
    q = dict(r=r, w=p.weights, a=p.weights * r, om=om, ka=ka, omr=Sr / (2 * om), omg=Sg / (2 * om),
             kar=ka / (6 * r), karr=-5 * ka / (36 * r * r))
    q["omrr"] = (Srr / 2 - q["omr"] ** 2) / om
    q["omrg"] = (Srg / 2 - q["omr"] * q["omg"]) / om
    q["omgg"] = (Sgg / 2 - q["omg"] ** 2) / om
    q["c"] = r * q["kar"]
    return q


def _pair_sums(p, q, L=None, v=None, grid=False):
    """Row sums over all pairs: the integrals E..C; with L = (rho^x, gamma^x)
    the contraction's channels Yp, Yq [N, P]; with v = w^x rho the weight rows;
    with grid the grid-position sums [N, atoms, 3] and the D sums."""
    n = p.n_grid
    own = torch.nn.functional.one_hot(p.atom_of.long(), p.n_atom).to(F64)
    out = {}

    def put(k, lo, val):
        if k not in out:
            out[k] = val.new_empty((n,) + val.shape[1:])
        out[k][lo:lo + val.shape[0]] = val

    if L is not None:
        wr = (q["w"] * q["r"])[:, None]
        xp = q["w"][:, None] * L[0]
        xq = wr * (q["omr"][:, None] * L[0] + q["omg"][:, None] * L[1])
    step = max(16, min(1024, 12_000_000 // n))
    for lo in range(0, n, step):
        s = slice(lo, min(n, lo + step))
        at = lambda k: q[k][s, None]
        d = [p.coords[None, :, k] - p.coords[s, None, k] for k in range(3)]
        R2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        ig = 1 / (at("om") * R2 + at("ka"))
        igp = 1 / (q["om"] * R2 + q["ka"])
        isum = ig * igp / (ig + igp)                    # 1 / (g + g')
        phi = -1.5 * ig * igp * isum
        h = isum + ig
        ap = q["a"] * phi
        m = isum ** 2 + isum * ig + ig ** 2
        for k, t in (("E", ap), ("U", -ap * h), ("W", -ap * R2 * h), ("A", 2 * ap * m),
                     ("B", 2 * ap * m * R2), ("C", 2 * ap * m * R2 ** 2)):
            put(k, lo, t.sum(1))
        pg = -phi * h
        if L is not None:
            pgg = 2 * phi * (ig * igp + isum ** 2)
            t1 = -phi * (igp + isum) + at("c") * pgg
            put("Yp", lo, (phi + at("c") * pg + q["c"] * t1) @ xp + (R2 * t1) @ xq)
            put("Yq", lo, (R2 * (pg + q["c"] * pgg)) @ xp + (R2 ** 2 * pgg) @ xq)
        if v is not None:
            put("Ypv", lo, (phi + at("c") * pg) @ v)
            put("Yqv", lo, (R2 * pg) @ v)
            put("Yvv", lo, phi @ v)
        if grid:
            Ti, Tj, Ts = at("om") * ig, q["om"] * igp, (at("om") + q["om"]) * isum
            T = Ti + Tj + Ts
            TQ = T * h + Ti * ig + Ts * isum
            for k, t in (("Egr", -2 * ap * T), ("Ugr", 2 * ap * TQ), ("Wgr", 2 * ap * (R2 * TQ - h))):
                put(k, lo, torch.stack([(t * x) @ own for x in d], 2))
            S = T ** 2 + Ti ** 2 + Tj ** 2 + Ts ** 2
            dd = [[(-4 * ap * S * d[a] * d[b] + (2 * ap * T if a == b else 0)) @ own
                   for b in range(3)] for a in range(3)]
            put("D", lo, torch.stack([torch.stack(x, 2) for x in dd], 2))
    return out


def _response(q, t, L):
    """Sum over j of the second-derivative matrices with (rho^x, gamma^x), [N, P] each."""
    g = {k: x[:, None] for k, x in {**q, **{k: t[k] for k in "EUWABC"}}.items()}
    rx, gx = L
    dk, dw = g["kar"] * rx, g["omr"] * rx + g["omg"] * gx
    loc_r = (g["U"] * dk + g["W"] * dw + rx * (g["kar"] * g["U"] + g["omr"] * g["W"])
             + g["r"] * (g["kar"] * (g["A"] * dk + g["B"] * dw)
                         + g["omr"] * (g["B"] * dk + g["C"] * dw))
             + g["r"] * (g["karr"] * rx * g["U"] + (g["omrr"] * rx + g["omrg"] * gx) * g["W"]))
    loc_g = (rx * g["omg"] * g["W"] + g["r"] * g["omg"] * (g["B"] * dk + g["C"] * dw)
             + g["r"] * (g["omrg"] * rx + g["omgg"] * gx) * g["W"])
    return t["Yp"] + g["r"] * g["omr"] * t["Yq"] + loc_r, g["r"] * g["omg"] * t["Yq"] + loc_g


def _exact_problem(kind, p, trial=None):
    q = _points(p)
    beta = (3 / p.b ** 2) ** 0.75 / 32
    gamma_x = lambda g: 2 * torch.einsum("nk,xnk->nx", p.grad_rho, g)
    if kind == "response":
        L = (trial[0].T.contiguous(), gamma_x(trial[1]))
        fr, fg = _response(q, _pair_sums(p, q, L), L)
        return {"f_rho_t": fr.T.contiguous(), "f_gamma_t": fg.T.contiguous()}
    L = v = wx = None
    M, P = p.n_atom, p.n_pert
    own = torch.nn.functional.one_hot(p.atom_of.long(), M).to(F64)
    if kind != "scf":
        L = (p.rho_x.T.contiguous(), gamma_x(p.grad_rho_x))
    if p.w_x is not None:
        # the owner atom's entry from translational invariance
        wx = p.w_x.T.reshape(-1, M, 3) * (1 - own)[:, :, None]
        wx = (wx - own[:, :, None] * wx.sum(1, keepdim=True)).reshape(-1, P)
        v = wx * p.rho[:, None]
    t = _pair_sums(p, q, L if kind != "gradient" else None, v, grid=kind != "scf")
    fr = beta + t["E"] + q["r"] * (q["kar"] * t["U"] + q["omr"] * t["W"])
    fg = q["r"] * q["omg"] * t["W"]
    out = {"energy": (q["a"] * (beta + t["E"] / 2)).sum().reshape(1), "f_rho": fr, "f_gamma": fg}
    if kind == "scf":
        return out
    for k in ("Egr", "Ugr", "Wgr"):     # own slots by invariance
        z = t[k] * (1 - own)[:, :, None]
        t[k] = (z - own[:, :, None] * z.sum(1, keepdim=True)).reshape(-1, P)
    w = q["w"][:, None]
    grad = (w * (fr[:, None] * L[0] + fg[:, None] * L[1])).sum(0)
    # E_gr[A] = sum over i in A of a_i E^{A gr}_i
    grad = grad + torch.einsum("nm,nmk->mk", own * q["a"][:, None], t["Egr"].view(-1, M, 3)).reshape(-1)
    if wx is not None:
        grad = grad + wx.T @ (q["r"] * (beta + t["E"]))
    out["grad"] = grad
    if kind == "gradient":
        return out
    Yr, Yg = _response(q, t, L)
    r, omr, omg = (q[k][:, None] for k in ("r", "omr", "omg"))
    Zr = t["Egr"] + q["c"][:, None] * t["Ugr"] + r * omr * t["Wgr"]
    Zg = r * omg * t["Wgr"]
    H = L[0].T @ (w * (Yr + 2 * Zr)) + L[1].T @ (w * (Yg + 2 * Zg))
    if wx is not None:
        Wr, Wg = t["Ypv"] + r * omr * t["Yqv"], r * omg * t["Yqv"]
        H = H + 2 * (L[0].T @ (w * Wr + wx * fr[:, None]) + L[1].T @ (w * Wg + wx * fg[:, None]))
        H = H + wx.T @ (r * (t["Yvv"] + 2 * t["Egr"]))
    DS = torch.einsum("na,nbxy->axby", own * q["a"][:, None], t["D"])
    blk = torch.eye(M, dtype=F64, device=DS.device)[:, None, :, None]
    DS = DS * (1 - blk)
    DS = DS - blk * DS.sum(2, keepdim=True)
    H = H + DS.reshape(P, P)
    out["hess"] = (H + H.T) / 2
    if kind == "fock":
        out["fock_rho"] = (Yr + Zr).T.contiguous()
        out["fock_gamma"] = (Yg + Zg).T.contiguous()
    return out


def exact(case, seed):
    if case["kind"] == "batch":
        got = []
        for m, k in enumerate(_batch_sizes(case)):
            one = dict(case, kind="hessian", n_water=k)
            p = inputs.make_problem(k, case["n_pa"], seed + 97 * m)
            d = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
            p = dataclasses.replace(p, **{f: d(getattr(p, f)) for f in (
                "coords", "weights", "rho", "grad_rho", "rho_x", "grad_rho_x", "atom_of")})
            got.append(_exact_problem(one["kind"], p))
        return {"energy": torch.cat([g["energy"] for g in got]), "hess": [g["hess"] for g in got]}
    n = 3 * case["n_water"] * case["n_pa"]
    if n > (110000 if case["kind"] == "scf" else 45000):
        return None      # the pair passes in plain torch would take too long
    return _exact_problem(case["kind"], *_problem(case, seed))
