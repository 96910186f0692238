"""Coarse grids, on which a wave of the grid pass takes whole atoms: sizes on both
sides of the rule (points per atom against atoms), atom counts that leave part of
the waves without an atom, atoms without points, one group and as many as atoms,
with and without the pair integrals and with moving weights, against the FP64
oracle; the batch equals the single path bit for bit."""
import dataclasses

import numpy as np
import pytest

import oracle
from gpu_util import normwise, relerr
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu


def groups(pl):
    from paper_2208_14639_amd import vv10
    return vv10.vv10_get_tiles(pl.handle)[1]


def thinned(p, keep):
    """p with the first keep[k mod len(keep)] points of every atom k."""
    rank = np.arange(p.n_grid) - np.searchsorted(p.atom_of, p.atom_of)
    sel = np.flatnonzero(rank < np.asarray(keep)[p.atom_of % len(keep)])
    cut = lambda a: np.ascontiguousarray(a[sel])
    return dataclasses.replace(
        p, **{f: cut(getattr(p, f)) for f in ("atom_of", "offsets", "coords", "weights", "rho",
                                              "grad_rho", "radii")},
        rho_x=np.ascontiguousarray(p.rho_x[:, sel]),
        grad_rho_x=np.ascontiguousarray(p.grad_rho_x[:, sel]))


@pytest.mark.parametrize("waters,n_pa,want", [(1, 13, 1), (1, 14, 3), (2, 27, 2), (2, 28, 6),
                                              (7, 33, 6), (9, 121, 7), (9, 122, 27), (20, 20, 15)])
def test_groups_follow_the_rule(waters, n_pa, want):
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(waters, n_pa, 5, with_derivatives=False)
    with vv10.Plan(p, prec="fp64") as pl:
        assert groups(pl) == want


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("waters,n_pa,keep,bgroups", [
    (2, 24, (24,), 0), (3, 40, (40,), 0), (5, 66, (66, 1, 64, 65), 0), (7, 33, (33, 0, 7), 0),
    (6, 70, (70,), 1), (6, 70, (70, 0, 0, 0, 70), 18), (11, 20, (20,), 0)])
def test_against_the_oracle(waters, n_pa, keep, bgroups, prec):
    import torch
    from paper_2208_14639_amd import vv10
    p = thinned(inputs.make_problem(waters, n_pa, 40 + waters), keep)
    g, gx = oracle.problem_inputs(p)
    args = (p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C, p.rho_x, gx)
    H0, _ = oracle.hessian_terms(*args)
    G0 = oracle.gradient(*args)
    e0, fr0, _ = oracle.energy_potential(p.coords, p.weights, p.rho, g, p.b, p.C)
    tiles = (0, bgroups) if bgroups else None
    with vv10.Plan(p, prec=prec, tiles=tiles) as pl:
        got = [pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True, energy=True,
                                potential=True) for _ in range(2)]   # the second without integrals
        grads = [o["grad"] for o in got] + [pl.gradient(p.rho_x, p.grad_rho_x)]
    with vv10.Plan(p, prec=prec, tiles=tiles) as pl:
        grads.append(pl.gradient(p.rho_x, p.grad_rho_x))             # forms E, U, W itself
        torch.cuda.synchronize()
    for o in got:
        H = o["hess"].cpu().numpy()
        if prec == "fp64":
            assert normwise(H, H0) < 1e-10
            assert normwise(o["f_rho"].cpu().numpy(), fr0) < 1e-10
            assert relerr(o["energy"].item(), e0) < 1e-10
        else:
            assert np.max(np.abs(H - H0)) <= 1e-5
            assert normwise(o["f_rho"].cpu().numpy(), fr0) <= 1e-5
            assert relerr(o["energy"].item(), e0) <= 1e-6
    for G in grads:
        assert normwise(G.cpu().numpy(), G0) < (1e-10 if prec == "fp64" else 1e-5)


def test_moving_weights():
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(4, 30, 44, weights="becke")
    g, gx = oracle.problem_inputs(p)
    H0, _ = oracle.hessian_terms(p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C,
                                 p.rho_x, gx, w_x=p.w_x)
    with vv10.Plan(p, prec="fp64") as pl:
        o = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True, w_x=p.w_x)
        torch.cuda.synchronize()
    assert normwise(o["hess"].cpu().numpy(), H0) < 1e-10


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_batch_equals_single(prec):
    import torch
    from paper_2208_14639_amd import vv10
    probs = [inputs.make_problem(k, n_pa, 60 + k) for k, n_pa in ((6, 30), (2, 200), (14, 25), (9, 70))]
    with vv10.Batch(probs, prec=prec) as b:
        _, blocks = b.run()
        torch.cuda.synchronize()
        got = [h.cpu().numpy() for h in blocks]
    for p, h in zip(probs, got):
        with vv10.Plan(p, prec=prec) as pl:
            ref = pl.hessian_terms(p.rho_x, p.grad_rho_x)["hess"]
            torch.cuda.synchronize()
        assert np.array_equal(h, ref.cpu().numpy()), (p.n_atom, prec)
