"""The grid pass (Section II.B grid-position intermediates, with the pair
integrals) where an atom's 64-point chunks do not divide among the four waves
of a workgroup: 1 to 6 chunks per atom, whole and ragged, in one atom group,
one per atom and between; energy, potential, Hessian and Fock coefficients
against the FP64 oracle, in FP64 and FP32."""
import functools

import numpy as np
import pytest

import oracle
from gpu_util import normwise, relerr
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu

BOUNDS = {"fp64": dict(energy=1e-10, pot=1e-10, hess=None, fock=1e-10),
          "fp32": dict(energy=1e-6, pot=1e-5, hess=1e-5, fock=5e-5)}


@functools.lru_cache(maxsize=8)
def case(n_pa):
    p = inputs.make_problem(2, n_pa, 500 + n_pa)
    g, gx = oracle.problem_inputs(p)
    args = (p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C, p.rho_x, gx)
    H, _ = oracle.hessian_terms(*args)
    e, fr, fg = oracle.energy_potential(p.coords, p.weights, p.rho, g, p.b, p.C)
    return p, e, fr, fg, H, oracle.fock_nuclear_terms(*args)


@pytest.mark.parametrize("bgroups", [1, 4, 6])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_pa", [1, 63, 64, 65, 193, 256, 257, 383])
def test_chunks(n_pa, prec, bgroups):
    import torch
    from paper_2208_14639_amd import vv10
    p, e, fr, fg, H, fock = case(n_pa)
    b = BOUNDS[prec]
    with vv10.Plan(p, prec=prec, tiles=(0, bgroups)) as pl:
        out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, fock=True, energy=True, potential=True)
        torch.cuda.synchronize()
        out = {k: v.cpu().numpy() for k, v in out.items()}
    assert relerr(out["energy"][0], e) <= b["energy"]
    assert normwise(out["f_rho"], fr) <= b["pot"] and normwise(out["f_gamma"], fg) <= b["pot"]
    if prec == "fp64":
        assert normwise(out["hess"], H) <= 1e-10
    else:
        assert np.max(np.abs(out["hess"] - H)) <= b["hess"]
    assert normwise(out["fock_rho"], fock[0]) <= b["fock"]
    assert normwise(out["fock_gamma"], fock[1]) <= b["fock"]
