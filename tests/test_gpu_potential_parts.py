"""Where the pair integrals behind the potential come from (Section II.A): the
pair pass's splits, the grid pass's atom groups (all six rows, or A, B, C beside
E, U, W that the plan holds), the gradient pass's, or the plan itself; and the
energy's block sums, added by the block that ends last.  From one 256-point
block (one split) to blocks of several; every order of calls on one plan, twice,
against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import normwise, relerr
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu

TOL64 = 1e-10
ORDERS = ["ee", "en", "ne", "gen", "eng", "nn"]


@pytest.mark.parametrize("n_water,n_pa", [(1, 8), (1, 85), (1, 171), (2, 350)])
def test_sources_of_the_integrals(n_water, n_pa):
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(n_water, n_pa, 91 + n_pa)
    g, gx = oracle.problem_inputs(p)
    e0, fr0, fg0 = oracle.energy_potential(p.coords, p.weights, p.rho, g, p.b, p.C)
    args = (p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C, p.rho_x, gx)
    H0, _ = oracle.hessian_terms(*args)
    G0 = oracle.gradient(*args)
    for order in ORDERS:
        with vv10.Plan(p, prec="fp64") as pl:
            for call in order:
                if call == "g":
                    G = pl.gradient(p.rho_x, p.grad_rho_x)
                    assert normwise(G.cpu().numpy(), G0) < TOL64, order
                    continue
                if call == "e":
                    e, fr, fg = pl.energy_potential()
                else:
                    out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True,
                                           energy=True, potential=True)
                    e, fr, fg = out["energy"], out["f_rho"], out["f_gamma"]
                    assert normwise(out["hess"].cpu().numpy(), H0) < TOL64, order
                    assert normwise(out["grad"].cpu().numpy(), G0) < TOL64, order
                torch.cuda.synchronize()
                assert relerr(e.cpu().numpy()[0], e0) < TOL64, order
                assert normwise(fr.cpu().numpy(), fr0) < TOL64, order
                assert normwise(fg.cpu().numpy(), fg0) < TOL64, order
