"""Counts of partial pair integrals around the lengths that the potential kernel
loads together (8 and 16): atom groups of the grid and gradient passes, j splits of
the pair pass, against the FP64 oracle; a partial left out or added twice would
change the potential far beyond the tolerance."""
import pytest

import oracle
from gpu_util import normwise, problem, relerr

pytestmark = pytest.mark.gpu

TOL64 = 1e-10


def check(p, e, fr, fg):
    g = oracle.gamma(p.grad_rho)
    e0, fr0, fg0 = oracle.energy_potential(p.coords, p.weights, p.rho, g, p.b, p.C)
    assert relerr(e.item(), e0) < TOL64
    assert normwise(fr.cpu().numpy(), fr0) < TOL64
    assert normwise(fg.cpu().numpy(), fg0) < TOL64


@pytest.mark.parametrize("groups", [1, 2, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33])
def test_atom_groups(groups):
    from paper_2208_14639_amd import vv10
    p = problem(11, 21, 311)
    with vv10.Plan(p, prec="fp64", tiles=(0, groups)) as pl:
        out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, energy=True, potential=True)
        check(p, out["energy"], out["f_rho"], out["f_gamma"])
    with vv10.Plan(p, prec="fp64", tiles=(0, groups)) as pl:
        pl.gradient(p.rho_x, p.grad_rho_x)          # three rows a group
        check(p, *pl.energy_potential())
    with vv10.Plan(p, prec="fp64", tiles=(0, groups)) as pl:
        pl.energy_potential()
        out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, energy=True, potential=True)   # A, B, C alone
        check(p, out["energy"], out["f_rho"], out["f_gamma"])


@pytest.mark.parametrize("n_pa", [85, 300, 600, 683, 768, 1280, 1365, 1366])
def test_pair_splits(n_pa):
    """1 to 16 splits of one water's grid."""
    from paper_2208_14639_amd import vv10
    p = problem(1, n_pa, 17)
    with vv10.Plan(p, prec="fp64") as pl:
        check(p, *pl.energy_potential())
