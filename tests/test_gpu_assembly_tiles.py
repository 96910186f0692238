"""The assembly GEMM's tile sizes (1 to 4 column blocks a side, uneven last
tiles: 5 = 3 + 2 and 7 = 4 + 3 blocks), with and without the rows of moving
weights, on grids from fewer points than slices up; and the gradient's point
slices on the same grids, with atoms that own no points: against the FP64
oracle."""
import types

import numpy as np
import pytest

import oracle
from gpu_util import normwise
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu

TOL64 = 1e-10


@pytest.mark.parametrize("weights", ["atomic", "becke"])
@pytest.mark.parametrize("n_water,n_pa", [(1, 5), (2, 60), (5, 21), (7, 23), (8, 11), (11, 10)])
def test_tiles_and_slices(n_water, n_pa, weights):
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(n_water, n_pa, 61 + n_water, weights=weights)
    g, gx = oracle.problem_inputs(p)
    args = (p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C, p.rho_x, gx)
    w_x = p.w_x if weights == "becke" else None
    H0, _ = oracle.hessian_terms(*args, w_x=w_x)
    G0 = oracle.gradient(*args, w_x=w_x)
    with vv10.Plan(p, prec="fp64") as pl:
        out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True, w_x=w_x)
        G = pl.gradient(p.rho_x, p.grad_rho_x, w_x=w_x)
        torch.cuda.synchronize()
    assert normwise(out["hess"].cpu().numpy(), H0) < TOL64
    assert normwise(out["grad"].cpu().numpy(), G0) < TOL64
    assert normwise(G.cpu().numpy(), G0) < TOL64


def test_gradient_with_more_atoms_than_points():
    """600 atoms, 12 of them with points: one slice, no tile of most atoms."""
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(4, 6, 67)
    n_atom, extra = 600, 3 * (600 - p.n_atom)
    rng = np.random.default_rng(68)
    q = types.SimpleNamespace(
        n_grid=p.n_grid, n_atom=n_atom, coords=p.coords, weights=p.weights, atom_of=p.atom_of,
        rho=p.rho, grad_rho=p.grad_rho, b=p.b, C=p.C,
        rho_x=np.concatenate([p.rho_x, rng.normal(size=(extra, p.n_grid))]),
        grad_rho_x=np.concatenate([p.grad_rho_x, rng.normal(size=(extra, p.n_grid, 3))]))
    g, gx = oracle.problem_inputs(q)
    G0 = oracle.gradient(q.atom_of, n_atom, q.coords, q.weights, q.rho, g, q.b, q.C, q.rho_x, gx)
    with vv10.Plan(q, prec="fp64") as pl:
        G = pl.gradient(q.rho_x, q.grad_rho_x)
        torch.cuda.synchronize()
    assert normwise(G.cpu().numpy(), G0) < TOL64
