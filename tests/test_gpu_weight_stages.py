"""The fused main and weight contraction in split-BF16 (Section II.B E_{G,G},
E_{G,w}, E_{w,w} pair parts) at each of its one to four column blocks, where a
j split holds an odd number of its 32-point stages: 2016 points in five splits
of 13 stages (the last one 12), so that the last stage has no partner, the load
of the stage after it repeats it and the points past the grid are clamped.
Against the FP64 oracle with the bounds of the mixed modes."""
import numpy as np
import pytest

import oracle
from gpu_util import normwise
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu

H_ABS, V_NORM, COEF_NORM = 1e-5, 1e-5, 1e-6


@pytest.mark.parametrize("n_water,n_pa", [(1, 672), (2, 336), (4, 168), (6, 112)])
def test_odd_stage_count_with_weights(n_water, n_pa):
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(n_water, n_pa, 83 + n_water, weights="becke")
    assert p.n_grid == 2016
    g, gx = oracle.problem_inputs(p)
    args = (p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C, p.rho_x, gx)
    H, _ = oracle.hessian_terms(*args, w_x=p.w_x)
    G = oracle.gradient(*args, w_x=p.w_x)
    coef = oracle.weight_coefficients(p.coords, p.weights, p.rho, g, p.b, p.C)
    with vv10.Plan(p, prec="bf16x3", tiles=(5, 0)) as pl:
        out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True, w_x=p.w_x,
                               w_coef=True)
        assert vv10.vv10_get_tiles(pl.handle)[0] == 5
        torch.cuda.synchronize()
        out = {k: v.cpu().numpy() for k, v in out.items()}
    assert np.max(np.abs(out["hess"] - H)) <= H_ABS
    assert normwise(out["grad"], G) <= V_NORM
    assert normwise(out["w_coef"], coef) <= COEF_NORM
