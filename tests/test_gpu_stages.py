"""The split-BF16 contraction (E_{G,G} pair part, Section II.B) where a j split
holds an odd number of its 32-point stages: 2016 points in five splits of 13
stages (the last one 12), so that the last stage has no partner, the load of
the stage after it repeats it, and the points past the grid are clamped.  One,
four, eight and twelve column blocks (four and eight waves), against the FP64
oracle with the bounds of the mixed modes; and the same splits in FP32, whose
chunks are the same 32 points."""
import numpy as np
import pytest

import oracle
from gpu_util import normwise, relerr
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu

E_REL, H_ABS, V_NORM = 1e-6, 1e-5, 1e-5


@pytest.mark.parametrize("prec", ["bf16x3", "fp32"])
@pytest.mark.parametrize("n_water,n_pa", [(1, 672), (6, 112), (14, 48), (21, 32)])
def test_odd_stage_count(n_water, n_pa, prec):
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(n_water, n_pa, 71 + n_water)
    assert p.n_grid == 2016
    g, gx = oracle.problem_inputs(p)
    args = (p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C, p.rho_x, gx)
    H, _ = oracle.hessian_terms(*args)
    G = oracle.gradient(*args)
    e, _, _ = oracle.energy_potential(p.coords, p.weights, p.rho, g, p.b, p.C)
    with vv10.Plan(p, prec=prec, tiles=(5, 0)) as pl:
        out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True, energy=True)
        assert vv10.vv10_get_tiles(pl.handle)[0] == 5
        torch.cuda.synchronize()
        out = {k: v.cpu().numpy() for k, v in out.items()}
    assert relerr(out["energy"][0], e) <= E_REL
    assert np.max(np.abs(out["hess"] - H)) <= H_ABS
    assert normwise(out["grad"], G) <= V_NORM
