"""The contraction's own kernels (one to four column blocks) on splits with an odd
number of 32-point stages, which a small call runs only apart from its grid pass:
with timed stages, on a plan that holds the pair integrals, and screened; and the
one launch of both on the same splits.  2016 points in five splits of 13 stages (the
last one 12) and in three of 21, against the FP64 oracle with each mode's bounds;
timed and held equal the one launch bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import normwise
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("splits", [5, 3])
@pytest.mark.parametrize("n_water,n_pa", [(1, 672), (3, 224), (4, 168), (7, 96)])
def test_odd_stages_apart(n_water, n_pa, splits, prec):
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(n_water, n_pa, 171 + n_water)
    assert p.n_grid == 2016
    g, gx = oracle.problem_inputs(p)
    H, _ = oracle.hessian_terms(p.atom_of, p.n_atom, p.coords, p.weights, p.rho, g, p.b, p.C,
                                p.rho_x, gx)
    got = {}
    for how in ("one launch", "timed", "screened"):
        with vv10.Plan(p, prec=prec, tiles=(splits, 0),
                       screening=1e-30 if how == "screened" else 0.0) as pl:
            if how == "timed":
                vv10.vv10_set_timing(pl.handle, 1)
            got[how] = pl.hessian_terms(p.rho_x, p.grad_rho_x)["hess"].cpu().numpy()
            assert vv10.vv10_get_tiles(pl.handle)[0] == splits
            if how == "timed":
                assert vv10.vv10_stage_times(pl.handle)["contract"] > 0
            if how == "one launch":
                got["held"] = pl.hessian_terms(p.rho_x, p.grad_rho_x)["hess"].cpu().numpy()
            torch.cuda.synchronize()
    for how, h in got.items():
        if prec == "fp64":
            assert normwise(h, H) < 1e-10, how
        else:
            assert np.max(np.abs(h - H)) <= 1e-5, how
    assert np.array_equal(got["timed"], got["one launch"])
    assert np.array_equal(got["held"], got["one launch"])
