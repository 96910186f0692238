"""The grid pass and the contraction of a small call as one launch (one to four
column blocks; in FP64 each number of column quads) against the same passes
apart, which a call with timed stages runs: bit for bit, with the pair integrals
formed by the call or, E, U and W, held by the plan; at ragged sizes, with one
split and several, and either side of the limit of 2560 grid units."""
import numpy as np
import pytest

from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("n_water,n_pa", [(1, 9), (2, 131), (3, 100), (4, 77), (5, 64), (6, 150),
                                          (5, 750), (6, 500)])
def test_together_equals_apart(n_water, n_pa, prec):
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(n_water, n_pa, 31 + n_water)
    res = []
    for timed in (False, True):
        for first in (False, True):
            with vv10.Plan(p, prec=prec) as pl:
                if timed:
                    vv10.vv10_set_timing(pl.handle, 1)
                if first:
                    pl.energy_potential()
                out = pl.nuclear_terms(p.rho_x, p.grad_rho_x, hess=True, grad=True, resp=True,
                                       fock=True, energy=True, potential=True)
                torch.cuda.synchronize()
                res.append({k: v.cpu().numpy() for k, v in out.items()})
    for a, b in ((0, 2), (1, 3)):
        for k in res[a]:
            assert np.isfinite(res[a][k]).all()
            assert np.array_equal(res[a][k], res[b][k]), (k, prec)
