"""FP64 contraction with 1 to 4 quads of columns in the last 16-column block
(v_mfma_f64_4x4x4 past a multiple of 16), through the trial response
(Section II.B, f^{rho,t}, f^{gamma,t}), which takes any column count: one
column group from 1 to 128 columns, two and three groups whose last block
holds 1 to 16 columns or none, all against the FP64 oracle; and screening at
tau = 0 and at a tau that drops nothing (bitwise the same)."""
import functools

import numpy as np
import pytest

import oracle
from gpu_util import normwise
from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu

TOL64 = 1e-10


@functools.lru_cache(maxsize=1)
def problem():
    return inputs.make_problem(1, 100, 909)


@pytest.mark.parametrize("n_t", [1, 4, 5, 9, 12, 13, 16, 17, 54, 61, 81, 116, 121, 125, 128,
                                 129, 135, 139, 142, 257, 260])
def test_trial_columns(n_t):
    import torch
    from paper_2208_14639_amd import vv10
    p = problem()
    rt, gt = inputs.trial_densities(p, n_t, 4)
    g = oracle.gamma(p.grad_rho)
    want = oracle.response_rows(0, p.n_grid, p.coords, p.weights, p.rho, g, p.b, p.C, rt,
                                oracle.gamma_x(p.grad_rho, gt))
    got = {}
    for tau in (0.0, 1e-300):
        with vv10.Plan(p, prec="fp64", screening=tau) as pl:
            got[tau] = [t.cpu().numpy() for t in pl.trial_response(rt, gt)]
    for a, b, w in zip(got[0.0], got[1e-300], want):
        assert normwise(a, w) < TOL64
        assert np.array_equal(a, b)
