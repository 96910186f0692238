"""The gradient's point sums: one launch for grids of at most 1024 points, slices
beyond, whose sums share the buffer of the atom groups' partial integrals: as many
as it has room for, and room for one slice of every atom where the atoms outnumber
its points (one atom group)."""
import types

import numpy as np
import pytest

import oracle
from gpu_util import normwise
from paper_2208_14639_amd import inputs


@pytest.mark.parametrize("n,n_atom", [(1, 9000), (1050, 9000), (1050, 400), (27000, 18)])
def test_footprint_holds_a_slice_of_every_atom(n, n_atom):
    from paper_2208_14639_amd import vv10
    npad, ntiles = (n + 255) // 256 * 256, (n + 63) // 64 + n_atom
    groups = max(1, min(n_atom, -(-8192 // ntiles)))
    want = 8 * (3 * ntiles * n_atom + 3 * max(groups * npad, n_atom) + 3 * npad)
    assert vv10.vv10_gradient_footprint_bytes(n, n_atom) == want


@pytest.mark.gpu
@pytest.mark.parametrize("weights", ["atomic", "becke"])
@pytest.mark.parametrize("n_pa,n_atom,room", [(85, 3, 256), (341, 3, 341), (342, 3, 426),
                                              (350, 400, 3), (350, 1280, 1), (350, 1300, 0)])
def test_against_the_oracle(n_pa, n_atom, room, weights):
    import torch
    from paper_2208_14639_amd import vv10
    p = inputs.make_problem(1, n_pa, 71, weights=weights)
    npad = (p.n_grid + 255) // 256 * 256
    if n_atom > p.n_atom:
        assert npad // n_atom == room           # what one atom group's buffer holds
    extra = 3 * (n_atom - p.n_atom)
    rng = np.random.default_rng(72)
    more = lambda a, *s: np.concatenate([a, 0.1 * rng.normal(size=(extra, *s))])
    q = types.SimpleNamespace(
        n_grid=p.n_grid, n_atom=n_atom, coords=p.coords, weights=p.weights, atom_of=p.atom_of,
        rho=p.rho, grad_rho=p.grad_rho, b=p.b, C=p.C, rho_x=more(p.rho_x, p.n_grid),
        grad_rho_x=more(p.grad_rho_x, p.n_grid, 3))
    w_x = more(p.w_x, p.n_grid) if weights == "becke" else None
    if w_x is not None:                          # the owner's entries, from the others'
        w = w_x.reshape(n_atom, 3, -1)
        own, i = p.atom_of, np.arange(p.n_grid)
        w[own, :, i] = 0.0
        w[own, :, i] = -w.sum(0).T
    g, gx = oracle.problem_inputs(q)
    G0 = oracle.gradient(q.atom_of, n_atom, q.coords, q.weights, q.rho, g, q.b, q.C, q.rho_x, gx, w_x=w_x)
    with vv10.Plan(q, prec="fp64", tiles=(0, 1)) as pl:
        got = [pl.gradient(q.rho_x, q.grad_rho_x, w_x=w_x) for _ in range(2)]
        torch.cuda.synchronize()
    for G in got:
        assert normwise(G.cpu().numpy(), G0) < 1e-10
