"""j splits of grids that do not fill the chip: in FP64 as many as leave 256 points
each (1 to 5 column blocks, which hold different numbers of workgroups a CU), and
the Hessian against the FP64 oracle."""
import pytest

from gpu_util import normwise, oracle_hessian, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waters,n_pa,want", [(1, 80, 1), (1, 200, 3), (1, 300, 4), (2, 100, 3),
                                              (3, 70, 3), (4, 50, 3), (4, 60, 3), (5, 30, 2),
                                              (5, 51, 3), (8, 32, 3)])
def test_splits_of_small_grids(waters, n_pa, want):
    from paper_2208_14639_amd import vv10
    p = problem(waters, n_pa, 81)
    with vv10.Plan(p, prec="fp64") as pl:
        assert vv10.vv10_get_tiles(pl.handle)[0] == want
        H = pl.hessian_terms(p.rho_x, p.grad_rho_x)["hess"]
        again = pl.hessian_terms(p.rho_x, p.grad_rho_x)["hess"]
    assert normwise(H.cpu().numpy(), oracle_hessian(waters, n_pa, 81)[0]) < 1e-10
    assert normwise(again.cpu().numpy(), oracle_hessian(waters, n_pa, 81)[0]) < 1e-10
