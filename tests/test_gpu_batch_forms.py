"""The persistent contraction's two forms (lists of at most five column blocks
per group, and any list) and, in FP64, the column quads of a batch item: batches
whose widest molecule has 1, 2, 5 and 6 blocks, its last block holding 9, 2, 8
and 1 columns (and 9 columns of a 16-column block in the narrower molecules
beside it), against the single-molecule path, bit for bit."""
import numpy as np
import pytest

from paper_2208_14639_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("waters", [(1, 1), (2, 1), (8, 3, 1), (9, 4, 2)])
def test_forms_match_the_single_path(waters, prec):
    import torch
    from paper_2208_14639_amd import vv10
    probs = [inputs.make_problem(k, 31 + 13 * m, 400 + 10 * k + m) for m, k in enumerate(waters)]
    with vv10.Batch(probs, prec=prec) as b:
        _, blocks = b.run()
        torch.cuda.synchronize()
        got = [h.cpu().numpy() for h in blocks]
    for p, h in zip(probs, got):
        with vv10.Plan(p, prec=prec) as pl:
            ref = pl.hessian_terms(p.rho_x, p.grad_rho_x)["hess"]
            torch.cuda.synchronize()
        assert np.array_equal(h, ref.cpu().numpy()), (p.n_atom, prec)
