"""vv10_prepare that reports a HIP error (one that earlier code left on the
thread) returns only after the stream has run what it enqueued: its page-locked
words and device blocks are free for the next plan then.  The next plan on the
same sizes is unaffected."""
import ctypes
import re

import pytest

from gpu_util import oracle_energy, problem, relerr

pytestmark = pytest.mark.gpu


def test_error_is_returned_after_the_stream_is_idle():
    import torch
    from paper_2208_14639_amd import vv10
    p = problem(2, 60, 31)
    stream = torch.cuda.Stream()
    with vv10.Plan(p, prec="fp64") as pl:
        args = (pl.coords, pl.weights, pl.atom_of, pl.rho, pl.grad_rho)
        torch.cuda.synchronize()
        maps = open("/proc/self/maps").read()
        hip = ctypes.CDLL(re.search(r"\S+/libamdhip64\.so\S*", maps).group(0))
        a = torch.ones((8192, 8192), device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for _ in range(20):           # tens of milliseconds ahead of the call
                b = a @ a
        assert hip.hipSetDevice(1 << 20) != 0          # no such device
        with pytest.raises(vv10.VV10Error) as err:
            vv10.vv10_prepare(p.b, p.C, p.n_grid, p.n_atom, *args, vv10.VV10_FP64, stream)
        assert err.value.status == vv10.VV10_E_HIP
        assert stream.query()
        del b
    with vv10.Plan(p, prec="fp64") as pl:
        e = pl.energy_potential()[0].item()
    assert relerr(e, oracle_energy(2, 60, 31)[0]) < 1e-10
