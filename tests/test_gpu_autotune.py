"""The autotuner times the calls that a program runs: without stage events (which
take small grids through two launches in place of one), and its record holds
tiles that a plan accepts."""
import pytest

from paper_2208_14639_amd import autotune, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "bf16x3"])
@pytest.mark.parametrize("waters,n_pa", [(2, 150), (7, 40)])
def test_tunes_untimed_calls(monkeypatch, waters, n_pa, prec):
    from paper_2208_14639_amd import vv10

    def no_stage_events(*a):
        raise AssertionError("the tuner timed stages")

    monkeypatch.setattr(vv10, "vv10_set_timing_stages", no_stage_events)
    monkeypatch.setattr(vv10, "vv10_set_timing", no_stage_events)
    p = inputs.make_problem(waters, n_pa, 91)
    rec = autotune.tune(p, prec, repeats=2, log=lambda *a: None)
    assert rec["call_ms"] > 0
    cache = {autotune.bucket_key(p.n_grid, p.n_atom, prec): rec}
    tiles = autotune.lookup(p.n_grid, p.n_atom, prec, cache)
    with vv10.Plan(p, prec=prec, tiles=tiles) as pl:
        assert vv10.vv10_get_tiles(pl.handle) == tiles
