"""The momentum rows at every grid size, precision and gather, alone and with other
averaged fields: six waves share the transforms and the gathered velocity, through
whole or split exchanges.  Two steps reach every stage, the t = tau limit included.

Bars: those of the whole-run tests, 1e-12 in float64 and 1e-5 on the mixed path."""

from __future__ import annotations

import pytest

from gpu_util import compare_value, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("N", [64, 128, 192, 256, 384, 512, 1024])
@pytest.mark.parametrize("fields,interp", [(("h", "zeta"), "bilinear"), (("u", "q"), "cubic")])
def test_two_steps_match_the_oracle(N, prec, tol, fields, interp):
    from oracle.lagmean import Params, Run as OracleRun
    from paper_2208_02682_amd import Run, make_config
    from synth.workloads import scaled_run
    say(f"momentum rows N={N} {prec} {fields} {interp}")
    w = scaled_run(N, Ro=0.1, ratio=1.0, periods=1.0, seeds=(74, 75), precision=prec)
    u, v, h = w.initial_state()
    o = OracleRun(Params(N=N, dt=w.dt, nu8=w.nu8, fields=fields, interp=interp, momentum=True), u, v, h)
    o.begin_interval()
    o.step(2)
    ref = o.end_interval()
    with Run(make_config(N, precision=prec, dt=w.dt, nu8=w.nu8, fields=fields, interp=interp, momentum=True)) as run:
        run.set_state(u, v, h)
        run.begin_interval()
        run.step(2)
        run.end_interval()
        got = {**run.field_outputs(), **run.momentum_outputs()}
    assert set(got) == set(ref) and {"S2_mom_x", "S2_mom_y"} <= set(ref)
    for k in ref:
        err = compare_value(k, got[k], ref[k])
        say(f"  {k}: {err:.1e}")
        assert err < tol, (k, err)
