"""How a stage's work is spread over launches does not show in the results: column
groups that ride with the next stage's rows are done when a call returns, whatever
the calls' lengths, in a single run and in a batch; and the two-dimensional flow's
kernels at every grid size.

Splits of the same steps are compared bit for bit; against the oracle the bar is
that of the whole-run tests, 1e-12 in float64."""

from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu
SIZES = [64, 128, 192, 256, 384, 512, 1024]


def _start(N, prec, seed=80, **kw):
    from paper_2208_02682_amd import Run, make_config
    from synth.workloads import scaled_run
    w = scaled_run(N, Ro=0.1, ratio=1.0, periods=1.0, seeds=(seed, seed + 1), precision=prec)
    run = Run(make_config(N, precision=prec, dt=w.dt, nu8=w.nu8, **kw))
    run.set_state(*w.initial_state())
    run.begin_interval()
    return run


def _finish(run):
    run.end_interval()
    out = run.field_outputs()
    run.close()
    return out


@pytest.mark.parametrize("kw", [{}, {"momentum": True}, {"interp": "cubic"}, {"fields": ("u", "q")}], ids=str)
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("N", SIZES)
def test_calls_of_any_length_give_the_same_bits(N, prec, kw):
    from paper_2208_02682_amd import Batch
    say(f"stage launches N={N} {prec} {kw}")
    whole = _start(N, prec, **kw)
    whole.step(3)
    ref = _finish(whole)
    parts = _start(N, prec, **kw)
    parts.step(1)
    parts.step(2)
    got = {"1 + 2 steps": _finish(parts)}
    profiled = _start(N, prec, **kw)
    profiled.step_profiled(3)
    got["a pass at a time"] = _finish(profiled)
    runs = [_start(N, prec, seed=s, **kw) for s in (90, 80)]
    with Batch() as b:
        for r, n in zip(runs, (2, 3)):
            b.add(r, n)
        while b.step(1):
            pass
        for r in runs:
            b.remove(r)
    got["batched"] = _finish(runs[1])
    runs[0].close()
    for how, g in got.items():
        assert set(g) == set(ref)
        for k in ref:
            assert np.array_equal(g[k], ref[k]), (how, k)


@pytest.mark.parametrize("interp", ["bilinear", "cubic"])
@pytest.mark.parametrize("N", SIZES)
def test_two_dimensional_flow_at_every_size(N, interp):
    from oracle.euler2d import Euler2D as Oracle
    from paper_2208_02682_amd import Euler2D
    from synth.euler import two_vortex_vorticity
    say(f"two-dimensional flow N={N} {interp}")
    dt = 0.32 / N
    z0 = two_vortex_vorticity(N)
    o = Oracle(N, dt, z0, interp=interp)
    o.begin_interval()
    o.step(3)
    ref = o.end_interval()
    got = []
    for calls in ((3,), (1, 2)):
        with Euler2D(N, dt, interp=interp) as e:
            e.set_vorticity(z0)
            e.begin_interval()
            for n in calls:
                e.step(n)
            e.end_interval()
            got.append(e.outputs())
            # a second interval starts from this one's end
            e.begin_interval()
            e.step(1)
            e.end_interval()
            assert np.all(np.isfinite(e.read("zeta")))
    for k, a in got[0].items():
        assert np.array_equal(a, got[1][k]), k
        err = np.linalg.norm(a - ref[k]) / np.linalg.norm(ref[k])
        assert err < 1e-12, (k, err)
