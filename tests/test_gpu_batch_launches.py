"""A batched group's launches are merged up to a number of runs and apart beyond: on
both sides of that line every member gives the bits it gives alone."""

from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _start(w, u, v, h, N, prec, kw):
    from paper_2208_02682_amd import Run, make_config
    run = Run(make_config(N, precision=prec, dt=w.dt, nu8=w.nu8, **kw))
    run.set_state(u, v, h)
    run.begin_interval()
    return run


def _finish(run):
    run.end_interval()
    out = run.field_outputs()
    run.close()
    return out


@pytest.mark.parametrize("N,prec,counts", [(64, "fp32", (40, 41)), (64, "fp64", (20, 21)), (128, "fp32", (10, 11)),
                                           (128, "fp64", (5, 6)), (192, "fp32", (8, 9)), (192, "fp64", (14, 15)),
                                           (256, "fp32", (2, 3)), (256, "fp64", (1, 2)), (384, "fp32", (8, 9)),
                                           (384, "fp64", (14, 15))])
@pytest.mark.parametrize("kw", [{}, {"momentum": True}, {"interp": "cubic", "fields": ("u", "q")}], ids=str)
def test_members_give_the_bits_of_a_run_alone(N, prec, counts, kw):
    from paper_2208_02682_amd import Batch
    from synth.workloads import scaled_run
    w = scaled_run(N, Ro=0.1, ratio=1.0, periods=1.0, seeds=(60, 61), precision=prec)
    u, v, h = w.initial_state()
    other = scaled_run(N, Ro=0.1, ratio=1.0, periods=1.0, seeds=(62, 63), precision=prec).initial_state()
    alone = _start(w, u, v, h, N, prec, kw)
    alone.step(2)
    ref = _finish(alone)
    for m in counts:
        say(f"batch launches N={N} {prec} {kw} x{m}")
        mine = {0, m // 2, m - 1}
        runs = [_start(w, *((u, v, h) if i in mine else other), N, prec, kw) for i in range(m)]
        with Batch() as b:
            for r in runs:
                b.add(r, 2)
            b.step(1)
            b.step_static(1)
            for r in runs:
                b.remove(r)
        for i, r in enumerate(runs):
            if i in mine:
                got = _finish(r)
                for k in ref:
                    assert np.array_equal(got[k], ref[k]), (m, i, k)
            else:
                r.close()
