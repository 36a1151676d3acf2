"""Run.step_profiled times the launches that Run.step makes: their sum is the step's
time, and below 512^2 (rows and columns in two launches a stage) no column pass is
timed that a step does not run."""

from __future__ import annotations

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,prec,kw", [(64, "fp64", {}), (128, "fp32", {}), (192, "fp64", {"momentum": True}),
                                       (256, "fp32", {}), (384, "fp32", {}), (128, "fp32", {"interp": "cubic"}),
                                       (64, "fp64", {"fields": ("u", "q")}), (512, "fp32", {})], ids=str)
def test_the_parts_are_those_of_a_step(N, prec, kw):
    from paper_2208_02682_amd import Run, make_config
    from synth.workloads import scaled_run
    say(f"profiled steps N={N} {prec} {kw}")
    w = scaled_run(N, Ro=0.1, ratio=1.0, periods=1.0, seeds=(50, 51), precision=prec)
    merged = N < 512 and not ({"interp", "fields"} & set(kw))
    with Run(make_config(N, precision=prec, dt=w.dt, nu8=w.nu8, **kw)) as run:
        run.set_state(*w.initial_state())
        run.begin_interval()
        run.step(20)
        step = min(run.step_timed(32) for _ in range(5)) / 32
        parts = min((run.step_profiled(32) for _ in range(5)), key=sum)
    say(f"  step {1e3 * step:.1f} us, parts {[round(4e3 * p, 2) for p in parts]}")
    assert all(p > 0 for p in parts)
    # a stage's closing columns are one launch a call, not four a step
    assert (parts[2] < 0.1 * parts[1]) == merged
    assert 4 * sum(parts) < 1.4 * step
