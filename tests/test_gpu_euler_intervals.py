"""The two-dimensional flow over several intervals on one handle: the column-pass
outputs kept between calls and the two sets of state fields are those of the present
state, whatever came before.

Against the oracle 1e-12, as for a first interval; handles compared bit for bit."""

from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu
SIZES = [64, 128, 192, 256, 384, 512, 1024]


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("between", [0, 1], ids=["directly", "after a step outside"])
@pytest.mark.parametrize("N", SIZES)
def test_second_interval_matches_the_oracle(N, between):
    from oracle.euler2d import Euler2D as Oracle
    from paper_2208_02682_amd import Euler2D
    from synth.euler import two_vortex_vorticity
    say(f"second interval N={N} steps between {between}")
    dt, z0 = 0.32 / N, two_vortex_vorticity(N)
    o = Oracle(N, dt, z0)
    with Euler2D(N, dt) as e:
        e.set_vorticity(z0)
        for x in (o, e):
            x.begin_interval()
            x.step(3)
            x.end_interval()
            if between:
                x.step(between)
            x.begin_interval()
            x.step(2)
        ref = o.end_interval()
        e.end_interval()
        got = e.outputs()
    assert set(got) == set(ref)
    for k in ref:
        err = _rel(got[k], ref[k])
        assert err < 1e-12, (k, err)


@pytest.mark.parametrize("interp", ["bilinear", "cubic"])
@pytest.mark.parametrize("N", SIZES)
def test_a_used_handle_gives_the_bits_of_a_fresh_one(N, interp):
    from paper_2208_02682_amd import Euler2D
    from synth.euler import two_vortex_vorticity
    say(f"used handle N={N} {interp}")
    dt, z0 = 0.32 / N, two_vortex_vorticity(N)

    def interval(e):
        e.set_vorticity(z0)
        e.begin_interval()
        e.step(2)
        e.end_interval()
        return e.outputs()

    with Euler2D(N, dt, interp=interp) as e:
        fresh = interval(e)
        # an odd number of steps before each: the other set of fields is the present one
        e.step(1)
        again = [interval(e)]
        e.set_vorticity(-z0)
        e.begin_interval()
        e.step(3)
        again.append(interval(e))
    for g in again:
        for k in fresh:
            assert np.array_equal(g[k], fresh[k]), k
