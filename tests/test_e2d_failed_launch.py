"""A refused kernel launch in lm_e2d_step leaves the handle at the last step whose
launches all went out (no GPU: the C ABI's host code on the stand-in runtime)."""

import os
import subprocess

import pytest

from host_asan import harness

pytestmark = pytest.mark.skipif(not harness.available(), reason="hipcc / clang++ not installed")


def test_steps_whose_launches_failed_do_not_count():
    harness.build()
    exe = os.path.join(harness.OUT, "fail_launch")
    subprocess.run([harness.CLANG, "-O1", "-g", "-std=c++17", *harness.SAN_LINK, "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I", harness.INCLUDE, os.path.join(harness.HERE, "fail_launch.cpp"),
                    os.path.join(harness.OUT, "liblagmean_asan.so"), "-ldl", "-Wl,-rpath," + harness.OUT,
                    "-o", exe], check=True)
    env = dict(os.environ)
    env.update(harness.ENV)
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env, timeout=120)
    assert p.returncode == 0, p.stdout[-2000:]
    rows = [tuple(int(x) for x in line.split()) for line in p.stdout.splitlines()]
    for profiled in (0, 1):
        got = [r for r in rows if r[0] == profiled]
        assert len(got) >= 12  # four launches a step at least
        assert all(st == -4 for _, _, st, _, _ in got)
        first = [r[3] for r in got]
        # no step counts before its launches, all but the last one before the call's end
        assert first[:5] == [0] * 5 and first == sorted(first) and max(first) == 2
        assert all(after == 2 for *_, after in got)
