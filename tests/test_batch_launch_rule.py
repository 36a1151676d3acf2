"""Which form a batched group's launches take (no GPU): merged while its row blocks
leave the chip idle, the passes apart beyond, on the sides that were measured faster
(csrc/step_kernels.hpp, batch_merged_runs).  A large batch in merged launches is
slower than in passes of their own at every size."""

import subprocess

import pytest

from host_asan import harness

pytestmark = pytest.mark.skipif(not harness.available(), reason="hipcc not installed")
SIZES = [64, 128, 192, 256, 384, 512, 1024]
# (N, precision): runs measured faster merged, runs measured faster apart
MEASURED = {(64, "fp32"): (28, 48), (64, "fp64"): (12, 28), (128, "fp32"): (10, 16), (128, "fp64"): (5, 7),
            (192, "fp32"): (7, 13), (192, "fp64"): (7, 18), (256, "fp32"): (2, 5), (256, "fp64"): (1, 2),
            (384, "fp32"): (7, 16), (384, "fp64"): (7, None)}


@pytest.fixture(scope="module")
def limits(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src = d / "rule.hip"
    rows = "".join(f'std::printf("{N} {p} %d\\n", lm::batch_merged_runs<{t}, {N}>());\n'
                   for N in SIZES for p, t in (("fp32", "float"), ("fp64", "double")))
    src.write_text('#include <cstdio>\n#include "step_kernels.hpp"\nint main() {\n' + rows + "}\n")
    exe = str(d / "rule")
    subprocess.run([harness.HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-I", harness.INCLUDE,
                    "-I", harness.CSRC, "-c", str(src), "-o", exe + ".o"], check=True)
    subprocess.run([harness.CLANG, exe + ".o", "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, check=True).stdout
    return {(int(n), p): int(v) for n, p, v in (line.split() for line in out.splitlines())}


@pytest.mark.parametrize("key", sorted(MEASURED), ids=str)
def test_each_side_takes_the_form_measured_faster(limits, key):
    merged, apart = MEASURED[key]
    assert limits[key] >= merged
    assert apart is None or limits[key] < apart
    assert limits[key] < 64  # a large batch never merges


@pytest.mark.parametrize("N", [512, 1024])
def test_large_grids_never_merge(limits, N):
    assert limits[N, "fp32"] == limits[N, "fp64"] == 0
