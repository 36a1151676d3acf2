"""Which form a batched group's launches take (no GPU): merged while its row blocks
leave the chip idle, the passes apart beyond, on the sides that were measured faster
(csrc/step_kernels.hpp, batch_merged_runs).  A large batch in merged launches is
slower than in passes of their own at every size.  And which column tiles: half-width
ones only for groups of few runs (batch_tile)."""

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
    rows = "".join(f'std::printf("{N} {p} %d", lm::batch_merged_runs<{t}, {N}>());\n'
                   f'for (int m = 1; m <= 64; ++m) for (int w = -1; w <= 1; ++w) '
                   f'std::printf(" %d", lm::batch_tile<{t}, {N}>(m, w));\nstd::puts("");\n'
                   for N in SIZES for p, t in (("fp32", "float"), ("fp64", "double")))
    src.write_text('#include <cstdio>\n#include "step_kernels.hpp"\nint main() {\n' + rows + "}\n")
    exe = str(d / "rule")
    subprocess.run([harness.HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-I", harness.INCLUDE,
                    "-I", harness.CSRC, "-c", str(src), "-o", exe + ".o"], check=True)
    subprocess.run([harness.CLANG, exe + ".o", "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, check=True).stdout
    res = {}
    for line in out.splitlines():
        n, p, v, *tiles = line.split()
        res[int(n), p] = int(v), {(m, w): int(tiles[3 * (m - 1) + w + 1]) for m in range(1, 65) for w in (-1, 0, 1)}
    return res


@pytest.mark.parametrize("key", sorted(MEASURED), ids=str)
def test_each_side_takes_the_form_measured_faster(limits, key):
    merged, apart = MEASURED[key]
    limit = limits[key][0]
    assert limit >= merged
    assert apart is None or limit < apart
    assert limit < 64  # a large batch never merges


@pytest.mark.parametrize("N", [512, 1024])
def test_large_grids_never_merge(limits, N):
    assert limits[N, "fp32"][0] == limits[N, "fp64"][0] == 0


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("N", SIZES)
def test_half_width_tiles_are_for_few_runs(limits, N, prec):
    limit, tile = limits[N, prec]
    for (m, w), got in tile.items():
        wide = N < 512 and m >= 8 and m > limit and w < 0
        assert got == (0 if wide else w), (m, w)
    assert tile[1, -1] == -1
    assert tile[64, -1] == (0 if N < 512 else -1)
