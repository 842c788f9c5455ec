"""The kernels that the benchmark names for a step's stages are instances of kernel templates in
the sources, with as many arguments as those have parameters."""

import glob
import os
import re

import pytest

import bench

CSRC = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "paper_1611_01545_amd", "csrc")


def _templates():
    found = {}
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"(?:template <([^>]*)>\s*(?://[^\n]*\s*)*)?(?:static )?__global__[^;{]*?void\s+(k_\w+)\s*\(",
                             text):
            found[m[2]] = len(m[1].split(",")) if m[1] else 0
    return found


@pytest.mark.parametrize("n", [64, 256, 1024, 2048])
def test_named_kernels_exist(n):
    templates = _templates()
    assert len(templates) > 20
    for stage in ("deposit", "fft_x_r2c", "fft_y_fwd", "fft_z", "fft_y_inv", "fft_x_c2r",
                  "force_grad", "interp_kick_drift"):
        name = bench.step_stage_kernel(stage, n)
        base, args = re.fullmatch(r"(k_\w+)<(.*)>", name).groups()
        assert templates.get(base) == len(args.split(",")), (stage, name)
    assert bench.step_stage_kernel("resort", n) is None
