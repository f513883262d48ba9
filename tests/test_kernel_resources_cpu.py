"""Registers of the projection kernel, from the compiler's report: what serves rare primitives (rectangles of hundreds of
tiles) must not cost the wavefronts per SIMD that hide the memory latency of all others."""
import os
import re
import subprocess

import pytest

from paper_2503_21364_amd import build as hip_build


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    cmd = [hip_build.hipcc(), *hip_build.COMMON, *hip_build.UNITS["preprocess.hip"], "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(hip_build.CSRC, "preprocess.hip"), "-o", str(tmp_path_factory.mktemp("obj") / "preprocess.o")]
    text = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    kernels = {}
    for part in text.split("Function Name: ")[1:]:
        m = re.match(r"_ZN3lmk17preprocess_kernelILj(\d)E", part)
        if m:
            kernels[int(m.group(1))] = {k: int(v) for k, v in re.findall(r" ([A-Z][A-Za-z]+(?: Spill| \[[^\]]*\])?): (\d+)", part)}
    return kernels


# (512 registers per SIMD lane, in granules of eight; degrees 2 and 3 hold 28 and 48 of SH coefficients in flight)
@pytest.mark.parametrize("degree,vgprs", [(0, 72), (1, 80), (2, 128), (3, 128)])
def test_projection_keeps_its_wavefronts(report, degree, vgprs):
    r = report[degree]
    assert r["VGPRs"] <= vgprs and r["VGPRs Spill"] == 0 and r["ScratchSize [bytes/lane]"] == 0, r
