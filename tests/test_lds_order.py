"""Lanes that read from LDS what other lanes of their wavefront stored there: the hardware keeps the order of a
wavefront's LDS operations, the compiler only between fences, since store and load of one lane go to different
addresses.  Checked on the intermediate code of the kernels that do this, without a GPU."""
import os
import re
import subprocess

import pytest

from paper_2501_12956_amd import build


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not found")
@pytest.mark.parametrize("source,kernel,handovers", [
    ("cholesky.hip", "chol_panel_kernel", 2),      # sum of a leaf of the inverse, the leaf itself
    ("hessian.hip", "hessian_f16_kernel", 2),      # turned 32 x 32 piece: written, free again
    ("update_t.hip", "t_delta_kernel", 3),         # stage: written, free again; sums turned through it
])
def test_handovers_within_a_wavefront_are_ordered(tmp_path, source, kernel, handovers):
    out = tmp_path / "device.ll"
    res = subprocess.run([build._hipcc(), *[f if f != "-O3" else "-O1" for f in build.FLAGS], "--cuda-device-only", "-S",
                          "-emit-llvm", os.path.join(build.CSRC, source), "-o", str(out)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    bodies = re.findall(r"^define [^\n]*amdgpu_kernel[^\n]*@\w*%s\w*\(.*?^}" % kernel, out.read_text(), re.S | re.M)
    assert bodies
    for body in bodies:
        for order in ("release", "acquire"):
            assert len(re.findall(r'fence syncscope\("wavefront"\) %s' % order, body)) >= handovers
