"""No kernel of the library spills registers to scratch memory: the ones around
the step (fields, re-equilibration, statistics, filter, checkpoints) and the
corrector's.  Compiles the device code on the host (about a minute)."""
import os
import re
import shutil
import subprocess

import pytest

from test_kernel_resources import CSRC, HIPCC, ROOT


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="hipcc not available")
@pytest.mark.parametrize("source,least", [("lbm_kernels.hip", 70), ("lbm_nn.hip", 15)])
def test_no_kernel_uses_scratch(source, least, tmp_path):
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "--cuda-device-only",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(CSRC, source), "-o", str(tmp_path / "k.o")]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", out.stderr)
    scratch = [int(v) for v in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", out.stderr)]
    assert len(names) == len(scratch) >= least
    assert not [(n, s) for n, s in zip(names, scratch) if s]
