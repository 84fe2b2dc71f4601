"""Lanes of a wave that hand rows to each other through LDS without a barrier order
their accesses for the compiler too: a wave barrier alone is no fence, and a store may
then move past another lane's read of it.  Looked for in the intermediate code of the
training kernels, before any optimisation."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2002_03644_amd import build as B


def test_every_wave_barrier_is_fenced(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = str(tmp_path / "nn.ll")
    subprocess.run([hipcc, *B.COMMON, *B.UNITS["hlbm_nn.hip"], "--cuda-device-only", "-S",
                    "-emit-llvm", "-Xclang", "-disable-llvm-passes", "-o", out,
                    os.path.join(B.CSRC, "hlbm_nn.hip")], check=True, capture_output=True)
    code = [line.strip() for line in open(out) if line.strip() and line.strip()[0] != ";"]
    at = [k for k, line in enumerate(code) if re.search(r"call void @llvm.amdgcn.wave.barrier", line)]
    assert at
    for k in at:
        assert code[k - 1].startswith('fence syncscope("wavefront") release'), code[k - 1:k + 2]
        assert code[k + 1].startswith('fence syncscope("wavefront") acquire'), code[k - 1:k + 2]
