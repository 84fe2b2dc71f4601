"""No sweep that a plan can reach keeps registers in scratch memory: a spill in the
row loop costs a trip through memory per row, and more than the wave it makes room
for gains.  The FP32 moments of a batch leave room for all eight waves of a SIMD.
Read from the metadata of the built library's kernels."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2002_03644_amd import _lib

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("needs llvm-readelf")
    lib = open(_lib.LIB_PATH, "rb").read()
    out = {}
    d = tmp_path_factory.mktemp("co")
    # the device code objects: ELF files in the fat binary, after the host's own
    for k, m in enumerate(re.finditer(rb"\x7fELF\x02\x01\x01\x40", lib)):
        f = str(d / f"{k}.co")
        with open(f, "wb") as h:
            h.write(lib[m.start():])
        notes = subprocess.run([READELF, "--notes", f], capture_output=True, text=True).stdout
        for entry in re.split(r"\n\s+- \.a", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry)
            count = {k: re.search(rf"\.{k}:\s+(\d+)", entry)
                     for k in ("vgpr_spill_count", "vgpr_count", "sgpr_count")}
            if name and all(count.values()):
                out[name.group(1)] = {k: int(v.group(1)) for k, v in count.items()}
    assert len(out) > 50, "kernel metadata not found"
    return out


# two-step widths that FP64 plans cannot take are built but never launched
@pytest.mark.parametrize("kernel", [r"f(32|64)6k_stepI", r"f(32|64)12k_step_batchI", r"f327k_step2I",
                                    r"f647k_step2ILi(64|128)E", r"f(32|64)13k_step_batch2I",
                                    r"f(32|64)10k_residentI", r"f6412k_tile_batchI"])
def test_sweeps_do_not_spill(registers, kernel):
    found = {n: c["vgpr_spill_count"] for n, c in registers.items() if re.search(kernel, n)}
    assert found
    assert not {n: c for n, c in found.items() if c}


def test_batch_moments_fill_the_simd(registers):
    found = [c for n, c in registers.items() if re.search(r"f3215k_batch_momentsE", n)]
    assert len(found) == 1
    assert found[0]["vgpr_count"] <= 64 and found[0]["sgpr_count"] <= 80
    assert found[0]["vgpr_spill_count"] == 0
