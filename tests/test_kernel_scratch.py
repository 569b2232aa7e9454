"""Scratch memory of the GEMM kernels, as the built library states it."""
import os
import re
import subprocess

import pytest

from paper_2406_06858_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
SCRATCH_256 = 72                  # bytes a lane


@pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(READELF)), reason="no object tools")
def test_registers_do_not_spill(tmp_path):
    """None, but for the 256x256 tile, whose accumulators and fragments take all registers and which keeps a few values of a lane there
    across its main loop."""
    lib = tmp_path / "lib.so"
    lib.symlink_to(build.LIB)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    found = []
    for o in (p for p in tmp_path.iterdir() if "gfx950" in p.name):
        notes = subprocess.run([READELF, "--notes", str(o)], check=True, capture_output=True, text=True).stdout
        found += re.findall(r"\.name:\s+(_ZN4flux\d+gemm_kernel\S+)\s+\.private_segment_fixed_size:\s+(\d+)", notes)
    assert len(found) >= 10 * build.N_CFGS
    for name, scratch in found:
        assert int(scratch) <= (SCRATCH_256 if "TileCfgILi256ELi256E" in name else 0), name
