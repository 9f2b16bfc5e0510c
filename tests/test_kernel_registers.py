"""Vector registers of the camera kernels that read F32 coefficients, from the
metadata of the built library.  A SIMD has 512 a lane, handed out in eights: 96
leave room for five waves, 104 for four.  These kernels took 94 (97 for the
layouts of 5 SH terms and fewer density terms) and, after two fields were put
in the middle of their argument block, 121 to 140."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from tests.test_device_code import LIB, LLVM, _code_objects


@pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(f"{LLVM}/llvm-readelf")),
                    reason="needs the built library and the ROCm LLVM tools")
def test_coefficient_kernels_keep_their_waves(tmp_path):
    found = {}
    for k, co in enumerate(_code_objects(tmp_path)):
        path = tmp_path / f"regs{k}.elf"
        path.write_bytes(co)
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(path)], check=True, capture_output=True,
                               text=True).stdout
        for block in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", block).group(1)
            found[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1))
    # mode 0 (F32 coefficients), one lane per ray, plain and skip walks of every layout
    kernels = {n: v for n, v in found.items()
               if re.match(r"_ZN3fpo3dev17render_cam_kernelILi0ELb[01]ELi\d+ELi\d+ELb0ELi1ELi1E", n)}
    assert len(kernels) >= 7, sorted(found)[:20]
    assert all(v <= 100 for v in kernels.values()), kernels
