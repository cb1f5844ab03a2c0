"""The sweep kernels address their LDS from 0, which needs every byte of it to be dynamic: the
code objects in the built library state the static LDS of each kernel (CPU)."""
import os
import re
import subprocess

import pytest

import paper_2207_12848_amd.build as build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs " + READELF)
def test_sweep_kernels_have_no_static_lds(tmp_path):
    lib = open(build.OUT, "rb").read()
    found = {}
    for at in (m.start() for m in re.finditer(b"\x7fELF\x02\x01", lib)):
        if int.from_bytes(lib[at + 18:at + 20], "little") != 224:  # EM_AMDGPU
            continue
        obj = tmp_path / "object"
        obj.write_bytes(lib[at:])
        notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("  - .agpr_count")[1:]:
            size = int(re.search(r"\.group_segment_fixed_size: (\d+)", kernel).group(1))
            found[re.search(r"\.symbol: +'?(\S+?)\.kd", kernel).group(1)] = size
    sweeps = {k: v for k, v in found.items() if "k_sweepI" in k}
    assert len(sweeps) == 16 and set(sweeps.values()) == {0}
    assert any(v > 0 for v in found.values())  # (the numbers are there)
