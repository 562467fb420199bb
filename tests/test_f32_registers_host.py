"""The fp32 matrix-core kernels of narrow heads keep their sums and operands in registers: the scratch
memory of each, from the metadata of the built library.  (A few values that are written before a
loop and read after it cost nothing that can be measured.)"""
import glob
import os
import re
import subprocess

import pytest

from paper_2310_01655_amd import build as lib_build

READELF, OBJDUMP = "/opt/rocm/llvm/bin/llvm-readelf", "/opt/rocm/llvm/bin/llvm-objdump"
MOST = 32                                                # bytes a lane


@pytest.mark.skipif(not os.path.exists(READELF), reason="no reader of the metadata")
@pytest.mark.parametrize("kernel,variants", [("f32_bwd_kernel", 32), ("f32_rows_kernel", 34)])
def test_scratch_of_narrow_kernels(tmp_path, kernel, variants):
    if not os.path.exists(lib_build.LIB):
        lib_build.build()
    copy = tmp_path / "lib.so"
    copy.symlink_to(lib_build.LIB)
    subprocess.run([OBJDUMP, "--offloading", str(copy)], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    scratch = {}
    for path in glob.glob(str(tmp_path / "*gfx950")):
        notes = subprocess.run([READELF, "--notes", path], check=True, stdout=subprocess.PIPE, text=True).stdout
        for m in re.finditer(r"\.name: +(\S+)\n.*?\.private_segment_fixed_size: +(\d+)", notes, re.S):
            if re.search(r"\d%sILi4E" % kernel, m[1]):
                scratch[m[1]] = int(m[2])
    assert len(scratch) == variants
    assert max(scratch.values()) <= MOST, sorted(scratch.items(), key=lambda x: -x[1])[:8]
