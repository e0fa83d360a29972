"""What the compiler gave the kernels of libld.so whose launches count on a place on every CU, from
the metadata of the code object in the built library."""
import os
import re
import subprocess

import pytest

from paper_1807_02752_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name: {field: number}} over the gfx950 code objects of the library."""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf here")
    if not os.path.exists(build.LIB):
        build.build()
    data = open(build.LIB, "rb").read()
    found = {}
    for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", data):          # OS ABI 64: an AMD GPU code object
        path = str(tmp_path_factory.mktemp("co") / "k.co")
        open(path, "wb").write(data[m.start():])
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True).stdout
        for block in re.split(r"\n  - (?=\.\w)", notes):
            name = re.search(r"\.name: +(\S+)", block)
            if name:
                found[name.group(1)] = {k: int(v) for k, v in re.findall(r"\.(\w+): +(\d+)\n", block)}
    assert found
    return found


def test_four_frames_of_the_row_dp_fit_a_cu(kernels):
    # four frames of five waves a CU, however their waves fall on its SIMDs: seven waves a SIMD (512
    # VGPRs in eights), and no scratch memory in the row recursion
    (name,) = [k for k in kernels if "k_vpx_fit" in k]
    f = kernels[name]
    assert f["vgpr_count"] <= 72 and f["sgpr_count"] <= 96, f
    assert f["vgpr_spill_count"] == 0 and f["private_segment_fixed_size"] == 0, f
