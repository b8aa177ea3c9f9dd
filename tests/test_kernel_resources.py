"""Register budgets of the built kernels, read from the code objects of the library (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2510_10467_amd import build as hip_build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: (vector registers of both kinds, bytes of scratch per lane)}"""
    if hip_build.is_stale():
        hip_build.build()
    where = tmp_path_factory.mktemp("code_objects")
    lib = shutil.copy(hip_build.LIB, where / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True, capture_output=True)
    found = {}
    for name in sorted(os.listdir(where)):
        if "gfx950" not in name:
            continue
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(where / name)], check=True, capture_output=True,
                               text=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            field = {key: value for key, value in re.findall(r"\.(name|vgpr_count|private_segment_fixed_size):\s+(\S+)", entry)}
            found[field["name"]] = (int(field["vgpr_count"]), int(field["private_segment_fixed_size"]))
    return found


def test_two_waves_of_every_quantiser_share_a_simd(kernels):
    """A SIMD has 512 vector registers a lane: above 256 a kernel runs one wave on it and nothing covers its latencies (groups of 128
    with offsets, one to four planes: 119 us with 258 registers, 90 us with 226)."""
    quantisers = {name: use for name, use in kernels.items() if "quantize_kernel" in name}
    # four group sizes; base precisions 1 to 3 with and without offsets in both residual forms, base precision 4 in one
    assert len(quantisers) == 4 * (3 * 4 + 2)
    for name, (registers, scratch) in quantisers.items():
        assert registers <= 256, f"{name}: {registers} vector registers"
        assert scratch == 0, f"{name}: {scratch} bytes of scratch"
