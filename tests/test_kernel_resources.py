"""Register budgets of the built kernels, read from the code objects of the library (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2510_10467_amd as bcq
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


def test_two_workgroups_of_the_128_x_64_tiles_share_a_cu(kernels):
    """The level form's price of these tiles beyond 256 workgroups counts on two of them per CU: 160 KiB of LDS and, of eight waves each, 128
    vector registers (128 x 64, p = 4 with offsets, 400 workgroups: 1024 columns 20.8 us with two per CU, 24.9 with one)."""
    tiles = {name: use for name, use in kernels.items() if "level_mfma_kernel" in name and "5ShapeILi2ELi4E" in name}
    assert len(tiles) == 8                                      # one to four planes with and without offsets
    for name, (registers, scratch) in tiles.items():
        assert registers <= 128 and scratch == 0, f"{name}: {registers} vector registers, {scratch} bytes of scratch"
    for p in (1, 2, 3, 4):
        for offsets in (False, True):
            for group in (64, 128, 256):
                used = bcq.level_layout(p, 104, 4096, group, offsets)["lds_bytes"]
                assert 2 * used <= 160 * 1024, f"p={p} offsets={offsets} group={group}: {used} bytes of LDS"


def test_one_request_at_one_precision_has_one_kernel(kernels):
    """plane_mfma_kernel<P, 1, false, .., false, ..> is what plane_mfma_single_kernel replaced: nothing launches it."""
    assert not [name for name in kernels if re.search(r"plane_mfma_kernelILi\dELi1ELb0ELb[01]ELb0E", name)]
    assert len([name for name in kernels if "plane_mfma_single_kernel" in name]) == 4 * 2 * 3       # planes, offsets, group sizes
