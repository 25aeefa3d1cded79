"""What the fp32 kernels' launch rules take from their registers (a lane has 512 for the waves of its SIMD): one work-group of eight waves per
compute unit where a second would leave another unit without one, and no values kept in memory."""
import os
import re
import subprocess

import pytest

from paper_2201_05596_amd import build as B

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(name, template arguments): (registers, bytes of scratch memory)} of the built object file."""
    obj, tmp = os.path.join(B.HERE, "_build", "gemm_f32.o"), tmp_path_factory.mktemp("f32")
    fat, co = str(tmp / "f.fat"), str(tmp / "f.co")
    if not os.path.exists(obj) or not os.path.exists(LLVM + "/llvm-readelf"):
        pytest.skip("needs the built object file and llvm-readelf")
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull], check=True, capture_output=True)
    subprocess.run([LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    "--input=" + fat, "--output=" + co], check=True, capture_output=True)
    notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", co], check=True, capture_output=True, text=True).stdout
    found = {}
    for name, args, scratch, registers in re.findall(
            r"\.name: +\S*?\d+(f32_[a-z_]+_kernel)I((?:Li\d+E)+)E\S*.*?\.private_segment_fixed_size: +(\d+).*?\.vgpr_count: +(\d+)", notes, re.S):
        found[name, tuple(map(int, re.findall(r"\d+", args)))] = (int(registers), int(scratch))
    return found


def test_one_tile_per_compute_unit(kernels):
    tiles = [r for (name, _), (r, _) in kernels.items() if name == "f32_tile_kernel"]
    assert len(tiles) == 8 and min(tiles) > 128


@pytest.mark.parametrize("name,waves,sets", [("f32_split_kernel", 8, 2), ("f32_rows_split_kernel", 8, 8), ("f32_split_kernel", 4, 1), ("f32_rows_split_kernel", 4, 4)])
def test_split_kernels(kernels, name, waves, sets):
    used = [r for (n, args), (r, _) in kernels.items() if n == name and args[0] == sets]
    assert len(used) == 4 and max(used) <= 256               # two waves per SIMD: one work-group of eight, two of four
    assert waves == 4 or min(used) > 128                     # ... and not two of eight


def test_no_scratch_memory(kernels):
    assert len(kernels) == 8 + 4 * 2 + 4 * 2 + 4 * 2 + 3 * 2
    assert [k for k, (_, scratch) in kernels.items() if scratch] == []
