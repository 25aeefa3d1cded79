"""One work-group of the fp32 tile kernel per compute unit: its eight waves take more than 128 of a lane's 512 registers, so that
the four waves per SIMD of two work-groups do not fit."""
import os
import re
import subprocess

import pytest

from paper_2201_05596_amd import build as B

LLVM = "/opt/rocm/llvm/bin"


def test_one_tile_per_compute_unit(tmp_path):
    obj, fat, co = os.path.join(B.HERE, "_build", "gemm_f32.o"), str(tmp_path / "f.fat"), str(tmp_path / "f.co")
    if not os.path.exists(obj) or not os.path.exists(LLVM + "/llvm-readelf"):
        pytest.skip("needs the built object file and llvm-readelf")
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull], check=True, capture_output=True)
    subprocess.run([LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    "--input=" + fat, "--output=" + co], check=True, capture_output=True)
    notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", co], check=True, capture_output=True, text=True).stdout
    used = re.findall(r"\.name: +(\S+).*?\.vgpr_count: +(\d+)", notes, re.S)
    tiles = [int(n) for name, n in used if "f32_tile_kernel" in name]
    assert len(tiles) == 8 and min(tiles) > 128
