"""Registers of kernels whose waves per SIMD their comments count on (512
registers a SIMD lane, allocated by eights), from the built library's metadata
(no GPU; needs the ROCm llvm tools)."""
import os
import re
import subprocess

import pytest

from paper_2502_08470_amd import build as B

TOOLS = "/opt/rocm/llvm/bin"
pytestmark = pytest.mark.skipif(not os.path.exists(f"{TOOLS}/llvm-readelf"), reason="no llvm-readelf")


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("objects")
    (tmp / "libsigkernel.so").symlink_to(B.LIB)
    subprocess.run([f"{TOOLS}/llvm-objdump", "--offloading", "libsigkernel.so"], cwd=tmp, check=True,
                   capture_output=True)
    out = {}
    for obj in tmp.glob("*amdgcn*"):
        notes = subprocess.run([f"{TOOLS}/llvm-readelf", "--notes", str(obj)], check=True, capture_output=True,
                               text=True).stdout
        for kernel in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            out[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", kernel).group(1))
    return out


@pytest.mark.parametrize("kernel,waves,count", [
    ("k_sweep_pipeId", 2, 44),     # FP64: orders 2..12, both schemes, with and without checkpoints
    ("k_adjoint_pipeId", 2, 22),
    ("k_adjoint_w2", 2, 20),
])
def test_waves_per_simd(registers, kernel, waves, count):
    mine = {k: v for k, v in registers.items() if kernel in k}
    assert len(mine) >= count
    over = {k: v for k, v in mine.items() if (v + 7) // 8 * 8 > 512 // waves}
    assert not over
