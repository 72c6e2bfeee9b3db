"""Strip-boundary records in LDS are written as words and read as words, pairs
of words, FP32 and FP64 values: the writes have to be ones that the compiler
orders against every read (no GPU; needs hipcc)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_08470_amd import build as B

pytestmark = pytest.mark.skipif(not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")),
                                reason="no hipcc")


def device_ir(tmp_path, body, *flags):
    src, out = tmp_path / "k.hip", tmp_path / "k.ll"
    src.write_text(f'#include "{B.CSRC}/sk_kernels.h"\n{body}\n')
    subprocess.run([B.hipcc(), *B.FLAGS, *flags, "-w", "--cuda-device-only", "-S", "-emit-llvm", str(src), "-o",
                    str(out)], check=True)
    return out.read_text()


def test_a_read_follows_the_write_before_it(tmp_path):
    """The FP64 coefficient is read before and after a record is written to a
    place that may be the same: two loads, not one kept."""
    ir = device_ir(tmp_path, """
__global__ void k(const double* q, int i, int j, double* out) {
    extern __shared__ __align__(16) unsigned char sk_smem[];
    const SkLds<unsigned> rec = (SkLds<unsigned>)sk_smem;
    const float c[5] = {0, 0, 1, 2, 3};
    const double a = *(SkLds<double>)(rec + 2 * i);
    sk_edge_write<float, 4>(rec + 2 * j, q[0], q[1], c, 7);
    out[0] = a;
    out[1] = *(SkLds<double>)(rec + 2 * i);
}""")
    assert len(re.findall(r"load double, ptr addrspace\(3\)", ir)) == 2


@pytest.mark.parametrize("kernel,plain", [
    ("k_sweep<float, 5, 0, true, 2, true>(const SweepArgs<float>)", False),
    ("k_sweep<double, 4, 20, false, 2, false>(const SweepArgs<double>)", False),
    ("k_sweep_pipe<float, 5, 0, true, 4>(const PipeArgs<float>)", False),
    ("k_adjoint_pipe<float, 5, 0, 4>(const AdjPipeArgs<float>)", False),
    # (its ring keeps the exponents in an array of their own, read as they are written)
    ("k_adjoint<float, 5, 0, 4, false>(const AdjArgs<float>)", True),
])
def test_words_are_written_as_aliasing_types(tmp_path, kernel, plain):
    ir = device_ir(tmp_path, f"template __global__ void {kernel};", "-Xclang", "-disable-llvm-passes")
    char = re.search(r'^(!\d+) = !\{!"omnipotent char"', ir, re.M).group(1)
    tags = set(re.findall(rf"^(!\d+) = !\{{{char}, {char}, i64 0\}}", ir, re.M))
    stores = re.findall(r"store i(?:32|64) [^\n]*ptr addrspace\(3\)[^\n]*!tbaa (!\d+)", ir)
    assert any(t in tags for t in stores)
    assert plain or all(t in tags for t in stores)
