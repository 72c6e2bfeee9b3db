"""The built kernels against a fault of the compiler's register allocator (seen
with the clang of ROCm 7.2): where it parks live registers (AGPR copies,
scratch stores) at the top of a block that ends a divergent region, it may put
them before the instruction that gives the other lanes back.  Those lanes'
values are lost, and the code after the region reads whatever the AGPRs or the
scratch memory held.  Kernels near their register limit are the ones at risk:
two builds with such a block gave FP64 gradients of order 10 and 12 that were
wrong, now and then, by hundreds of orders of magnitude.

A region's skip branch (s_cbranch_execz) leads to the block that restores
EXEC, so a vector write between that label and the restore is the fault.
(Regions so short that they have no skip branch are not looked at.)  No GPU;
needs the ROCm llvm-objdump."""
import os
import subprocess

import pytest

from paper_2502_08470_amd import build as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VECTOR = ("v_", "scratch_", "ds_", "global_", "flat_")
SCALAR_RESULT = ("v_readlane", "v_writelane", "v_readfirstlane", "v_cmp")


def early_writes(lines):
    """(kernel, label, instruction) of vector writes between the target of a
    region's skip branch and the EXEC restore that follows it."""
    found, kernel, body = [], None, []

    def scan():
        joins = {s.split()[1] for s in body if s.startswith("s_cbranch_execz L")}
        label, before = None, []
        for s in body:
            if s[0] == "<":
                label, before = (s[1:-2] if s[1:-2] in joins else None), []
            elif label is None:
                continue
            elif s.startswith("s_or_b64 exec, exec,"):
                found.extend((kernel, label, w) for w in before)
                label = None
            elif s.startswith(("s_branch", "s_cbranch", "s_endpgm")) or "saveexec" in s:
                label = None
            elif s.startswith(VECTOR) and not s.startswith(SCALAR_RESULT):
                before.append(s)

    for line in lines:
        s = line.split("//", 1)[0].strip()
        if s.startswith("<_Z"):
            scan()
            kernel, body = s[1:-2], []
        elif s:
            body.append(s)
    scan()
    return found


FAULT = """
<_Z1kv>:
s_and_saveexec_b64 s[12:13], s[60:61]
s_cbranch_execz L72
v_ldexp_f64 v[214:215], v[214:215], v2
<L72>:
v_readlane_b32 s1, v253, 19
v_accvgpr_write_b32 a28, v130
s_or_b64 exec, exec, s[12:13]
v_accvgpr_read_b32 v0, a28
"""


def test_the_fault_is_found_and_its_repair_is_not():
    assert early_writes(FAULT.splitlines()) == [("_Z1kv", "L72", "v_accvgpr_write_b32 a28, v130")]
    lines = FAULT.strip().splitlines()
    lines[6], lines[7] = lines[7], lines[6]
    assert early_writes(lines) == []


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_built_kernel_writes_before_the_restore(tmp_path):
    so = tmp_path / "libsigkernel.so"
    so.symlink_to(B.LIB)
    subprocess.run([OBJDUMP, "--offloading", so.name], cwd=tmp_path, check=True, capture_output=True)
    kernels, joins = 0, 0
    for obj in sorted(tmp_path.glob("*amdgcn*")):
        p = subprocess.Popen([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn", "--no-leading-addr",
                              str(obj)], stdout=subprocess.PIPE, text=True)
        lines = list(p.stdout)
        assert p.wait() == 0
        kernels += sum(line.startswith("<_Z") for line in lines)
        joins += sum("s_cbranch_execz L" in line for line in lines)
        assert early_writes(lines) == []
    assert kernels > 500 and joins > 10000
