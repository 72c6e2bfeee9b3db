"""The launcher of the increment Gram's strip bands refuses more coordinates
than the kernel's registers hold, whatever its caller tested (no GPU: the
refusal comes before any device call; needs hipcc)."""
import os
import shutil
import subprocess

import pytest

from paper_2502_08470_amd import build as B

pytestmark = pytest.mark.skipif(not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")),
                                reason="no hipcc")

MAIN = """
#include <cstdio>
#include <cstdlib>
#include "%s/sk_launch.h"
int main(int, char** v) {
    GramArgs<float> a{};
    a.split = atoi(v[1]);
    a.dpad = atoi(v[2]);
    printf("%%d", (int)SkLaunch<float>::gram_band(a, 1, 256, 1, nullptr));
}
"""


def test_refused_before_the_launch(tmp_path):
    src, exe = tmp_path / "m.hip", tmp_path / "m"
    src.write_text(MAIN % B.CSRC)
    subprocess.run([B.hipcc(), *B.FLAGS, "-w", "-c", str(src), "-o", f"{exe}.o"], check=True)
    subprocess.run([B.hipcc(), f"--offload-arch={B.ARCH}", f"{exe}.o", B.LIB,
                    f"-Wl,-rpath,{os.path.dirname(B.LIB)}", "-o", str(exe)], check=True)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1")
    for split, dpad in ((1, 64), (0, 68), (1, 49)):
        r = subprocess.run([str(exe), str(split), str(dpad)], check=True, capture_output=True, text=True, env=env)
        assert int(r.stdout) == 1, (split, dpad)  # hipErrorInvalidValue
