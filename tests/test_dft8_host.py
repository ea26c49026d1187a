"""CPU run of the transforms of csrc/dft8.h (tests/host/dft8_exactness.cpp), in the form of either blind rotation, on
random operands and on the ends of their ranges: the rounded products equal exact 64-bit integer ones, and no
value is further from its integer than the bound derived for the transforms of fft512.h; and of whole steps
lane by lane, with each kernel's own exchanges and with the key where the upload stores it for that kernel."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_transforms_with_pending_cosines_are_exact_on_the_host(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++") or not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime.h")):
        pytest.skip("no g++ or no HIP headers")
    exe = str(tmp_path / "dft8_exactness")
    b = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                        os.path.join(ROOT, "tests", "host", "dft8_exactness.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert b.returncode == 0, b.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout
    m = re.search(r"wrong 0 largest distance fft512 (\S+) table (\S+) shifted (\S+)", r.stdout)
    assert m, r.stdout
    steps = re.search(r"whole steps: wrong 0 largest distance (\S+)", r.stdout)
    assert steps and float(steps.group(1)) < 2 ** -10.5, r.stdout
    # the worst case is bounded by about 2^-10.5 (10 u log2(512) times the operands' norms); a wrong rounding needs 0.5
    assert max(float(v) for v in m.groups()) < 2 ** -10.5, r.stdout
