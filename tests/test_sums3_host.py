"""CPU run of the three sums from which the wave blind rotation recovers an external product (csrc/sums3.h): equal to
integer arithmetic mod 2^32, and no value further from where it is rounded to than the derived bounds."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_three_sums_give_the_product_on_the_host(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++") or not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime.h")):
        pytest.skip("no g++ or no HIP headers")
    exe = str(tmp_path / "sums3")
    b = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                        os.path.join(ROOT, "tests", "host", "sums3.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert b.returncode == 0, b.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout
    # 10 u log2(512) times the operands' norms, with factors of 22 bits (low) and 21 bits (top); a wrong rounding needs 0.5
    seen = re.findall(r"wrong 0 distance low (\S+) top (\S+) (\S+)", r.stdout)
    random = re.findall(r"random +wrong 0 distance low (\S+) top (\S+) (\S+)", r.stdout)
    assert len(seen) == r.stdout.count("distance") >= 30, r.stdout
    assert max(float(v[0]) for v in seen) < 2 ** -4.5, r.stdout
    assert max(float(x) for v in seen for x in v[1:]) < 2 ** -5.5, r.stdout
    # the largest that csrc/sums3.h quotes, from random operands and from all of them
    for runs, low, top in ((random, 3.5e-5, 1.8e-5), (seen, 3.5e-3, 1.8e-3)):
        assert max(float(v[0]) for v in runs) <= low, r.stdout
        assert max(float(x) for v in runs for x in v[1:]) <= top, r.stdout
