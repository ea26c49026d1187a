"""What the compiler reports for the device kernels, with the build's own flags: no kernel needs scratch memory, and every
blind rotation exists with and without the recording of its rounding distance.  Scratch is memory that the runtime sets up for a
queue when the first kernel that needs it is dispatched, and tfhe_gate_batch_noalloc promises that no allocation of any
kind happens inside; a blind rotation without the recording form is one that tfhe_rounding_margin_enable cannot look at."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1806_03461_amd import build


def test_no_kernel_uses_scratch_memory():
    if not shutil.which("hipcc"):
        pytest.skip("no hipcc")
    r = subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage", "-o", os.devnull,
                        os.path.join(build.CSRC, "kernels.hip")], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout
    names = re.findall(r"Function Name: (\S+)", r.stdout)
    scratch = [int(v) for v in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stdout)]
    assert len(names) == len(scratch) and any("blind_rotate_wave_kernel" in n for n in names), r.stdout
    assert [(n, s) for n, s in zip(names, scratch) if s] == []
    # _ZN..blind_rotate_x_kernelILb<MARGIN>E..., the recording form first among its template arguments
    rotations = [re.search(r"(blind_rotate\w*?_kernel)(?:ILb([01])E(\w*?)EEv)?", n).groups() for n in names if "blind_rotate" in n]
    plain, recording = ({(name, rest) for name, margin, rest in rotations if margin == form} for form in "01")
    assert len(plain) == 5 and len(rotations) == 10 and plain == recording, rotations
