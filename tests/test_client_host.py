"""CPU run of the client's encryption and decryption loops (tests/host/client.cpp): each instruction set that this
processor has, the sharing out over threads, and whole calls on several threads -- plain, under
AddressSanitizer and UndefinedBehaviorSanitizer, and under ThreadSanitizer."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_1806_03461_amd as T
import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("options", [["-O3"], ["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"],
                                     ["-O1", "-g", "-fsanitize=thread"]], ids=["plain", "address", "thread"])
def test_client_loops_on_the_host(tmp_path, options):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++") or not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime.h")):
        pytest.skip("no g++ or no HIP headers")
    exe = str(tmp_path / "client")
    b = subprocess.run(["g++", "-std=c++17", *options, "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include", "-pthread",
                        os.path.join(ROOT, "tests", "host", "client.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert b.returncode == 0, b.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and "client: ok" in r.stdout, r.stdout


def test_threaded_calls_match_the_oracle(real_keys):
    """3,333 samples: encryption and decryption both run on several threads; any phase is decrypted."""
    sk, _ = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
    rng = np.random.default_rng(3333)
    bits = rng.integers(0, 2, 3333).astype(np.uint8)
    ct = T.tfhe_encrypt(sk, 98, bits)
    assert np.array_equal(ct, real_keys.encrypt(bits, 98))
    assert np.array_equal(T.tfhe_decrypt(sk, ct), bits)
    ct[:, -1] += rng.integers(0, 1 << 32, 3333, dtype=np.uint64).astype(np.uint32)
    assert np.array_equal(T.tfhe_decrypt(sk, ct), real_keys.decrypt(ct))
