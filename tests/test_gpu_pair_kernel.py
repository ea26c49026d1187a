"""The blind rotation for two gates per CU (the next key row in registers) on what the parity tests check the others with:
rotation amounts on every boundary, keys with every factor at an end of its range, against the oracle's bytes."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_SCRIPT = r"""
import sys
import torch
sys.path[:0] = [sys.argv[1], sys.argv[1] + "/tests"]
import paper_1806_03461_amd as T, workloads
from oracle import oracle as orc
import test_gpu_parity as parity
sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
parity.test_rotation_amounts_at_every_boundary((T, sk, ck), orc.Keys(orc.default_params(), workloads.KEY_SEED))
print("boundaries ok", flush=True)
parity.LAUNCHES = [(1, 2 ** -10.5)]
for pattern in parity.EXTREMES:
    parity.test_extreme_key_limbs_stay_exact((T, sk, ck), orc, pattern)
    print(pattern, "ok", flush=True)
"""


def test_extreme_keys_and_rotations_on_the_kernel_of_two_gates_per_cu():
    env = {k: v for k, v in os.environ.items() if not k.startswith("TFHE_")}
    env.update(TFHE_LATENCY_BATCH="0", TFHE_PAIR_BATCH="1000000")
    r = subprocess.run([sys.executable, "-c", _SCRIPT, ROOT], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=200)
    assert r.returncode == 0, r.stdout
    assert r.stdout.count(" ok") == 6, r.stdout
