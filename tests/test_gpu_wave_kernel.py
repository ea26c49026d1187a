"""GPU parity of the blind rotation that keeps one gate per wavefront (large batches), against the four-wave
kernels -- which the parity tests compare with the oracle -- and against the oracle itself.

All arithmetic is exact modulo 2^32, so the bar is equal bytes.  The sizes are where the kernel and the
rule that selects it can go wrong: fewer gates than waves of a workgroup, a ragged last workgroup, a round
of eight gates per CU, one item to either side of it (the remainder goes to another kernel), and
multiplexer pairs split between the two launches.
"""
import os
import subprocess
import sys

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_SCRIPT = r"""
import hashlib, sys
import numpy as np, torch
sys.path.insert(0, sys.argv[1])
import paper_1806_03461_amd as T, workloads
sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
rng = np.random.default_rng(61)
h = hashlib.sha256()
# arbitrary words reach every rotation amount, encryptions do not hit rounding ties
for count in (1, 3, 4, 5, 66):
    a, b = (torch.from_numpy(rng.integers(0, 1 << 32, (count, 501), dtype=np.uint64).astype(np.uint32).view(np.int32)).cuda() for _ in range(2))
    a[0] = torch.from_numpy(((np.arange(501) * 64 + 1) % 2048 << 21).astype(np.uint32).view(np.int32))
    for op in ("NAND", "XOR"):
        out = torch.empty_like(a)
        T.tfhe_gate_batch(ck, op, a, b, out, count)
        torch.cuda.synchronize()
        h.update(T.to_host(out).tobytes())
s, a, b = (T.to_device(T.tfhe_encrypt(sk, 300 + k, rng.integers(0, 2, 7).astype(np.uint8))) for k in range(3))
out = torch.empty_like(a)
T.tfhe_mux_batch(ck, s, a, b, out, 7)
W = rng.choice(np.array([-1, 0, 1], np.int8), (9, 13), p=[0.45, 0.1, 0.45])
res = torch.empty((9, 501), dtype=torch.int32, device="cuda")
x = T.to_device(T.tfhe_encrypt(sk, 310, rng.integers(0, 2, 13).astype(np.uint8)))
T.bnn_dense_encrypted_opts(ck, x, 13, W, np.arange(2, 11).astype(np.int32), 9, res, 0, T.LOWER_MUX_COMPARATOR)
torch.cuda.synchronize()
h.update(T.to_host(out).tobytes() + T.to_host(res).tobytes())
P = T.Params(300, 1024, 1, 2, 8, 5, 3, -15, -25)          # another gadget base and step count
sk2, ck2 = T.tfhe_keygen(P, 777)
a, b = (T.to_device(T.tfhe_encrypt(sk2, 320 + k, rng.integers(0, 2, 6).astype(np.uint8))) for k in range(2))
out = torch.empty_like(a)
T.tfhe_gate_batch(ck2, "AND", a, b, out, 6)
torch.cuda.synchronize()
h.update(T.to_host(out).tobytes())
print("digest", h.hexdigest())
"""


def test_small_batches_equal_the_four_wave_kernels():
    """Every batch on the wave kernel, and none: the same bytes."""
    digests = []
    for gates_from in ("1", "1000000000"):
        env = {k: v for k, v in os.environ.items() if not k.startswith("TFHE_")}
        env["TFHE_WAVE_GATES_FROM"] = gates_from
        r = subprocess.run([sys.executable, "-c", _SCRIPT, ROOT], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                           text=True, timeout=200)
        assert r.returncode == 0, r.stdout
        digests.append([l for l in r.stdout.splitlines() if l.startswith("digest")][-1])
    assert digests[0] == digests[1]


_BOTH_FORMS = r"""
import hashlib, sys
import numpy as np, torch
sys.path.insert(0, sys.argv[1])
import paper_1806_03461_amd as T
cus = torch.cuda.get_device_properties(0).multi_processor_count
# rotation amounts are read 64 steps at a time: one step, and one to either side of a whole reading
for n, bgbit, t, basebit in ((1, 10, 8, 2), (63, 10, 8, 2), (64, 10, 8, 2), (65, 10, 8, 2), (300, 8, 5, 3), (500, 10, 8, 2)):
    sk, ck = T.tfhe_keygen(T.Params(n, 1024, 1, 2, bgbit, t, basebit, -15, -25), 900 + n)
    # one workgroup per CU, two on every CU with some of their waves, whole ones
    for count in (5, 4 * cus + 6, 6 * cus + 5):
        amounts = (64 * np.arange(n + 1)[None, :] + np.arange(count)[:, None]) % 2048           # every one of 0 .. 2047, where there are as many
        a = torch.from_numpy((amounts << 21).astype(np.uint32).view(np.int32)).cuda()
        b, out = torch.zeros_like(a), torch.empty_like(a)
        T.tfhe_gate_batch(ck, "NAND", a, b, out, count)
        torch.cuda.synchronize()
        print("digest", n, bgbit, count, hashlib.sha256(T.to_host(out).tobytes()).hexdigest(), flush=True)
"""


def test_step_counts_and_rotations_on_both_forms_equal_the_four_wave_kernels():
    """The forms for one and for two workgroups per CU are different code: either with every rotation amount, with step counts
    around the 64 amounts that are read at a time, and with another gadget base."""
    found = []
    for gates_from in ("1", "1000000000"):
        env = {k: v for k, v in os.environ.items() if not k.startswith("TFHE_")}
        env["TFHE_WAVE_GATES_FROM"] = gates_from
        r = subprocess.run([sys.executable, "-c", _BOTH_FORMS, ROOT], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                           text=True, timeout=200)
        assert r.returncode == 0, r.stdout
        found.append([l for l in r.stdout.splitlines() if l.startswith("digest")])
    assert len(found[0]) == 18 and len({l.split()[-1] for l in found[0]}) == 18 and found[0] == found[1], found


def test_two_keys_on_two_streams():
    """900 gates for each of two keys at a time, on two streams: the lone form's workgroups share the CUs.  The same bytes as
    one key after the other, three times."""
    import torch
    import paper_1806_03461_amd as T
    rng = np.random.default_rng(90)
    keys = [T.tfhe_keygen(T.default_params(), seed)[1] for seed in (workloads.KEY_SEED, 5)]
    a, b = (torch.from_numpy(rng.integers(0, 1 << 32, (900, 501), dtype=np.uint64).astype(np.uint32).view(np.int32)).cuda() for _ in range(2))
    want, got = ([torch.empty_like(a) for _ in keys] for _ in range(2))
    streams = [torch.cuda.Stream() for _ in keys]
    for ck, out in zip(keys, want):
        T.tfhe_gate_batch(ck, "XOR", a, b, out, 900)
        torch.cuda.synchronize()
    assert not torch.equal(*want)
    for _ in range(3):
        for out in got:
            out.zero_()
        torch.cuda.synchronize()
        for ck, stream, out in zip(keys, streams, got):
            T.tfhe_gate_batch(ck, "XOR", a, b, out, 900, stream=stream.cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


_EXTREMES = r"""
import sys
import torch
sys.path[:0] = [sys.argv[1], sys.argv[1] + "/tests"]
import paper_1806_03461_amd as T, workloads
from oracle import oracle as orc
import test_gpu_parity as parity
read = T.tfhe_rounding_margin_read
def margin(ck):
    worst = read(ck)
    print("largest distance read", worst, flush=True)
    return worst
T.tfhe_rounding_margin_read = margin
sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
parity.test_rotation_amounts_at_every_boundary((T, sk, ck), orc.Keys(orc.default_params(), workloads.KEY_SEED))
print("boundaries ok", flush=True)
parity.LAUNCHES = [(1, float(sys.argv[2]))]
for pattern in parity.EXTREMES:
    parity.test_extreme_key_limbs_stay_exact((T, sk, ck), orc, pattern)
    print(pattern, "ok", flush=True)
"""


@pytest.mark.parametrize("kernel,knobs,bound", [("wave", {"TFHE_WAVE_GATES_FROM": "1"}, 2 ** -4.5), ("four waves", {"TFHE_LATENCY_BATCH": "0"}, 2 ** -10.5)],
                         ids=["wave", "four_waves"])
def test_extreme_keys_and_rotations_on_the_kernels_of_larger_batches(kernel, knobs, bound, say):
    """The parity test with rotation amounts on every boundary is too small to leave the latency kernel by itself: the
    same check, and extreme keys on a few gates, with every launch on the others."""
    env = {k: v for k, v in os.environ.items() if not k.startswith("TFHE_")}
    r = subprocess.run([sys.executable, "-c", _EXTREMES, ROOT, repr(bound)], env={**env, **knobs}, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=200)
    assert r.returncode == 0, r.stdout
    assert r.stdout.count(" ok") == 6 and r.stdout.count("largest distance read") == 5, r.stdout
    say(kernel + ": " + "; ".join(l for l in r.stdout.splitlines() if "distance read" in l or l.endswith("ok")))


@pytest.mark.parametrize("count", [769, 1024, 1025, 1281, 2047, 2048, 2049, 2900])
def test_batches_around_a_round(real_keys, count):
    """Default dispatch on a CU's worth of rounds: the first and last gates and a few between equal the oracle's,
    and all of them equal the same gates evaluated in small batches."""
    import torch
    import paper_1806_03461_amd as T
    sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
    rng = np.random.default_rng(count)
    a, b = rng.integers(0, 2, count).astype(np.uint8), rng.integers(0, 2, count).astype(np.uint8)
    cta, ctb = T.tfhe_encrypt(sk, 401, a), T.tfhe_encrypt(sk, 402, b)
    da, db = T.to_device(cta), T.to_device(ctb)
    out, small = torch.empty_like(da), torch.empty_like(da)
    T.tfhe_gate_batch(ck, "NOR", da, db, out, count)
    for at in range(0, count, 250):
        n = min(250, count - at)
        T.tfhe_gate_batch(ck, "NOR", da[at:], db[at:], small[at:], n)
    torch.cuda.synchronize()
    assert torch.equal(out, small)
    host = T.to_host(out)
    for i in (0, 3, count // 2, count - 2, count - 1):
        assert np.array_equal(host[i], real_keys.gate("NOR", cta[i], ctb[i])), i


def test_rounding_margin_and_multiplexers_of_a_large_batch(real_keys):
    """1,041 multiplexers = 2,082 items: a round on the wave kernel and a remainder elsewhere.  They decrypt to
    s ? a : b, sampled ones equal the oracle's, and the transform outputs stay far from a rounding tie."""
    import torch
    import paper_1806_03461_amd as T
    sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
    rng = np.random.default_rng(8)
    m = 1041
    s, a, b = (rng.integers(0, 2, m).astype(np.uint8) for _ in range(3))
    cts, cta, ctb = T.tfhe_encrypt(sk, 411, s), T.tfhe_encrypt(sk, 412, a), T.tfhe_encrypt(sk, 413, b)
    out = torch.empty((m, 501), dtype=torch.int32, device="cuda")
    T.tfhe_rounding_margin_enable(ck, True)
    T.tfhe_mux_batch(ck, T.to_device(cts), T.to_device(cta), T.to_device(ctb), out, m)
    worst = T.tfhe_rounding_margin_read(ck)
    T.tfhe_rounding_margin_enable(ck, False)
    assert 0 < worst < 1e-3, worst          # derived bound 2^-4.5; measured 6e-5 with a generated key
    host = T.to_host(out)
    assert np.array_equal(T.tfhe_decrypt(sk, host), np.where(s == 1, a, b))
    for i in (0, 1, 1022, 1023, 1024, 1025, m - 1):
        assert np.array_equal(host[i], real_keys.mux(cts[i], cta[i], ctb[i])), i


@pytest.mark.parametrize("count", [1, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513])
def test_batches_around_the_small_limits(real_keys, count):
    """One item to either side of each change of kernel: one, two or three gates per CU in the blind rotation, 32, 64 or
    128 gates and an eighth or a sixteenth of the mask words per workgroup in the key switch.  First and last gates
    equal the oracle's, all equal the same gates in other batches."""
    import torch
    import paper_1806_03461_amd as T
    sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
    rng = np.random.default_rng(1000 + count)
    cta, ctb = (T.tfhe_encrypt(sk, 420 + k, rng.integers(0, 2, count).astype(np.uint8)) for k in range(2))
    da, db = T.to_device(cta), T.to_device(ctb)
    out, other = torch.empty_like(da), torch.empty_like(da)
    T.tfhe_gate_batch(ck, "XNOR", da, db, out, count)
    step = 31 if count <= 256 else 300
    for at in range(0, count, step):
        n = min(step, count - at)
        T.tfhe_gate_batch(ck, "XNOR", da[at:], db[at:], other[at:], n)
    torch.cuda.synchronize()
    assert torch.equal(out, other)
    host = T.to_host(out)
    for i in {0, count // 2, count - 1}:
        assert np.array_equal(host[i], real_keys.gate("XNOR", cta[i], ctb[i])), i
