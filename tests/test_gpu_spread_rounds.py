"""GPU parity where a partial round goes to a launch of its own: on the wave kernel with one workgroup per CU, or five or six
gates per CU spread evenly over two workgroups, where some waves have no gate, alone and behind a whole round; and three or
five gates per CU behind a round, which the four-wave kernel takes."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def check(real_keys, count):
    """First and last gates of each launch equal the oracle's, and all of them the same gates in small batches."""
    import torch
    import paper_1806_03461_amd as T
    sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
    rng = np.random.default_rng(count)
    cta, ctb = (T.tfhe_encrypt(sk, 430 + k, rng.integers(0, 2, count).astype(np.uint8)) for k in range(2))
    da, db = T.to_device(cta), T.to_device(ctb)
    out, small = torch.empty_like(da), torch.empty_like(da)
    T.tfhe_gate_batch(ck, "NAND", da, db, out, count)
    for at in range(0, count, 250):
        n = min(250, count - at)
        T.tfhe_gate_batch(ck, "NAND", da[at:], db[at:], small[at:], n)
    torch.cuda.synchronize()
    assert torch.equal(out, small)
    host = T.to_host(out)
    for i in {0, count // 2, min(2048, count - 1), count - 1}:
        assert np.array_equal(host[i], real_keys.gate("NAND", cta[i], ctb[i])), i


@pytest.mark.parametrize("count", [1027, 1535, 1536, 1537, 3072, 3329, 3583])
def test_partial_rounds_on_the_wave_kernel(real_keys, count):
    check(real_keys, count)


@pytest.mark.parametrize("count", [2561, 2816, 3073, 3328])
def test_partial_rounds_behind_a_round_on_the_four_wave_kernel(real_keys, count):
    check(real_keys, count)
