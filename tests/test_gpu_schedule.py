"""Circuits whose levels are filled by launch size: gates with slack run in later launches than their depth,
multiplexer pairs included.  Every wire must hold the bytes that evaluating the circuit depth by depth gives,
each depth in a call of its own (a call of one depth has nothing to move)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,p,flag", [(64, 24, "LOWER_DEFAULT"), (40, 30, "LOWER_MUX_COMPARATOR"), (33, 48, "LOWER_PLUS_ONE"),
                                      (9, 300, "LOWER_SHARE_GATES")])
def test_filled_levels_leave_every_wire_unchanged(d, p, flag):
    import torch
    import paper_1806_03461_amd as T
    sk, ck = T.tfhe_keygen(T.default_params(), workloads.KEY_SEED)
    rng = np.random.default_rng(d)
    W = (2 * rng.integers(0, 2, (p, d)) - 1).astype(np.int8)
    Tt = rng.integers(1, d, p).astype(np.int32)
    gates, outs, nw = T.bnn_dense_lower_opts(d, W, Tt, p, 0, getattr(T, flag))
    x = rng.integers(0, 2, d).astype(np.uint8)
    wires = np.zeros((nw, 501), np.uint32)
    wires[:d] = T.tfhe_encrypt(sk, 71, x)
    wires[d], wires[d + 1] = T.tfhe_trivial(T.default_params(), 0), T.tfhe_trivial(T.default_params(), 1)
    whole, by_depth = T.to_device(wires), T.to_device(wires)
    T.tfhe_gate_stream(ck, gates, whole, nw)

    depth, level = np.zeros(nw, np.int64), np.zeros(len(gates), np.int64)
    for g, r in enumerate(gates):
        second = r["op"] == T.MUX_ELSE
        ins = [r["in0"], r["in1"]] + ([gates[g + 1]["in1"]] if r["op"] == T.MUX else [])
        level[g] = level[g - 1] if second else 1 + depth[ins].max()
        depth[r["out"]] = level[g]
    widths = np.bincount(level)[1:]
    assert widths.max() > 256 and len(widths) > 4       # wider than a gate per compute unit: the filling applies
    for l in range(1, len(widths) + 1):
        T.tfhe_gate_stream(ck, gates[level == l], by_depth, nw)
    torch.cuda.synchronize()
    assert torch.equal(whole, by_depth)
    # the layer call (slots of the wire pool are reused between the same levels)
    res = torch.empty((p, 501), dtype=torch.int32, device="cuda")
    T.bnn_dense_encrypted_opts(ck, T.to_device(wires[:d]), d, W, Tt, p, res, 0, getattr(T, flag))
    torch.cuda.synchronize()
    # filling did move gates: the pool is not the one that earliest levels give
    assert T.tfhe_last_layer_stats(ck)["pool_wires"] != T.tfhe_plan_wire_pool(gates, nw, d + 2, outs)[2]
    host = T.to_host(by_depth)
    want = np.stack([(host[o["wire"]] if not o["value"] else 0 - host[o["wire"]]) if o["wire"] >= 0 else
                     T.tfhe_trivial(T.default_params(), int(o["value"])) for o in outs])
    assert np.array_equal(T.to_host(res), want)
    S = ((W > 0) & (x == 1)).sum(1) + ((W < 0) & (x == 0)).sum(1)
    assert np.array_equal(T.tfhe_decrypt(sk, T.to_host(res)), (S >= Tt).astype(np.uint8))
