"""What a program built on this library has it do, as cases that can be timed and compared.

A server holds one client's cloud key on the GPU and evaluates gates, gate streams and layers on
ciphertexts; the client encrypts its bits and decrypts the answers on its host.  The cases cover
that work from the smallest call to the widest launch: a handful of gates (one gate's latency),
batches that leave the chip partly filled, batches that fill it many times, multiplexers, a lowered
circuit that a program keeps and runs again, single neurons (deep and narrow), layers with and
without the options that save gates, a convolution, and the client's side.  All use the benchmark
parameter set (n = 500, N = 1024); weights, thresholds and bits follow the distributions of the
benchmark configurations.  Ciphertexts are whole numbers: every output has to be the same bytes.
"""
import math
import random

import numpy as np
import torch

import paper_1806_03461_amd as T

KEY_SEED = 0x7A9A5EED
WORDS = 501                      # 32-bit words of a ciphertext
OPS = ["NAND", "AND", "OR", "NOR", "XOR", "XNOR"]

# largest drawn case, in bootstrapped gates (two per multiplexer): about the largest listed one
MOST_GATES = 110_000

_keys = {}


def _client():
    """The one key pair of this process: a server keeps its client's key on the GPU."""
    if "sk" not in _keys:
        _keys["sk"], _keys["ck"] = T.tfhe_keygen(T.default_params(), KEY_SEED)
        if torch.cuda.is_available():
            T.tfhe_cloud_key_upload(_keys["ck"])
    return _keys["sk"], _keys["ck"]


def listed():
    return [
        # one 8-gate call: the latency of a single bootstrapped gate, as an interactive circuit sees it
        {"name": "gates_8", "kind": "gates", "op": "NAND", "count": 8},
        # just past one gate per compute unit, an odd size: a narrow level of a circuit
        {"name": "gates_301", "kind": "gates", "op": "XNOR", "count": 301},
        # the largest batch of the call that allocates nothing (serving loops, graph capture)
        {"name": "noalloc_4096", "kind": "noalloc", "op": "OR", "count": 4096},
        # a saturating flat batch: what the gate rate is quoted on
        {"name": "gates_65536", "kind": "gates", "op": "XOR", "count": 65536},
        # three-input multiplexers, two blind rotations and one key switch each; odd count
        {"name": "mux_777", "kind": "mux", "count": 777},
        # a circuit lowered once, kept, and run on new wires: 784 -> 6 with Algorithm 1's comparator
        {"name": "stream_784x6", "kind": "stream", "d": 784, "p": 6, "zeros": 0.0, "flags": T.LOWER_MUX_COMPARATOR},
        # one 256-input neuron: 29 depths of at most 256 gates, latency-bound
        {"name": "neuron_256", "kind": "dense", "d": 256, "p": 1, "zeros": 0.0, "scores": False, "flags": T.LOWER_DEFAULT},
        # the last layer of a sparsified image network (half of the weights zero): 10 popcounts as scores
        {"name": "scores_256x10", "kind": "dense", "d": 256, "p": 10, "zeros": 0.5, "scores": True, "flags": T.LOWER_DEFAULT},
        # a tabular network's first layer: few units of wide fan-in
        {"name": "dense_1704x10", "kind": "dense", "d": 1704, "p": 10, "zeros": 0.0, "scores": False, "flags": T.LOWER_DEFAULT},
        # an image layer, a slice of its units, lowered with both options that save gates
        {"name": "shared_784x32", "kind": "dense", "d": 784, "p": 32, "zeros": 0.0, "scores": False,
         "flags": T.LOWER_PLUS_ONE | T.LOWER_SHARE_GATES},
        # a 3x3 convolution, 16 channels in, pad 1, on a tile of the image
        {"name": "conv_16x9x7", "kind": "conv", "c": 16, "h": 9, "w": 7, "o": 1, "k": 3, "pad": 1, "flags": T.LOWER_DEFAULT},
        # the client: encrypt a 16-channel 28x28 input and decrypt as many answer bits
        {"name": "client_12544", "kind": "client", "count": 12544},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above; sizes spread over their logarithm."""
    kind = rng.choice(["gates", "gates", "noalloc", "mux", "stream", "dense", "dense", "dense", "conv", "client"])
    if kind == "gates":
        return {"kind": kind, "op": rng.choice(OPS), "count": _log_int(rng, 1, 65536)}
    if kind == "noalloc":
        return {"kind": kind, "op": rng.choice(OPS), "count": _log_int(rng, 1, 4096)}
    if kind == "mux":
        return {"kind": kind, "count": _log_int(rng, 1, 20000)}
    if kind == "client":
        return {"kind": kind, "count": _log_int(rng, 10, 12544)}
    if kind == "conv":
        k = rng.choice([3, 3, 5])
        c = _log_int(rng, 1, 32)
        pad = rng.choice([0, k // 2])
        h, w = rng.randint(k, 16), rng.randint(k, 16)
        pixels = (h + 2 * pad - k + 1) * (w + 2 * pad - k + 1)
        while pixels * c * k * k * 7 > MOST_GATES and c > 1:
            c //= 2
        o = _log_int(rng, 1, max(1, min(32, MOST_GATES // (pixels * c * k * k * 7))))
        flags = rng.choice([T.LOWER_DEFAULT, T.LOWER_DEFAULT, T.LOWER_PLUS_ONE, T.LOWER_SHARE_GATES])
        return {"kind": kind, "c": c, "h": h, "w": w, "o": o, "k": k, "pad": pad, "flags": flags}
    d = _log_int(rng, 10, 1704)
    zeros = rng.choice([0.0, 0.0, 0.5])
    flags = rng.choice([T.LOWER_DEFAULT, T.LOWER_DEFAULT, T.LOWER_MUX_COMPARATOR, T.LOWER_PLUS_ONE, T.LOWER_SHARE_GATES,
                        T.LOWER_PLUS_ONE | T.LOWER_SHARE_GATES])
    p = _log_int(rng, 1, max(1, min(512, MOST_GATES // (8 * d))))
    case = {"kind": kind, "d": d, "p": p, "zeros": zeros, "flags": flags}
    if kind == "dense":
        case["scores"] = rng.random() < 0.25
    return case


def _weights(rng, shape, zeros):
    w = (2 * rng.integers(0, 2, shape) - 1).astype(np.int8)
    if zeros:
        w[rng.random(shape) < zeros] = 0
    return w


def _thresholds(rng, w):
    """One integer threshold per unit, uniform in [ceil(0.38 m), floor(0.62 m)] of its m non-zero weights."""
    m = (w.reshape(w.shape[0], -1) != 0).sum(axis=1)
    lo, hi = np.ceil(0.38 * m), np.floor(0.62 * m)
    hi = np.maximum(lo, hi)
    return (lo + np.floor(rng.random(w.shape[0]) * (hi - lo + 1))).astype(np.int32)


def _out_side(case):
    return case["h"] + 2 * case["pad"] - case["k"] + 1, case["w"] + 2 * case["pad"] - case["k"] + 1


def _layer(case, rng):
    """Weights and thresholds of a layer case, as the server holds them."""
    if case["kind"] == "conv":
        w = _weights(rng, (case["o"], case["c"], case["k"], case["k"]), 0.0)
    else:
        w = _weights(rng, (case["p"], case["d"]), case["zeros"])
    return w, None if case.get("scores") else _thresholds(rng, w)


def prepare(case, seed):
    sk, ck = _client()
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 1806])
    kind = case["kind"]

    def bits(n):
        return rng.integers(0, 2, n).astype(np.uint8)

    def encrypted(n, k):
        return T.to_device(T.tfhe_encrypt(sk, 1000 * seed + k, bits(n)))

    def empty(n):
        return torch.empty((n, WORDS), dtype=torch.int32, device="cuda")

    s = {"case": case, "ck": ck}
    if kind == "client":
        s["sk"], s["bits"], s["seed"] = sk, bits(case["count"]), 1000 * seed + 1
        s["answers"] = T.tfhe_encrypt(sk, 1000 * seed + 2, bits(case["count"]))
    elif kind in ("gates", "noalloc"):
        n = case["count"]
        s["a"], s["b"], s["out"] = encrypted(n, 1), encrypted(n, 2), empty(n)
    elif kind == "mux":
        n = case["count"]
        s["s"], s["a"], s["b"], s["out"] = encrypted(n, 1), encrypted(n, 2), encrypted(n, 3), empty(n)
    elif kind == "stream":
        w, t = _layer(case, rng)
        gates, _, nwires = T.bnn_dense_lower_opts(case["d"], w, t, case["p"], 0, case["flags"])
        wires = torch.zeros((nwires, WORDS), dtype=torch.int32, device="cuda")
        wires[:case["d"]] = encrypted(case["d"], 1)
        for bit in (0, 1):
            wires[case["d"] + bit] = T.to_device(T.tfhe_trivial(T.default_params(), bit))
        s["gates"], s["wires"], s["nwires"] = gates, wires, nwires
    elif kind == "dense":
        s["w"], s["t"] = _layer(case, rng)
        s["x"] = encrypted(case["d"], 1)
        s["out_bits"] = int(case["d"]).bit_length() if case["scores"] else 0
        s["out"] = empty(case["p"] * max(1, s["out_bits"]))
    else:
        s["w"], s["t"] = _layer(case, rng)
        ho, wo = _out_side(case)
        s["x"], s["out"] = encrypted(case["c"] * case["h"] * case["w"], 1), empty(case["o"] * ho * wo)
    return s


def run(s):
    case, ck = s["case"], s["ck"]
    kind = case["kind"]
    if kind == "client":
        return {"ciphertexts": T.tfhe_encrypt(s["sk"], s["seed"], s["bits"]), "answers": T.tfhe_decrypt(s["sk"], s["answers"])}
    if kind == "gates":
        T.tfhe_gate_batch(ck, case["op"], s["a"], s["b"], s["out"], case["count"])
    elif kind == "noalloc":
        T.tfhe_gate_batch_noalloc(ck, case["op"], s["a"], s["b"], s["out"], case["count"])
    elif kind == "mux":
        T.tfhe_mux_batch(ck, s["s"], s["a"], s["b"], s["out"], case["count"])
    elif kind == "stream":
        T.tfhe_gate_stream(ck, s["gates"], s["wires"], s["nwires"])
        return s["wires"]
    elif kind == "dense":
        T.bnn_dense_encrypted_opts(ck, s["x"], case["d"], s["w"], s["t"], case["p"], s["out"], s["out_bits"], case["flags"])
    else:
        T.bnn_conv_encrypted_opts(ck, s["x"], case["c"], case["h"], case["w"], s["w"], s["t"], 1, case["pad"], s["out"],
                                  case["flags"])
    return s["out"]


# One blind rotation: 500 steps of 8 complex 512-point transforms (5 N log2 N), their twists, and 16
# pointwise products of 512 complex values; one key switch: three quarters of 1,024 x 8 rows of 501 words.
ROTATION_FLOPS = 500 * (8 * 5 * 512 * 9 + 8 * 512 * 6 + 16 * 512 * 8)
SWITCH_OPS = 1024 * 8 * 3 // 4 * WORDS
KEY_BYTES = 4 * (500 * 4 * 2 * 1024 + 1024 * 8 * 3 * WORDS)      # both evaluation keys, as a client sends them
CT_BYTES = 4 * WORDS


def work(case):
    """Bytes: inputs, outputs and the cloud key, once each.  Operations: every gate's transforms and switch."""
    kind = case["kind"]
    if kind == "client":
        # each ciphertext written or read once; one 64-bit mixing step (about 8 operations) per word
        return {"bytes": 2 * case["count"] * (CT_BYTES + 1), "flops": case["count"] * WORDS * 10}
    if kind in ("gates", "noalloc", "mux"):
        rotations = case["count"] * (2 if kind == "mux" else 1)
        switches = case["count"]
        cts = case["count"] * (4 if kind == "mux" else 3)
    else:
        # the circuit of one set of weights: the gate count varies by a few per cent between sets
        rng = np.random.default_rng([7, 1806])
        w, t = _layer(case, rng)
        if kind == "conv":
            gates, outs, nwires = T.bnn_conv_lower_opts(case["c"], case["h"], case["w"], w, t, 1, case["pad"], case["flags"])
            cts = case["c"] * case["h"] * case["w"] + outs.size
        else:
            bits = int(case["d"]).bit_length() if case.get("scores") else 0
            gates, outs, nwires = T.bnn_dense_lower_opts(case["d"], w, t, case["p"], bits, case["flags"])
            cts = nwires if kind == "stream" else case["d"] + outs.size
        rotations = int(gates.size)
        switches = int((gates["op"] != T.MUX_ELSE).sum())
    return {"bytes": KEY_BYTES + cts * CT_BYTES, "flops": rotations * ROTATION_FLOPS + switches * SWITCH_OPS}


def tolerance(case):
    return "exact"
