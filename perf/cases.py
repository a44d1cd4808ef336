"""Workloads of the fused FFN and convolution chains, called the way a program that uses the library calls
them: operands and output on the device, ONE workspace registered for the process, the plan left to the
library's chooser, one asynchronous call per layer on the current stream.

    standard:  Y = act(X W1) W2          gated:  Y = (act(X W1) .* (X W3)) W2
    conv    :  Y = conv1x1(act(conv_k(X, W1)), W2), k = 1 or 3, channels-last

Shapes are (M, K, N1, N2): rows, model width, hidden width, output width.
"""
import math

import torch

from paper_2512_12949_amd import binding as ff
from paper_2512_12949_amd import inputs

_ACTS = {"relu": inputs.ACT_RELU, "gelu": inputs.ACT_GELU_TANH, "silu": inputs.ACT_SILU}
_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_CALL = {"bf16": ff.ffuse_ffn, "f16": ff.ffuse_ffn_f16, "f32": ff.ffuse_ffn_f32}
_CONV = {"bf16": ff.ffuse_conv_chain, "f16": ff.ffuse_conv_chain_f16}


def _ffn(M, K, N1, N2, dtype, act, gated=False, dist="normal"):
    return {"kind": "ffn", "M": M, "K": K, "N1": N1, "N2": N2, "dtype": dtype, "act": act, "gated": gated, "dist": dist}


def _conv(B, H, W, IC, OC1, OC2, k1, dtype="bf16"):
    return {"kind": "conv", "B": B, "H": H, "W": W, "IC": IC, "OC1": OC1, "OC2": OC2, "k1": k1, "dtype": dtype, "act": "relu"}


def listed():
    cases = {
        # the fp32 mode, on the benchmark's small chain: what one checks a schedule or a training script with
        "tiny_f32": _ffn(128, 256, 1024, 256, "f32", "relu"),
        # generating one token for one user: a single row through a 7B-class gated layer
        "token1": _ffn(1, 4096, 11008, 4096, "bf16", "silu", gated=True),
        # generating for a batch: 16 rows through a 70B-class gated layer; 1.4 GB of weights per call
        "decode16": _ffn(16, 8192, 28672, 8192, "bf16", "silu", gated=True),
        # the smallest transformer layers, 128 tokens: a call is launches and waits more than bytes
        "small128": _ffn(128, 384, 1536, 384, "bf16", "gelu"),
        # a short prompt, or a large decode batch, through a 7B-class gated layer
        "prompt128": _ffn(128, 4096, 11008, 4096, "bf16", "silu", gated=True),
        # sizes that divide nothing evenly: rows, widths and hidden width off every tile
        "ragged": _ffn(333, 1016, 2744, 1016, "f16", "gelu"),
        # a prompt of a few hundred tokens through a wide standard layer: neither bytes nor flops alone
        "prompt512": _ffn(512, 4096, 16384, 4096, "bf16", "gelu"),
        # prefill of long prompts: the benchmark's gated and standard layers
        "prefill2048": _ffn(2048, 4096, 11008, 4096, "bf16", "silu", gated=True),
        "prefill4096": _ffn(4096, 4096, 16384, 4096, "bf16", "gelu"),
        # very many rows of a narrow model (an encoder over a corpus): the intermediate is 512 MB
        "rows32768": _ffn(32768, 1024, 8192, 1024, "f16", "relu", dist="uniform"),
        # bottleneck blocks of a convolutional network: an early and a late stage
        "conv_early": _conv(1, 56, 56, 64, 256, 64, 1),
        "conv_late": _conv(1, 14, 14, 256, 256, 1024, 3),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def _width(rng, lo, hi):
    """A layer width: as published models have them (multiples of 128), or any multiple of 8."""
    return _log(rng, lo, hi, rng.choice((8, 128)))


# the most a drawn case may cost: flops, weight bytes and intermediate bytes, with room for shapes that run
# less efficiently than the largest listed ones
_MAX_FLOPS = 0.6e12
_MAX_WEIGHTS = 1.3e9
_MAX_HIDDEN = 500e6


def draw(rng):
    kind = rng.choice(("f32", "decode", "decode", "short", "short", "mid", "mid", "long", "conv1", "conv3"))
    if kind == "f32":
        return _ffn(_log(rng, 16, 256), _width(rng, 64, 512), _width(rng, 256, 2048), _width(rng, 64, 512), "f32",
                    rng.choice(("relu", "gelu", "silu")), gated=rng.random() < 0.3)
    if kind in ("conv1", "conv3"):
        side = _log(rng, 7, 56)
        c = 64 * _log(rng, 1, 8)
        out = 8 * _log(rng, 8, 256) if kind == "conv3" else c
        return _conv(_log(rng, 1, 4), side, side, c, 8 * _log(rng, 8, 64) if kind == "conv3" else 4 * c, out, 3 if kind == "conv3" else 1,
                     rng.choice(("bf16", "bf16", "f16")))
    rows = {"decode": (1, 64), "short": (65, 256), "mid": (257, 2048), "long": (2049, 32768)}[kind]
    dims = {"decode": (1024, 8192), "short": (128, 4096), "mid": (256, 4096), "long": (256, 4096)}[kind]
    while True:
        M = _log(rng, *rows)
        K = _width(rng, *dims)
        N2 = K if rng.random() < 0.8 else _width(rng, *dims)
        N1 = min(28672, int(K * rng.uniform(2.0, 4.5)) // 8 * 8) if rng.random() < 0.5 else _width(rng, 2 * dims[0], 4 * dims[1])
        gated = rng.random() < 0.5
        c = _ffn(M, K, N1, N2, rng.choice(("bf16", "bf16", "f16")), "silu" if gated else rng.choice(("relu", "gelu")), gated=gated)
        if work(c)["flops"] <= _MAX_FLOPS and 2 * N1 * ((2 if gated else 1) * K + N2) <= _MAX_WEIGHTS and 2 * M * N1 <= _MAX_HIDDEN:
            return c


_workspace = None


def _register_workspace():
    """The process's one workspace: enough for every chain of these ranges."""
    global _workspace
    if _workspace is None:
        need = max(ff.ffuse_workspace_bytes(ff.DTYPE_CODE[c["dtype"]], c["gated"], c["M"], c["K"], c["N1"], c["N2"])
                   for c in listed() if c["kind"] == "ffn")
        _workspace = torch.empty(max(need, 1 << 30), dtype=torch.uint8, device="cuda")
        ff.ffuse_set_workspace(_workspace)


def _tensors(case, seed):
    """The operands of a case in the order of its call (X, W1, W3 or None, W2), from the seed alone."""
    dt = _TORCH[case["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def tensor(shape, scale):
        t = torch.empty(shape, dtype=dt, device="cuda")
        if case.get("dist") == "uniform":
            return t.uniform_(-scale, scale, generator=gen)
        return t.normal_(0.0, scale, generator=gen)

    if case["kind"] == "conv":
        B, H, W, IC, OC1, OC2, k = (case[n] for n in ("B", "H", "W", "IC", "OC1", "OC2", "k1"))
        return (tensor((B, H, W, IC), 1.0), tensor((k, k, IC, OC1), (k * k * IC) ** -0.5), None,
                tensor((1, 1, OC1, OC2), OC1 ** -0.5))
    M, K, N1, N2 = (case[n] for n in ("M", "K", "N1", "N2"))
    X, W1 = tensor((M, K), 1.0), tensor((K, N1), K ** -0.5)
    W3 = tensor((K, N1), K ** -0.5) if case["gated"] else None
    return X, W1, W3, tensor((N1, N2), N1 ** -0.5)


def prepare(case, seed):
    _register_workspace()
    s = {"kind": case["kind"], "act": _ACTS[case["act"]]}
    s["call"] = (_CONV if case["kind"] == "conv" else _CALL)[case["dtype"]]
    s["X"], s["W1"], s["W3"], s["W2"] = _tensors(case, seed)
    shape = (case["B"], case["H"], case["W"], case["OC2"]) if case["kind"] == "conv" else (case["M"], case["N2"])
    s["Y"] = torch.empty(shape, dtype=_TORCH[case["dtype"]], device="cuda")
    return s


def run(state):
    if state["kind"] == "conv":
        state["call"](state["X"], state["W1"], state["W2"], state["act"], state["Y"])
    else:
        state["call"](state["X"], state["W1"], state["W3"], state["W2"], state["act"], state["Y"])
    return state["Y"]


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "conv":
        pix, kk = case["B"] * case["H"] * case["W"], case["k1"] ** 2
        IC, OC1, OC2 = case["IC"], case["OC1"], case["OC2"]
        return {"bytes": e * (pix * IC + kk * IC * OC1 + OC1 * OC2 + pix * OC2), "flops": 2 * pix * OC1 * (kk * IC + OC2)}
    M, K, N1, N2 = (case[n] for n in ("M", "K", "N1", "N2"))
    g = 2 if case["gated"] else 1
    return {"bytes": e * (M * K + g * K * N1 + N1 * N2 + M * N2), "flops": 2 * M * N1 * (g * K + N2)}


# Measured against the same chain in 64 bits over 23 shapes of these ranges (two roundings to the operand type
# in all: the intermediate's and the output's): rel 2.4e-3, max 1.2e-2 in bf16; 3.0e-4 and 1.3e-3 in fp16;
# 3.5e-7 and 1.6e-6 in fp32.  Stated: about four times that.
_TOLERANCE = {"bf16": {"rel": 1e-2, "max": 0.05}, "f16": {"rel": 1.2e-3, "max": 5e-3}, "f32": {"rel": 1.5e-6, "max": 7e-6}}


def tolerance(case):
    return dict(_TOLERANCE[case["dtype"]])


_EXACT_ACT = {"relu": torch.relu, "gelu": lambda v: torch.nn.functional.gelu(v, approximate="tanh"),
              "silu": torch.nn.functional.silu}


def exact(case, seed):
    """The chain in 64 bits, with nothing rounded between its products."""
    X, W1, W3, W2 = (None if t is None else t.double() for t in _tensors(case, seed))
    act = _EXACT_ACT[case["act"]]
    if case["kind"] == "ffn":
        h = act(X @ W1)
        if W3 is not None:
            h *= X @ W3
        return h @ W2
    k, H, W = case["k1"], case["H"], case["W"]
    padded = torch.nn.functional.pad(X, (0, 0, k // 2, k // 2, k // 2, k // 2))
    h = sum(padded[:, i:i + H, j:j + W].reshape(-1, case["IC"]) @ W1[i, j] for i in range(k) for j in range(k))
    return (act(h) @ W2[0, 0]).reshape(case["B"], H, W, case["OC2"])
