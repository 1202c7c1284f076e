"""The work that programs have this library do, as cases that can be timed: products with quantised weights at decode and
prefill batch sizes, decoding of whole layers, and the quantiser's side (encoder, search, block-wise loop, group scales).

A case is a dict of plain values; `prepare` makes what a program has in hand before the call (weights, activations,
outputs, a context), `run` makes one pass through the library's public calls and returns what they wrote.  Inputs are
drawn on the device from the seed: indices uniform over the code, log-normal fp16 gains, standard normal activations and
weights (the distributions of paper_2603_11021_amd/synth.py).  Layer sizes are those of the Llama-3-8B- and
70B-shaped transformer blocks of that module, and sizes between and below them, odd ones among them.
"""
import math

import numpy as np
import torch

from paper_2603_11021_amd import LLVQ, LLVQ_ANGULAR, LLVQ_EUCLIDEAN
from paper_2603_11021_amd.synth import N_SHELL2, chi_gain_levels

DTYPES = {"int8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
SIZES = {"int8": 1, "f16": 2, "bf16": 2, "f32": 4}
# bytes of a block's stored word and gain: 48-bit index + fp16 gain; 64-bit index + fp16 gain; index and gain in one 64-bit
# word (llvq_repack); 47-bit index + one gain bit in a 48-bit word
WORDS = {"u48": 8, "u64": 10, "packed": 8, "gain_bit": 6}

_contexts = {}


def _context(m_max):
    """One context per union of shells, kept as a serving or quantising program keeps it."""
    if m_max not in _contexts:
        _contexts[m_max] = LLVQ(m_max, 0)
    return _contexts[m_max]


def _kb(K):
    return (K + 23) // 24


def listed():
    return [
        # the decode unit: indices of the first shell to int8 vectors; the smallest call, where launch and latency count
        {"name": "decode_unit", "kind": "decode", "n": 65536, "m_max": 13, "out": "int8", "code": "shell2", "words": "u48"},
        # one layer at batch 1: the matrix-vector product of token generation
        {"name": "gemv_4096", "kind": "matmul", "N": 4096, "K": 4096, "M": 1, "x": "f16", "m_max": 13, "words": "u48"},
        # the linear layers of a transformer block, generating for one sequence and for sixteen
        {"name": "block_8b_m1", "kind": "block", "hidden": 4096, "kv": 1024, "ffn": 14336, "M": 1, "x": "f16"},
        {"name": "block_8b_m16", "kind": "block", "hidden": 4096, "kv": 1024, "ffn": 14336, "M": 16, "x": "f16"},
        # prompts: a short one, one of a ragged length, and a long one
        {"name": "block_8b_m64", "kind": "block", "hidden": 4096, "kv": 1024, "ffn": 14336, "M": 64, "x": "bf16"},
        {"name": "block_8b_m250", "kind": "block", "hidden": 4096, "kv": 1024, "ffn": 14336, "M": 250, "x": "f16"},
        {"name": "block_8b_m1024", "kind": "block", "hidden": 4096, "kv": 1024, "ffn": 14336, "M": 1024, "x": "bf16"},
        # loading: every layer of the largest block reconstructed to dense bf16 weights
        {"name": "load_70b", "kind": "load", "hidden": 8192, "kv": 1024, "ffn": 28672, "out": "bf16"},
        # the encoder side of the index map on a layer's worth of lattice points, not a multiple of anything
        {"name": "encode_2000003", "kind": "encode", "n": 2000003, "words": "u48"},
        # quantising a slice of a layer: nearest directions, indices, gain reset and error propagation, column by column
        {"name": "gptq_4096x384", "kind": "gptq", "N": 4096, "K": 384},
        # the closed-form group scales of a whole layer after the loop
        {"name": "group_scales_1024", "kind": "group_scales", "N": 1024, "K": 4096},
        # the larger union of shells (55-bit indices) at batch 1
        {"name": "gemv_4096_m19", "kind": "matmul", "N": 4096, "K": 4096, "M": 1, "x": "f16", "m_max": 19, "words": "u64"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case.  The largest listed products (9.1 M blocks at M = 1024) and the largest listed load (36 M blocks,
    1.7 GB written) bound what is drawn."""
    kind = rng.choice(["decode", "matmul", "matmul", "block", "block", "block", "load", "encode", "quantize", "gptq", "group_scales", "union19"])
    if kind == "decode":
        out = rng.choice(["int8", "f16", "bf16", "f32"])
        return {"kind": kind, "n": _log(rng, 1000, 16_000_000), "m_max": 13, "out": out, "code": rng.choice(["union", "union", "shell2"]),
                "words": rng.choice(["u48", "u48", "u64"])}
    if kind == "matmul":
        return {"kind": kind, "N": _log(rng, 512, 14336), "K": _log(rng, 512, 14336), "M": _log(rng, 1, 1024), "x": rng.choice(["f16", "bf16"]),
                "m_max": 13, "words": rng.choice(["u48", "u48", "u64", "packed", "gain_bit"])}
    if kind == "block":
        M = _log(rng, 1, 1024)
        hidden = 8 * _log(rng, 128, 512 if M > 64 else 1024)
        return {"kind": kind, "hidden": hidden, "kv": rng.choice([hidden, hidden // 4, hidden // 8]), "ffn": int(3.5 * hidden) if rng.random() < 0.5
                else 8 * _log(rng, hidden // 4, int(0.4 * hidden)), "M": M, "x": rng.choice(["f16", "bf16"])}
    if kind == "load":
        hidden = 8 * _log(rng, 128, 1000)
        return {"kind": kind, "hidden": hidden, "kv": hidden // 4, "ffn": int(3.5 * hidden), "out": rng.choice(["f16", "bf16"])}
    if kind == "encode":
        return {"kind": kind, "n": _log(rng, 1000, 4_000_000), "words": rng.choice(["u48", "u48", "u64"])}
    if kind == "quantize":
        return {"kind": kind, "n": _log(rng, 256, 65536), "metric": rng.choice(["angular", "angular", "euclidean"])}
    if kind == "gptq":
        return {"kind": kind, "N": _log(rng, 128, 4096), "K": 24 * rng.randint(2, 16)}
    if kind == "group_scales":
        return {"kind": kind, "N": _log(rng, 64, 1024), "K": _log(rng, 192, 4096)}
    if rng.random() < 0.5:
        return {"kind": "decode", "n": _log(rng, 1000, 4_000_000), "m_max": 19, "out": rng.choice(["int8", "f16", "bf16"]), "code": "union", "words": "u64"}
    return {"kind": "matmul", "N": _log(rng, 512, 4096), "K": _log(rng, 512, 4096), "M": _log(rng, 1, 16), "x": rng.choice(["f16", "bf16"]),
            "m_max": 19, "words": "u64"}


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _indices(g, n, high, words):
    idx = torch.randint(0, high, (n,), dtype=torch.int64, device="cuda", generator=g)
    return idx if words == "u64" else idx.view(torch.uint8).view(n, 8)[:, :6].contiguous()


def _gains(g, n):
    return torch.exp(0.5 * torch.randn(n, device="cuda", generator=g)).to(torch.float16)


def _activations(g, M, K, x):
    """M rows of K values, zero-padded to whole blocks of 24 channels."""
    a = torch.zeros((M, 24 * _kb(K)), dtype=DTYPES[x], device="cuda")
    a[:, :K] = torch.randn((M, K), device="cuda", generator=g).to(DTYPES[x])
    return a


def _second_moments(g, K):
    """Second moments of correlated inputs with unequal variances, damped, as calibration gives them."""
    z = torch.randn((2 * K, K), device="cuda", generator=g)
    x = (z + 0.6 * z.roll(1, 1) + 0.3 * z.roll(7, 1)) * torch.linspace(1.0, 3.0, K, device="cuda")
    return x.t() @ x / (2 * K) + 0.05 * torch.eye(K, device="cuda")


# launches of a transformer block: layers that read the same input go together
def _block_layers(case):
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [((h, kv, kv), h), ((h,), h), ((f, f), h), ((h,), f)]


def _prepare_decode(case, g):
    q = _context(case["m_max"])
    n, out = case["n"], DTYPES[case["out"]]
    high = N_SHELL2 if case["code"] == "shell2" else q.num_points
    return {"q": q, "idx": _indices(g, n, high, case["words"]), "gain": _gains(g, n), "out": torch.empty((n, 24), dtype=out, device="cuda")}


def _run_decode(s):
    if s["out"].dtype == torch.int8:
        return s["q"].llvq_decode_i8(s["idx"], out=s["out"])
    return s["q"].llvq_decode(s["idx"], s["gain"], out_dtype=s["out"].dtype, out=s["out"])


def _prepare_matmul(case, g):
    q = _context(case["m_max"])
    N, KB, words = case["N"], _kb(case["K"]), case["words"]
    s = {"q": q, "N": N, "KB": KB, "words": words, "x": _activations(g, case["M"], case["K"], case["x"]),
         "y": torch.empty((case["M"], N), dtype=torch.float32, device="cuda")}
    if words == "gain_bit":
        # one integer carries shape and gain: any 47-bit index (half of the code) under one gain bit
        s["idx"] = _indices(g, N * KB, 1 << 48, "u48")
        s["lut"] = torch.from_numpy(chi_gain_levels(1)).to("cuda")
        return s
    s["idx"] = _indices(g, N * KB, q.num_points, "u64" if words == "u64" else "u48")
    s["gain"] = _gains(g, N * KB)
    if words == "packed":
        s["idx"] = q.llvq_repack(s["idx"], s.pop("gain"))
    return s


def _run_matmul(s):
    q, words = s["q"], s["words"]
    if words == "gain_bit":
        return q.llvq_matmul_coded(s["x"], s["idx"], s["N"], s["KB"], 47, gain_lut=s["lut"], out=s["y"])
    if words == "packed":
        return q.llvq_matmul_coded(s["x"], s["idx"], s["N"], s["KB"], 48, out=s["y"])
    return q.llvq_matmul(s["x"], s["idx"], s["gain"], s["N"], s["KB"], out=s["y"])


def _prepare_block(case, g):
    q = _context(13)
    launches = []
    inputs = {}
    for Ns, K in _block_layers(case):
        KB = _kb(K)
        if K not in inputs:
            inputs[K] = _activations(g, case["M"], K, case["x"])
        launches.append({"x": inputs[K], "KB": KB, "Ns": list(Ns), "idx": [_indices(g, N * KB, q.num_points, "u48") for N in Ns],
                         "gain": [_gains(g, N * KB) for N in Ns],
                         "y": [torch.empty((case["M"], N), dtype=torch.float32, device="cuda") for N in Ns]})
    return {"q": q, "launches": launches}


def _run_block(s):
    for c in s["launches"]:
        if len(c["Ns"]) == 1:
            s["q"].llvq_matmul(c["x"], c["idx"][0], c["gain"][0], c["Ns"][0], c["KB"], out=c["y"][0])
        else:
            s["q"].llvq_matmul_multi(c["x"], c["idx"], c["gain"], c["Ns"], c["KB"], outs=c["y"])
    return [c["y"] for c in s["launches"]]


def _prepare_load(case, g):
    q = _context(13)
    layers = []
    for Ns, K in _block_layers(case):
        for N in Ns:
            n = N * _kb(K)
            layers.append((_indices(g, n, q.num_points, "u48"), _gains(g, n), torch.empty((n, 24), dtype=DTYPES[case["out"]], device="cuda")))
    return {"q": q, "layers": layers}


def _run_load(s):
    return [s["q"].llvq_decode(idx, gain, out_dtype=out.dtype, out=out) for idx, gain, out in s["layers"]]


def _prepare_encode(case, g):
    q = _context(13)
    pts = q.llvq_decode_i8(_indices(g, case["n"], q.num_points, "u64"))
    fmt = 1 if case["words"] == "u64" else 0
    out = torch.empty(case["n"], dtype=torch.int64, device="cuda") if fmt else torch.empty((case["n"], 6), dtype=torch.uint8, device="cuda")
    return {"q": q, "pts": pts, "fmt": fmt, "out": out}


def _run_encode(s):
    return s["q"].llvq_encode(s["pts"], fmt=s["fmt"], out=s["out"])


def _prepare_quantize(case, g):
    w = torch.randn((case["n"], 24), device="cuda", generator=g)
    if case["metric"] == "euclidean":
        w *= math.sqrt(5.5)                     # the typical block falls inside the ball
    return {"q": _context(13), "w": w, "metric": LLVQ_ANGULAR if case["metric"] == "angular" else LLVQ_EUCLIDEAN}


def _run_quantize(s):
    return s["q"].llvq_quantize(s["w"], s["metric"])


def _prepare_gptq(case, g):
    N, K = case["N"], case["K"]
    H = _second_moments(g, K).double().cpu().numpy()
    G = np.linalg.inv(H)
    U = torch.from_numpy(np.linalg.cholesky((G + G.T) / 2).T.astype(np.float32).copy()).to("cuda")
    W = 0.02 * torch.randn((N, K), device="cuda", generator=g)
    return {"q": _context(13), "W": W, "work": torch.empty_like(W), "U": U}


def _run_gptq(s):
    # The call overwrites its copy of the layer with exactly what llvq_decode makes of the indices and gains: those are
    # the quantised layer, and what is returned.
    s["work"].copy_(s["W"])
    return s["q"].llvq_gptq_quantize(s["work"], s["U"])


def _prepare_group_scales(case, g):
    q = _context(13)
    N, KB = case["N"], _kb(case["K"])
    K = 24 * KB
    gain = (0.1 * torch.exp(0.2 * torch.randn((N, KB), device="cuda", generator=g))).to(torch.float16)
    Wq = q.llvq_decode(_indices(g, N * KB, q.num_points, "u48"), gain.reshape(-1), out_dtype=torch.float32).reshape(N, K)
    W0 = Wq + 0.28 * Wq.square().mean().sqrt() * torch.randn((N, K), device="cuda", generator=g)      # a layer that Wq approximates at 2 bits
    return {"q": q, "Wq": Wq, "gain": gain, "W0": W0, "H": _second_moments(g, K), "Wq_out": torch.empty_like(Wq), "gain_out": torch.empty_like(gain)}


def _run_group_scales(s):
    s["Wq_out"].copy_(s["Wq"])                  # the call refines the layer and its gains in place
    s["gain_out"].copy_(s["gain"])
    scales = s["q"].llvq_gptq_group_scales(s["Wq_out"], s["W0"], s["H"], s["gain_out"], lam=1e-3)
    return [scales, s["gain_out"], s["Wq_out"]]


_PREPARE = {"decode": _prepare_decode, "matmul": _prepare_matmul, "block": _prepare_block, "load": _prepare_load, "encode": _prepare_encode,
            "quantize": _prepare_quantize, "gptq": _prepare_gptq, "group_scales": _prepare_group_scales}
_RUN = {"decode": _run_decode, "matmul": _run_matmul, "block": _run_block, "load": _run_load, "encode": _run_encode,
        "quantize": _run_quantize, "gptq": _run_gptq, "group_scales": _run_group_scales}


def prepare(case, seed):
    s = _PREPARE[case["kind"]](case, _generator(seed))
    s["kind"] = case["kind"]
    return s


def run(state):
    return _RUN[state["kind"]](state)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def _product_work(M, Ns, K, word_bytes):
    """Words read once, activations read once, outputs written once; one multiplication and one addition per weight and row."""
    n = sum(Ns)
    return {"bytes": n * _kb(K) * word_bytes + 2 * M * K + 4 * M * n, "flops": 2 * M * n * K}


def work(case):
    kind = case["kind"]
    if kind == "decode":
        word = (8 if case["words"] == "u64" else 6) + (0 if case["out"] == "int8" else 2)
        return {"bytes": case["n"] * (word + 24 * SIZES[case["out"]]), "flops": 0}
    if kind == "matmul":
        return _product_work(case["M"], (case["N"],), case["K"], WORDS[case["words"]])
    if kind == "block":
        parts = [_product_work(case["M"], Ns, K, 8) for Ns, K in _block_layers(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if kind == "load":
        n = sum(N * _kb(K) for Ns, K in _block_layers(case) for N in Ns)
        return {"bytes": n * (8 + 24 * SIZES[case["out"]]), "flops": 0}
    if kind == "encode":
        return {"bytes": case["n"] * (24 + (8 if case["words"] == "u64" else 6)), "flops": 0}
    if kind == "quantize":
        return {"bytes": case["n"] * (96 + 24 + 6 + 4), "flops": 0}
    N, KB = case["N"], _kb(case["K"])
    K = 24 * KB
    if kind == "gptq":
        # weights and factor in, indices and gains out; the error of every block column goes into the columns after it
        return {"bytes": 4 * N * K + 2 * K * K + 8 * N * KB, "flops": sum(2 * N * 24 * (K - 24 * (t + 1)) + N * 24 * 24 for t in range(KB))}
    # group scales: W0 H, the symmetric KB x KB system of every row, its factorisation
    return {"bytes": 4 * (3 * N * K + K * K) + 8 * N * KB, "flops": 3 * N * K * K + N * KB ** 3 // 3}


def tolerance(case):
    kind = case["kind"]
    if kind == "encode" or (kind == "decode" and case["out"] == "int8"):
        return "exact"
    if kind in ("decode", "load"):
        return {"rel": {"f16": 2e-4, "bf16": 2e-3, "f32": 1e-6}[case["out"]]}           # one rounding to the output type
    if kind in ("matmul", "block"):
        if case["M"] <= 2 or case.get("m_max") == 19:
            return {"rel": 1e-5}                # exact products, fp32 sums
        return {"rel": 5e-4 if case["x"] == "f16" else 3e-5}      # weights enter with 11 (fp16) or 16 bits (bf16: two terms)
    if kind == "quantize":
        return {"rel": 1e-5, "differ": 1e-3}    # candidates that tie within fp32 rounding are interchangeable
    if kind == "gptq":
        # a tie within fp32 rounding that falls the other way changes the blocks to its right in that row
        return {"rel": 1e-2, "max": 0.6, "differ": 5e-3}
    return {"rel": 5e-4}                        # group scales: fp32 factorisation, gains rounded to fp16
