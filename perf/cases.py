"""The calls that a user of this framework makes, at the sizes at which they are made.

Five kinds of work:

  linear     one `torq_linear` call: rotate and quantise the activations, then multiply with packed weights
  block      the linear layers of whole decoder blocks, one `torq_linear` call each: a decode step or a short chunk
  rotate     rotate and quantise alone (MXFP4, MXINT4 or NVFP4; dense or butterfly inter-block rotation): the
             offline preparation of weights, and activations for another consumer
  gram       calibration of the inter-block rotation, the block Gram matrix (whole, or one for each position)
  histogram  calibration of the intra-block rotation, the codeword histogram of packed codes

Activations are Student-t with outlier channels, weights Gaussian and rotated and quantised beforehand, as
`paper_2605_19561_amd/synth.py` draws them for the tests and the benchmark.
"""
import math

import torch

from paper_2605_19561_amd import binding as tq
from paper_2605_19561_amd import synth

DEVICE = "cuda:0"
FORMATS = {"mxfp4": tq.TORQ_FMT_MXFP4, "mxint4": tq.TORQ_FMT_MXINT4, "nvfp4": tq.TORQ_FMT_NVFP4}
MOST_FLOPS = 2.0 * 8192 * 28672 * 8192  # the largest listed product
MOST_ELEMENTS = 28672 * 8192            # the largest listed input of a streaming kernel


def listed():
    return [
        # one token through one square projection (LLaMA3-8B q or o): the smallest call, nothing kept but the weights
        {"name": "linear_1_row", "kind": "linear", "M": 1, "d": 4096, "N": 4096},
        # a decode step of one sequence through two LLaMA3-8B decoder blocks, buffers kept by the program
        {"name": "block_decode_1", "kind": "block", "M": 1, "blocks": 2, "hidden": 4096, "q": 4096, "kv": 1024, "ffn": 14336},
        # a decode step of sixteen sequences through a LLaMA3-70B block (454 MB of packed weights)
        {"name": "block_decode_16", "kind": "block", "M": 16, "blocks": 1, "hidden": 8192, "q": 8192, "kv": 1024, "ffn": 28672},
        # a decode step of a batch that is not a power of two through a Qwen3-32B block (G = 80 and 128)
        {"name": "block_decode_45", "kind": "block", "M": 45, "blocks": 1, "hidden": 5120, "q": 8192, "kv": 1024, "ffn": 25600},
        # a prefill chunk of ragged length through a LLaMA3-8B down projection (G = 112, long reduction)
        {"name": "linear_chunk_333", "kind": "linear", "M": 333, "d": 14336, "N": 4096},
        # prefill of 2048 tokens, LLaMA3-8B gate or up projection
        {"name": "linear_prefill_8b", "kind": "linear", "M": 2048, "d": 4096, "N": 14336},
        # prefill of 8192 tokens, LLaMA3-70B gate or up projection: the benchmark's step
        {"name": "linear_prefill_70b", "kind": "linear", "M": 8192, "d": 8192, "N": 28672},
        # offline preparation of that layer's weights
        {"name": "rotate_weights", "kind": "rotate", "M": 28672, "d": 8192, "format": "mxfp4", "butterfly": 0},
        # activations to NVFP4 through a calibrated butterfly
        {"name": "rotate_nvfp4_butterfly", "kind": "rotate", "M": 4096, "d": 8192, "format": "nvfp4", "butterfly": 128},
        # calibration: second moments of the blocks over 16384 tokens
        {"name": "gram", "kind": "gram", "M": 16384, "d": 8192, "positions": False},
        # calibration: the same kept apart by the position inside a block, over 4096 tokens
        {"name": "gram_positions", "kind": "gram", "M": 4096, "d": 4096, "positions": True},
        # calibration: codeword occupancy of the packed activations of the benchmark's step
        {"name": "histogram", "kind": "histogram", "M": 8192, "d": 8192},
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "block", "rotate", "rotate", "gram", "histogram"])
    d = 1024 * _log(rng, 1, 28)
    if kind == "linear":
        M, N = _log(rng, 1, 8192), _log(rng, 256, 28672)
        if rng.random() < 0.7:
            N = max(256, N // 128 * 128)  # layer widths are round numbers more often than not
        while 2.0 * M * N * d > MOST_FLOPS:
            M //= 2
        return {"kind": kind, "M": M, "d": d, "N": N}
    if kind == "block":
        hidden = 1024 * rng.randint(2, 8)
        return {"kind": kind, "M": _log(rng, 1, 300), "blocks": 1, "hidden": hidden, "q": 1024 * rng.randint(2, 8),
                "kv": rng.choice([512, 1024, 2048]), "ffn": 1024 * rng.randint(5, 28)}
    M = max(1, min(_log(rng, 64, 32768), MOST_ELEMENTS // d))
    if kind == "rotate":
        butterfly = rng.choice([0, 0, 32, 64, 128, 256])
        if butterfly and (d // 32) % butterfly:
            butterfly = 32
        return {"kind": kind, "M": M, "d": d, "format": rng.choice(sorted(FORMATS)), "butterfly": butterfly}
    if kind == "gram":
        positions = rng.random() < 0.4
        return {"kind": kind, "M": max(1, M // 4) if positions else M, "d": d, "positions": positions}
    return {"kind": kind, "M": M, "d": d}


def _activations(M, d, seed):
    return synth.activations(M, d, outliers=max(1, d // 200), seed=seed, device=DEVICE)


def _rotation(d, seed):
    G = synth.default_G(d)
    return tq.Rotation(d, G, *synth.rotations(G, seed))


def _weights(rot, N, d, seed):
    return tq.torq_rotate_quantize(rot, synth.weights(N, d, seed=seed, device=DEVICE))


def _layers(case):
    """(input width, output width) of the seven linear layers of each block: q, k, v, o, gate, up, down."""
    h, q, kv, ffn = case["hidden"], case["q"], case["kv"], case["ffn"]
    return [(h, q), (h, kv), (h, kv), (q, h), (h, ffn), (h, ffn), (ffn, h)] * case["blocks"]


def _prepare_block(case, seed):
    M, rots, xs, layers, need = case["M"], {}, {}, [], 16
    for i, (d, N) in enumerate(_layers(case)):
        if d not in rots:
            rots[d] = _rotation(d, seed + 100 + d)
            xs[d] = _activations(M, d, seed + 200 + d)
        wq, ws = _weights(rots[d], N, d, seed + 300 + i)
        layers.append((rots[d], xs[d], wq, ws, torch.empty((M, N), dtype=torch.bfloat16, device=DEVICE)))
        need = max(need, tq.torq_linear_workspace_bytes_n(M, N, d))
    return {"layers": layers, "workspace": torch.empty(need, dtype=torch.uint8, device=DEVICE)}


def prepare(case, seed):
    seed = 1000 * int(seed)
    kind = case["kind"]
    state = {"kind": kind}
    if kind == "block":
        state.update(_prepare_block(case, seed))
        return state
    M, d = case["M"], case["d"]
    if kind == "rotate" and not case["butterfly"] and M > 16384:
        x = synth.weights(M, d, seed=seed + 1, device=DEVICE)
    else:
        x = _activations(M, d, seed + 1)
    if kind == "linear":
        rot = _rotation(d, seed + 2)
        state.update(rot=rot, x=x, weights=_weights(rot, case["N"], d, seed + 3))
    elif kind == "rotate":
        G = case["butterfly"]
        if G:
            sigma = tq.torq_block_gram(x[: min(M, 1024)], G).cpu().numpy()
            rot = tq.ButterflyRotation(d, G, tq.torq_equalize_inter_butterfly(sigma)[1], synth.rotations(32, seed + 2)[1])
        else:
            rot = _rotation(d, seed + 2)
        # NVFP4's tensor-wide scale: the largest magnitude lands on the largest scale times the largest codeword
        state.update(rot=rot, x=x, format=FORMATS[case["format"]], global_scale=float(x.abs().max()) / (6 * 448))
    elif kind == "gram":
        state.update(x=x, G=synth.default_G(d), positions=case["positions"])
    else:
        state.update(d=d, codes=tq.torq_rotate_quantize(_rotation(d, seed + 2), x)[0])
    return state


def run(state):
    kind = state["kind"]
    if kind == "linear":
        return tq.torq_linear(state["rot"], state["x"], *state["weights"])
    if kind == "block":
        workspace = state["workspace"]
        return [tq.torq_linear(rot, x, wq, ws, out=out, workspace=workspace) for rot, x, wq, ws, out in state["layers"]]
    if kind == "rotate":
        if state["format"] == tq.TORQ_FMT_MXFP4:
            return tq.torq_rotate_quantize(state["rot"], state["x"])
        return tq.torq_rotate_quantize_fmt(state["rot"], state["x"], state["format"], state["global_scale"])
    if kind == "gram":
        return (tq.torq_block_gram_positions if state["positions"] else tq.torq_block_gram)(state["x"], state["G"])
    return tq.torq_code_histogram(state["codes"], state["d"])


def _linear_work(M, d, N):
    return M * d * 2 + N * d * 17 / 32 + M * N * 2, 2.0 * M * N * d + 2.0 * M * d * (synth.default_G(d) + 32)


def work(case):
    kind, M = case["kind"], case["M"]
    if kind == "block":
        each = [_linear_work(M, d, N) for d, N in _layers(case)]
        # the layers that share an input read it once
        shared = M * 2 * (case["blocks"] * (4 * case["hidden"]))
        return {"bytes": sum(b for b, _ in each) - shared, "flops": sum(f for _, f in each)}
    d = case["d"]
    if kind == "linear":
        b, f = _linear_work(M, d, case["N"])
        return {"bytes": b, "flops": f}
    if kind == "rotate":
        scales = d / 16 if case["format"] == "nvfp4" else d / 32
        inter = math.log2(case["butterfly"]) + 1 if case["butterfly"] else synth.default_G(d)
        return {"bytes": M * (d * 2.5 + scales), "flops": 2.0 * M * d * (inter + 32)}
    G = synth.default_G(d)
    if kind == "gram":
        # symmetric: half of the products
        return {"bytes": M * d * 2 + (32 if case["positions"] else 1) * G * G * 8, "flops": 1.0 * M * d * G}
    return {"bytes": M * d / 2 + 32 * 8 * 8, "flops": 1.0 * M * d}


def tolerance(case):
    """Four times what the path differs by from its own rotation and sums in 64 bits on the same inputs.  Rotated values
    at a rounding boundary fall to either side: up to 8e-5 of the packed bytes, or a block or two of a small input; one
    such code among the 4096 of a single row moves its products by 5e-3."""
    kind, M = case["kind"], case["M"]
    if kind == "histogram":
        return "exact"
    if kind == "gram":
        return {"rel": 1e-6, "max": 5e-6}
    if kind == "rotate":
        return {"differ": min(1e-2, 3e-4 + 4 / (M * case["d"] / 32))}
    return {"rel": 1.5e-2 if M < 16 else 6e-3, "max": 0.2}
