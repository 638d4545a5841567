"""The work that users of the SALR layer have it do, as cases that can be timed and compared.

A case is one of six kinds of pass through the public entry points:

    linear     ``linear``             the layer on a plain bitmap weight: token-by-token decoding, batches, prompts
    prepared   ``linear_prepared``    the same with the layer's slice table kept beside the weight (serving)
    2of4       ``linear_2of4``        the layer under a 2:4 mask
    qsalr      ``qsalr_linear``       the layer on 4-bit values
    backward   ``linear_backward``    a fine-tuning step's gradients: dX, dA, dB
    codec      ``mask_rows``, ``encode``, ``decode``   pruning a weight, packing it, and unpacking it again

``layers`` is how many layers of that shape one pass goes through, each with its own weight, as the decoder blocks of a
model do: at decode sizes a weight then comes from memory and not from a cache that the previous pass has filled.
Weights ~ N(0, 0.02) pruned by magnitude per row, activations and output gradients ~ N(0, 1), adapters ~ N(0, 0.01).
"""
from __future__ import annotations

import math

import torch

import paper_2601_16991_amd as salr


def _case(name, kind, layers, M, K, N, R, permille):
    return {"name": name, "kind": kind, "layers": layers, "M": M, "K": K, "N": N, "R": R, "permille": permille}


def listed():
    return [
        # the smallest layer of the workload list: what is left is the call itself
        _case("tiny_M16", "linear", 1, 16, 512, 512, 16, 500),
        # one token through the attention projections of an 8B model, served with slice tables
        _case("attn_decode_M1", "prepared", 8, 1, 4096, 4096, 32, 500),
        # a decoding batch through the up projections of an 8B model
        _case("up_decode_M16", "linear", 4, 16, 4096, 14336, 32, 500),
        # a small decoding batch through its down projections (long rows) at the higher sparsity
        _case("down_decode_M8_p70", "linear", 4, 8, 14336, 4096, 64, 700),
        # 4-bit values at the sparsity they are used with
        _case("qsalr_attn_decode_M16", "qsalr", 8, 16, 4096, 4096, 32, 200),
        # continuous batching: more tokens than a decode kernel is made for, fewer than a prompt
        _case("up_batch_M64", "linear", 4, 64, 4096, 14336, 32, 500),
        # nothing a multiple of anything: a short prompt on a layer of uneven sizes
        _case("ragged_M300", "linear", 1, 300, 2720, 2731, 24, 500),
        # prompts: the 8B up projection, plain and under the 2:4 mask, and the largest 70B layer
        _case("up_prefill_M2048", "linear", 1, 2048, 4096, 14336, 32, 500),
        _case("2of4_up_prefill_M2048", "2of4", 1, 2048, 4096, 14336, 32, 500),
        _case("down70b_prefill_M4096", "linear", 1, 4096, 28672, 8192, 64, 500),
        # a fine-tuning step of an attention projection
        _case("attn_backward_M2048", "backward", 1, 2048, 4096, 4096, 32, 500),
        # pruning and packing a layer when a model is converted, and checking the packed form
        _case("codec_down", "codec", 1, 0, 14336, 4096, 0, 500),
    ]


# The sizes the listed cases stand for: layers from 512 to 28672 wide and up to the 70B down projection's element count,
# 1 to 4096 tokens (128 and up in training steps), adapter ranks 0 to 128.
_DIM = (512, 28672)
_WEIGHT = 8192 * 28672
_TOKENS = (1, 4096)
_LAYER_BYTES = 96 << 20   # layers of a decode-sized pass: enough for about this much weight, at most eight


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear"] * 5 + ["prepared", "2of4", "qsalr", "backward", "codec"])
    while True:
        # contraction: mostly whole 128-column chunks, as the widths of models are, else any multiple of 32
        step = rng.choice([128, 128, 128, 128, 64, 32])
        K = max(512, _log_uniform(rng, *_DIM) // step * step)
        N = _log_uniform(rng, *_DIM)
        if rng.random() < 0.5:
            N = N // 128 * 128
        if kind == "backward":
            N = N // 64 * 64
        if kind == "prepared":
            M = _log_uniform(rng, 1, 128)
        elif kind == "backward":
            M = _log_uniform(rng, 128, 4096) // 32 * 32
        elif kind == "codec":
            M = 0
        else:
            M = _log_uniform(rng, *_TOKENS)
        # the gradients, the unpruned copies and sizes without a large-batch kernel of their own cost several times a
        # plain call
        most = _WEIGHT * 4096 // (16 if kind in ("backward", "codec") or K % 64 else 4)
        if N * K <= _WEIGHT // (4 if kind in ("backward", "codec") else 1) and M * N * K <= most:
            break
    R = 0 if kind == "codec" else rng.choice([0, 16, 32, 32, 64, 64, 128, rng.randint(3, 96)])
    if kind == "backward":
        R = max(R, 8)
    permille = 500 if kind == "2of4" else rng.choice([200, 200, 500]) if kind == "qsalr" else rng.choice([500, 500, 700, 300])
    layers = 1
    if 0 < M <= 128 and kind != "backward":
        layers = max(1, min(8, _LAYER_BYTES // max(1, N * K)))
    return {"kind": kind, "layers": layers, "M": M, "K": K, "N": N, "R": R, "permille": permille}


def _keep(case):
    return case["K"] - case["K"] * case["permille"] // 1000


def _normal(shape, std, gen):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, M, K, N, R = case["kind"], case["M"], case["K"], case["N"], case["R"]
    if kind == "codec":
        return {"kind": kind, "w": _normal((N, K), 0.02, gen), "keep": _keep(case)}
    layers = []
    for _ in range(case["layers"]):
        w = _normal((N, K), 0.02, gen)
        w_hat = salr.mask_nm(w, 2, 4) if kind == "2of4" else salr.mask_rows(w, _keep(case))
        del w
        bitmap, values, offsets = salr.encode(w_hat)
        del w_hat
        layer = {"x": _normal((M, K), 1.0, gen), "bitmap": bitmap, "values": values, "offsets": offsets,
                 "a": _normal((K, R), 0.01, gen) if R else None, "b": _normal((R, N), 0.01, gen) if R else None}
        if kind == "prepared":
            layer["table"] = salr.build_slice_table(bitmap, offsets, K)
        elif kind == "qsalr":
            layer["nnz"] = values.numel()
            layer["codes"], layer["scales"] = salr.nf4_quantize(values)
            del layer["values"]
        elif kind == "backward":
            layer["dy"] = _normal((M, N), 1.0, gen)
        layers.append(layer)
    # one workspace for all layers of the model, as their calls follow one another on a stream
    need = (salr.salr_linear_2of4_workspace_bytes(M, K, N, R) if kind == "2of4" else
            salr.salr_linear_workspace_bytes(M, K, N, R) if kind in ("linear", "prepared") else 0)
    return {"kind": kind, "layers": layers,
            "workspace": torch.empty(need, dtype=torch.uint8, device="cuda") if need else None}


def run(state):
    kind = state["kind"]
    if kind == "codec":
        w = state["w"]
        w_hat = salr.mask_rows(w, state["keep"])
        bitmap, values, offsets = salr.encode(w_hat)
        return w_hat, bitmap, values, offsets, salr.decode(bitmap, values, offsets, w.shape[0], w.shape[1])
    ws = state["workspace"]
    if kind == "linear":
        return [salr.linear(l["x"], l["bitmap"], l["values"], l["offsets"], l["a"], l["b"], ws) for l in state["layers"]]
    if kind == "prepared":
        return [salr.linear_prepared(l["x"], l["bitmap"], l["values"], l["offsets"], l["table"], l["a"], l["b"], ws)
                for l in state["layers"]]
    if kind == "2of4":
        return [salr.linear_2of4(l["x"], l["bitmap"], l["values"], l["offsets"], l["a"], l["b"], ws) for l in state["layers"]]
    if kind == "qsalr":
        return [salr.qsalr_linear(l["x"], l["bitmap"], l["codes"], l["scales"], l["offsets"], l["nnz"], l["a"], l["b"])
                for l in state["layers"]]
    return [salr.linear_backward(l["x"], l["dy"], l["bitmap"], l["values"], l["offsets"], l["a"], l["b"])
            for l in state["layers"]]


def work(case):
    """Each operand once in, each result once out; products as the matrix cores do them: the zeros of an unstructured mask
    are multiplied, those of a 2:4 mask are not."""
    kind, L, M, K, N, R = case["kind"], case.get("layers", 1), case["M"], case["K"], case["N"], case["R"]
    nnz = N * _keep(case)
    index = N * K // 8 + 4 * (N + 1)
    if kind == "codec":   # the weight in; the pruned weight, its packed form and the unpacked weight out
        return {"bytes": 6 * N * K + index + 2 * nnz, "flops": 0}
    weight = index + (nnz // 2 + nnz // 32 if kind == "qsalr" else 2 * nnz)
    adapters = 2 * R * (K + N)
    if kind == "backward":
        return {"bytes": L * (weight + 2 * adapters + 2 * M * (2 * K + N)), "flops": L * (2 * M * N * K + 4 * M * R * (K + N) + 2 * M * R * K)}
    base = 2 * M * N * K // (2 if kind == "2of4" else 1)
    return {"bytes": L * (weight + adapters + 2 * M * (K + N)), "flops": L * (base + 2 * M * R * (K + N))}


def tolerance(case):
    """The codec moves bits.  The layer rounds its results to bf16 (2^-9 of a value) and, once, the low-rank intermediate
    before them, so two correct sums in fp32 differ by a rounding here and there."""
    return "exact" if case["kind"] == "codec" else {"rel": 5e-3, "max": 0.04}
