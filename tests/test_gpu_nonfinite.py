"""Infinite activations and adapters: an output is infinite, NaN or finite exactly where the sums of the fp64 CPU oracle
are.  One infinite entry of X makes infinities where the weights of its column are nonzero and NaN where they are zero (every
kernel multiplies the zeros of the mask); nothing that a tile, a half step or a padded rank adds may turn those into NaN.  The
finite outputs keep the usual bar, max |Y - Y_ref| <= 1e-2 * max |Y_ref|."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import dev, to_dev_u16, to_dev_u32, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2
INF, NINF = 0x7F80, 0xFF80


def _kinds(a):
    return np.isnan(a) * 3 + np.isposinf(a) + np.isneginf(a) * 2


def _compare(got, ref, label):
    assert np.array_equal(_kinds(got), _kinds(ref)), f"{label}: {int(np.sum(_kinds(got) != _kinds(ref)))} outputs of another kind"
    fin = np.isfinite(ref)
    if fin.any():   # (an infinite gradient entry reaches all of dA)
        assert float(np.max(np.abs(got[fin] - ref[fin]))) <= REL_TOL * float(np.max(np.abs(ref[fin]))), label


def _layer(M, K, N, R, seed):
    """Weight and adapters whose entries in the infinite columns (the last 32) are not negative, so that the infinities of a sum agree."""
    w = wl.gaussian_bf16((N, K), 0.02, seed + 1)
    w[np.random.default_rng(seed).random((N, K)) >= 0.5] = 0
    w[:, -32:] &= 0x7FFF
    a = wl.gaussian_bf16((K, R), 0.05, seed + 2) if R else None
    b = wl.gaussian_bf16((R, N), 0.05, seed + 3) & np.uint16(0x7FFF) if R else None
    if R:
        a[-32:] &= 0x7FFF
    x = wl.gaussian_bf16((M, K), 1.0, seed)
    x[3, K - 30], x[M - 1, K - 3] = INF, NINF
    return x, w, a, b


# contractions that end in half a step, with and without a split; rank dimensions that do (ranks up to 32, and 65 to 96); both
HALF_STEPS = [(130, 96, 300, 0), (300, 160, 65, 64), (150, 8224, 40, 0), (200, 128, 300, 8), (200, 192, 70, 96), (300, 160, 65, 8),
              (131, 2720, 267, 24), (1030, 96, 14400, 8), (1100, 544, 2050, 32)]


# ranks that do not fill the padded ones, on the paths that compute T with A_cat padded by zero rows: the product of its own (ranks
# that are no multiple of 8, long rows), and the transposing pass of the fused kernel above 1024 tokens (the least workspace)
PADDED_RANKS = [(200, 128, 300, 5), (200, 128, 300, 61), (1100, 128, 300, 61), (150, 8256, 40, 72), (1100, 1024, 300, 33), (4100, 512, 33, 7)]


@pytest.mark.parametrize("M,K,N,R", HALF_STEPS + PADDED_RANKS)
@pytest.mark.parametrize("least", [False, True])
def test_linear(M, K, N, R, least):
    import paper_2601_16991_amd as salr
    x, w, a, b = _layer(M, K, N, R, M + K + N + R)
    rb, rv, ro = oracle.encode(w)
    print(f"[non-finite] M{M} K{K} N{N} R{R} least workspace {least}", flush=True)
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    size = salr.salr_linear_workspace_bytes_min(M, K, N, R)
    args = (to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), *((to_dev_u16(a), to_dev_u16(b)) if R else (None, None)))
    if least:
        salr.salr_sparse_lowrank_linear(*args, y, torch.empty(size, dtype=torch.uint8, device=dev()) if size else None)
    else:
        y = salr.linear(*args)
    torch.cuda.synchronize()
    ref = oracle.linear(x, w, a, b)
    assert np.isinf(ref[3]).any() and np.isinf(ref[M - 1]).any()
    _compare(y_to_f64(y), ref, "y")


# T formed by every workgroup, by the first of them beside their own work, by workgroups of their own, in a launch in front (rank 12);
# row tiles with a split, in one launch of one, two and four parts, without adapters in parts; large batches and, under 2:4, both of their
# kernels (row tiles of two rank steps last).  On the told workspace long rows and 17 to 64 tokens have kernels of their own.  Ranks that do not fill the padded ones.
CALLS = [(5, 512, 300, 5), (16, 1152, 4096, 24), (3, 2048, 500, 40), (16, 2048, 500, 12), (4, 12416, 160, 5), (20, 2048, 600, 7), (40, 1120, 2100, 33),
         (100, 1120, 300, 5), (16, 4096, 6000, 24), (24, 1120, 8384, 8), (128, 576, 16640, 40), (16, 1024, 8320, 0), (200, 128, 300, 20),
         (1024, 128, 3072, 40), (1536, 128, 2048, 40), (72, 1152, 300, 40)]


def _places(kind, K, R):
    """Of a 2:4 weight the zeros are not multiplied: X stays finite there.  Its calls and those with a table want rows of whole chunks."""
    if kind in ("2of4", "prepared") and K % 128:
        return []
    return (["x"] if kind != "2of4" else []) + (["a", "b"] if R else [])


@pytest.mark.parametrize("kind,M,K,N,R,where", [(kind, M, K, N, R, where) for M, K, N, R in CALLS for kind in ("plain", "prepared", "codes", "2of4")
                                                for where in _places(kind, K, R)])
def test_every_path(kind, M, K, N, R, where):
    """An infinite entry of X, of A_cat, or of B_cat in its last rank, which those that fill the padded ones must not meet."""
    import paper_2601_16991_amd as salr
    w = wl.gaussian_bf16((N, K), 0.02, M + K)
    if kind == "2of4":
        w = oracle.mask_nm(w, 2, 4)
    else:
        w[np.random.default_rng(M + K).random((N, K)) >= 0.5] = 0
    x = wl.gaussian_bf16((M, K), 1.0, M + N)
    a, b = (wl.gaussian_bf16((K, R), 0.05, 1), wl.gaussian_bf16((R, N), 0.05, 2)) if R else (None, None)
    if where == "x":
        w[:, K - 20] &= 0x7FFF
        if R:
            a[K - 20] &= 0x7FFF
            b &= 0x7FFF
        x[M - 1, K - 20] = NINF
    elif where == "a":
        a[K // 2, R - 1] = INF
    else:
        b[R - 1, N - 1], b[R - 1, N // 2] = INF, NINF
    rb, rv, ro = oracle.encode(w)
    args = [to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro)]
    ab = [to_dev_u16(a), to_dev_u16(b)] if R else [None, None]
    print(f"[non-finite] {kind} M{M} K{K} N{N} R{R}: {where}", flush=True)
    if kind == "codes":
        codes, scales = salr.nf4_quantize(args[2])
        w = oracle.decode(rb, salr.nf4_dequantize(codes, scales, rv.size).cpu().numpy().view(np.uint16)[:rv.size], ro, N, K)
        ys = [salr.qsalr_linear(args[0], args[1], codes, scales, args[3], rv.size, *ab)]
    elif kind == "prepared":
        ys = [salr.linear_prepared(*args, salr.build_slice_table(args[1], args[3], K), *ab)]
    else:
        ys = [(salr.linear if kind == "plain" else salr.linear_2of4)(*args, *ab)]
    if kind == "plain":
        told = salr.salr_linear_workspace_bytes(M, K, N, R)
        ys.append(torch.empty_like(ys[0]))
        salr.salr_sparse_lowrank_linear(*args, *ab, ys[1], torch.empty(told, dtype=torch.uint8, device=dev()) if told else None)
    torch.cuda.synchronize()
    ref = oracle.linear(x, w, a, b)
    assert not np.isfinite(ref).all()
    for y in ys:
        _compare(y_to_f64(y), ref, "y")


def test_quantised():
    import paper_2601_16991_amd as salr
    M, K, N, R = 129, 96, 40, 8
    x, w, a, b = _layer(M, K, N, R, 7)
    rb, rv, ro = oracle.encode(w)
    codes, scales = salr.nf4_quantize(to_dev_u16(rv))
    q = salr.nf4_dequantize(codes, scales, rv.size)
    print(f"[non-finite] quantised M{M} K{K} N{N} R{R}", flush=True)
    y = salr.qsalr_linear(to_dev_u16(x), to_dev_u32(rb), codes, scales, to_dev_u32(ro), rv.size, to_dev_u16(a), to_dev_u16(b))
    torch.cuda.synchronize()
    _compare(y_to_f64(y), oracle.linear(x, oracle.decode(rb, q.cpu().numpy().view(np.uint16), ro, N, K), a, b), "y")


@pytest.mark.parametrize("M,K,N,R", [(160, 256, 128, 8), (192, 288, 192, 96)])
def test_backward(M, K, N, R):
    """dX contracts over N (whole steps) and the ranks (half a step here)."""
    import paper_2601_16991_amd as salr
    x, w, a, b = _layer(M, K, N, R, M + K)
    x = wl.gaussian_bf16((M, K), 1.0, 11)
    a &= 0x7FFF
    w &= 0x7FFF
    dy = wl.gaussian_bf16((M, N), 1.0, 12)
    dy[5, N - 7] = INF
    rb, rv, ro = oracle.encode(w)
    print(f"[non-finite] backward M{M} K{K} N{N} R{R}", flush=True)
    got = salr.linear_backward(to_dev_u16(x), to_dev_u16(dy), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), to_dev_u16(a), to_dev_u16(b))
    torch.cuda.synchronize()
    for name, g, ref in zip(("dx", "da", "db"), got, oracle.linear_backward(x, dy, w, a, b)):
        _compare(y_to_f64(g), ref, name)
