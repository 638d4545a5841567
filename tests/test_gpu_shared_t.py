"""Decoding calls of the small-batch kernels whose first workgroups form T = X A_cat for all of them: against the fp64 oracle
(max |Y - Y_ref| <= 1e-2 * max |Y_ref|), and bit for bit where only who forms T and when is another."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import dev, to_dev_u16, to_dev_u32, to_host_u16, to_host_u32, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2

# As many row groups as T has slices and one row more; 2, 3 and 4 chunks a wave, fewer chunks than waves, uneven slices, rows of more than 32
# chunks (with a table: 64); tokens and ranks at the edges of the tiles of 16, 8 and 128 ranks, 4 pairs of rank tiles
SHAPES = [(1, 4096, 4096, 32, 0.5), (16, 4096, 4096, 32, 0.5), (16, 4096, 256, 32, 0.5), (5, 4096, 241, 8, 0.5), (16, 1152, 1024, 128, 0.5),
          (7, 128, 512, 40, 0.5), (9, 2048, 1040, 64, 0.3), (16, 2176, 800, 72, 0.5), (15, 3072, 8176, 16, 0.5), (16, 4224, 2000, 96, 0.5),
          (3, 4224, 1025, 128, 0.5), (16, 3968, 2500, 64, 0.9), (2, 1280, 530, 24, 1.0), (16, 8192, 512, 48, 0.5)]


def _layer(M, K, N, R, density):
    rng = np.random.default_rng(M + K + N)
    x = wl.gaussian_bf16((M, K), 1.0, M + K + N)
    w = wl.gaussian_bf16((N, K), 0.02, M + K + N + 1)
    w[rng.random((N, K)) >= density] = 0
    a, b = wl.gaussian_bf16((K, R), 0.05, 2), wl.gaussian_bf16((R, N), 0.05, 3)
    rb, rv, ro = oracle.encode(w)
    return [to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), to_dev_u16(a), to_dev_u16(b)], oracle.linear(x, w, a, b), rv.size


def _call(kind, args, M, K, N, R, extra, fill=0x5A):
    """One call on exactly the told workspace, whose bytes hold `fill` before."""
    import paper_2601_16991_amd as salr
    need = (salr.salr_qsalr_linear_workspace_bytes(M, K, N, R, extra[2]) if kind == "codes" else salr.salr_linear_workspace_bytes(M, K, N, R))
    buf = torch.full((need + 4096,), fill, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    x, bitmap, values, offsets, a, b = args
    if kind == "plain":
        salr.salr_sparse_lowrank_linear(x, bitmap, values, offsets, a, b, y, buf[:need])
    elif kind == "prepared":
        salr.salr_sparse_lowrank_linear_prepared(x, bitmap, values, offsets, extra, a, b, y, buf[:need])
    else:
        salr.salr_qsalr_linear(x, bitmap, extra[0], extra[1], offsets, extra[2], a, b, y, buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == fill).all())
    return y


def _kind(kind, args, K, N, nnz, ref):
    """What a kind of call takes beside the layer, and what it should give."""
    import paper_2601_16991_amd as salr
    if kind == "plain":
        return None, ref
    if kind == "prepared":
        return salr.build_slice_table(args[1], args[3], K), ref
    codes, scales = salr.nf4_quantize(args[2])
    w = oracle.decode(to_host_u32(args[1]), to_host_u16(salr.nf4_dequantize(codes, scales, nnz))[:nnz], to_host_u32(args[3]), N, K)
    return (codes, scales, nnz), oracle.linear(to_host_u16(args[0]), w, to_host_u16(args[4]), to_host_u16(args[5]))


@pytest.mark.parametrize("kind", ["plain", "prepared", "codes"])
@pytest.mark.parametrize("M,K,N,R,density", SHAPES)
def test_close_to_the_oracle_whoever_forms_t(kind, M, K, N, R, density):
    import paper_2601_16991_amd as salr
    args, ref, nnz = _layer(M, K, N, R, density)
    extra, ref = _kind(kind, args, K, N, nnz, ref)
    print(f"[shared t] {kind} M{M} K{K} N{N} R{R}", flush=True)
    y = _call(kind, args, M, K, N, R, extra)
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    assert torch.equal(_call(kind, args, M, K, N, R, extra, 0xFF), y)   # what the workspace held before is of no account
    # A_cat that starts inside a vector: a launch in front
    off = torch.empty(K * R + 1, dtype=args[4].dtype, device=dev())[1:].view(K, R).copy_(args[4])
    assert torch.equal(_call(kind, [*args[:4], off, args[5]], M, K, N, R, extra), y)
    salr.lib().salr_set_handover_polls(0)   # workgroups that do not find T at once form it themselves
    try:
        for _ in range(3):
            assert torch.equal(_call(kind, args, M, K, N, R, extra), y)
    finally:
        salr.lib().salr_set_handover_polls(-1)


@pytest.mark.parametrize("polls", [-1, 0])
@pytest.mark.parametrize("M,K,N,R", [(16, 1152, 1024, 128), (1, 4096, 4096, 32)])
def test_graph_replays_with_new_inputs(M, K, N, R, polls):
    """A captured call has the same tag on every replay: the words are clear again after each, whoever came last."""
    import paper_2601_16991_amd as salr
    args, _, _ = _layer(M, K, N, R, 0.5)
    ws = torch.full((salr.salr_linear_workspace_bytes(M, K, N, R),), 0x5A, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    other = torch.empty_like(y)
    x = args[0].clone()
    salr.salr_sparse_lowrank_linear(x, *args[1:], other, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    salr.lib().salr_set_handover_polls(polls)
    try:
        with torch.cuda.graph(graph):
            salr.salr_sparse_lowrank_linear(x, *args[1:], y, ws)
    finally:
        salr.lib().salr_set_handover_polls(-1)
    for turn in range(6):
        print(f"[shared t] M{M} K{K} N{N} R{R}: replay {turn}", flush=True)
        x.copy_(to_dev_u16(wl.gaussian_bf16((M, K), 1.0 + turn, turn)))
        y.zero_()
        graph.replay()
        if turn % 2:
            torch.cuda.synchronize()
            salr.salr_sparse_lowrank_linear(args[0], *args[1:], other, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, salr.linear(x, *args[1:]))
