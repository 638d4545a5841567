"""Row-tiled calls whose only slice adds the adapters in the launch that forms T (32, 64 or 128 rows a workgroup, four, two or one parts of
K): against the fp64 oracle (max |Y - Y_ref| <= 1e-2 * max |Y_ref|), and bit for bit where only the order in which T and the rows come
is another."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import dev, to_dev_u16, to_dev_u32, to_host_u16, to_host_u32, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2

# 130 tiles of 32, 64 and 128 rows and one row less or more; 4, 5 and 9 chunks a part, rows that end in 32, 64 and 96 columns of one;
# tokens at the edges of the tiles of sixteen and of the kernel's variants; ranks 1 to 256, and none
SHAPES = [(1, 2048, 4160, 32), (16, 2080, 4160, 1), (17, 4608, 4161, 33), (32, 2144, 4224, 0), (16, 2112, 4190, 16),
          (1, 1024, 8320, 32), (16, 1056, 8321, 128), (24, 1120, 8384, 8), (33, 1024, 8320, 16), (64, 2304, 8383, 64), (65, 1088, 8320, 32),
          (100, 1120, 8322, 40), (16, 1024, 8320, 0), (128, 1024, 8448, 0),
          (1, 512, 16640, 32), (16, 544, 16513, 200), (32, 608, 16640, 5), (64, 1152, 16770, 256), (128, 576, 16640, 16), (112, 512, 16640, 256)]


def _layer(M, K, N, R):
    rng = np.random.default_rng(M + K + N)
    x = wl.gaussian_bf16((M, K), 1.0, M + K + N)
    w = wl.gaussian_bf16((N, K), 0.02, M + K + N + 1)
    w[rng.random((N, K)) >= 0.5] = 0
    a, b = (wl.gaussian_bf16((K, R), 0.05, 2), wl.gaussian_bf16((R, N), 0.05, 3)) if R else (None, None)
    rb, rv, ro = oracle.encode(w)
    args = [to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), None if a is None else to_dev_u16(a), None if b is None else to_dev_u16(b)]
    return args, oracle.linear(x, w, a, b), rv.size


def _call(args, M, N, room, fill=0x5A):
    import paper_2601_16991_amd as salr
    buf = torch.full((room + 4096,), fill, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    salr.salr_sparse_lowrank_linear(*args, y, buf[:room] if room else None)
    torch.cuda.synchronize()
    assert bool((buf[room:] == fill).all())
    return y




@pytest.mark.parametrize("M,K,N,R", SHAPES)
def test_close_to_the_oracle_whatever_adds_the_adapters(M, K, N, R):
    import paper_2601_16991_amd as salr
    args, ref, _ = _layer(M, K, N, R)
    size = salr.salr_linear_workspace_bytes_fastest(M, K, N, R)
    print(f"[one launch] M{M} K{K} N{N} R{R}: {size} bytes", flush=True)
    y = _call(args, M, N, size)
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    assert torch.equal(_call(args, M, N, size, 0xFF), y)       # what the workspace held before is of no account
    assert torch.equal(_call(args, M, N, size + 65536), y)     # nor what it has beyond


@pytest.mark.parametrize("M,K,N,R", [s for s in SHAPES if s[3]])
def test_no_wait_for_the_low_rank_product(M, K, N, R):
    """Waves that do not find T at the end leave their sums to it: with no wait at all, and T long (112 x 512 x 16640 at rank 256), that is
    what most of them do.  Same bits."""
    import paper_2601_16991_amd as salr
    args, _, _ = _layer(M, K, N, R)
    size = salr.salr_linear_workspace_bytes_fastest(M, K, N, R)
    print(f"[one launch] M{M} K{K} N{N} R{R}: no wait", flush=True)
    y = _call(args, M, N, size)
    salr.lib().salr_set_handover_polls(0)
    try:
        for _ in range(3):
            assert torch.equal(_call(args, M, N, size), y)
    finally:
        salr.lib().salr_set_handover_polls(-1)


@pytest.mark.parametrize("M,K,N,R", [(16, 1056, 8321, 128), (64, 2304, 8383, 64), (1, 2048, 4160, 32), (64, 1152, 16770, 256)])
def test_four_bit_values(M, K, N, R):
    import paper_2601_16991_amd as salr
    args, _, nnz = _layer(M, K, N, R)
    codes, scales = salr.nf4_quantize(args[2])
    w = oracle.decode(to_host_u32(args[1]), to_host_u16(salr.nf4_dequantize(codes, scales, nnz))[:nnz], to_host_u32(args[3]), N, K)
    ref = oracle.linear(to_host_u16(args[0]), w, to_host_u16(args[4]), to_host_u16(args[5]))
    print(f"[one launch] quantised M{M} K{K} N{N} R{R}", flush=True)
    y = salr.qsalr_linear(args[0], args[1], codes, scales, args[3], nnz, args[4], args[5])
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))


@pytest.mark.parametrize("M,K,N,R", [(16, 1024, 8320, 32), (1, 2048, 4160, 32), (64, 512, 16640, 64)])
def test_graph_replays_with_new_inputs(M, K, N, R):
    """A captured call has the same tag on every replay: the words are clear again after each, eager calls on the same workspace between."""
    import paper_2601_16991_amd as salr
    args, _, _ = _layer(M, K, N, R)
    size = salr.salr_linear_workspace_bytes_fastest(M, K, N, R)
    ws = torch.full((size,), 0x5A, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    other = torch.empty_like(y)
    x = args[0].clone()
    salr.salr_sparse_lowrank_linear(x, *args[1:], other, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        salr.salr_sparse_lowrank_linear(x, *args[1:], y, ws)
    for turn in range(6):
        print(f"[one launch] M{M} K{K} N{N} R{R}: replay {turn}", flush=True)
        x.copy_(to_dev_u16(wl.gaussian_bf16((M, K), 1.0 + turn, turn)))
        y.zero_()
        graph.replay()
        if turn % 2:
            torch.cuda.synchronize()
            salr.salr_sparse_lowrank_linear(args[0], *args[1:], other, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, salr.linear(x, *args[1:]))
