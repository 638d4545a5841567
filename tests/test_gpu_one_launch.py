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

# M, K, N, R and the parts of K in a workgroup: calls that hand T over inside the launch (tests/test_routes.py holds them to it).  130 tiles of 32, 64
# and 128 rows and more; 4 to 32 chunks a part, rows that end in 32, 64 and 96 columns of one; tokens at the edges of the tiles of sixteen and of
# the kernel's variants; ranks 1 to 256, T in one, two and four slices
HANDED = [(16, 4096, 6000, 32, 4), (1, 3040, 6400, 5, 4), (9, 3104, 7168, 256, 4), (17, 1952, 4129, 1, 4), (32, 2048, 4159, 72, 4),
          (16, 1024, 8320, 32, 2), (9, 2048, 8289, 200, 2), (8, 2016, 11937, 96, 2), (24, 1120, 8384, 8, 2), (32, 928, 8384, 96, 2),
          (33, 1024, 8320, 16, 2), (64, 2048, 8289, 64, 2), (33, 1952, 9000, 250, 2), (65, 928, 8289, 8, 2), (100, 1120, 8322, 40, 2),
          (1, 512, 16640, 32, 1), (16, 416, 16609, 5, 1), (32, 608, 16640, 5, 1), (33, 640, 16609, 128, 1), (65, 512, 16639, 72, 1),
          (112, 544, 17000, 160, 1), (128, 576, 16640, 16, 1)]
# on 4-bit values, up to 16 tokens from 18 M entries on
HANDED_CODES = [c for c in HANDED if c[:3] not in ((16, 1024, 8320), (9, 2048, 8289))]
# no adapters, K in parts
PARTS = [(32, 2144, 4224, 0, 4), (16, 1024, 8320, 0, 2), (128, 1024, 8448, 0, 2)]
# beside them: what such sizes take with an N, a K or a rank that keeps them from it
OTHERS = [(1, 2048, 4160, 32), (16, 2080, 4160, 1), (17, 4608, 4161, 33), (16, 2112, 4190, 16), (1, 1024, 8320, 32), (16, 1056, 8321, 128),
          (64, 2304, 8383, 64), (65, 1088, 8320, 32), (16, 544, 16513, 200), (64, 1152, 16770, 256), (112, 512, 16640, 256)]
REPLAYED = [(16, 4096, 6000, 32, 4), (24, 1120, 8384, 8, 2), (33, 640, 16609, 128, 1)]


def _layer(M, K, N, R):
    rng = np.random.default_rng(M + K + N)
    x = wl.gaussian_bf16((M, K), 1.0, M + K + N)
    w = wl.gaussian_bf16((N, K), 0.02, M + K + N + 1)
    w[rng.random((N, K)) >= 0.5] = 0
    a, b = (wl.gaussian_bf16((K, R), 0.05, 2), wl.gaussian_bf16((R, N), 0.05, 3)) if R else (None, None)
    rb, rv, ro = oracle.encode(w)
    args = [to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), None if a is None else to_dev_u16(a), None if b is None else to_dev_u16(b)]
    return args, lambda: oracle.linear(x, w, a, b), rv.size


def _call(args, M, N, room, fill=0x5A):
    import paper_2601_16991_amd as salr
    buf = torch.full((room + 4096,), fill, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    salr.salr_sparse_lowrank_linear(*args, y, buf[:room] if room else None)
    torch.cuda.synchronize()
    assert bool((buf[room:] == fill).all())
    return y


def _without_waiting(call):
    """`call` three times, with waves that do not wait for T: what they find is left to chance, the bits are not."""
    import paper_2601_16991_amd as salr
    salr.lib().salr_set_handover_polls(0)
    try:
        return [call() for _ in range(3)]
    finally:
        salr.lib().salr_set_handover_polls(-1)


@pytest.mark.parametrize("M,K,N,R", [c[:4] for c in HANDED + PARTS] + OTHERS)
def test_close_to_the_oracle_whatever_adds_the_adapters(M, K, N, R):
    import paper_2601_16991_amd as salr
    args, ref, _ = _layer(M, K, N, R)
    size = salr.salr_linear_workspace_bytes_fastest(M, K, N, R)
    print(f"[one launch] M{M} K{K} N{N} R{R}: {size} bytes", flush=True)
    ref = ref()
    y = _call(args, M, N, size)
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    assert torch.equal(_call(args, M, N, size, 0xFF), y)       # what the workspace held before is of no account
    assert torch.equal(_call(args, M, N, size + 65536), y)     # nor what it has beyond


@pytest.mark.parametrize("M,K,N,R,parts", HANDED)
def test_no_wait_for_the_low_rank_product(M, K, N, R, parts):
    """Waves that do not find T when they look leave their sums to T's last workgroup, with no wait all that come before it.  Same bits."""
    import paper_2601_16991_amd as salr
    args, _, _ = _layer(M, K, N, R)
    size = salr.salr_linear_workspace_bytes_fastest(M, K, N, R)
    print(f"[one launch] M{M} K{K} N{N} R{R}: no wait", flush=True)
    y = _call(args, M, N, size)
    for again in _without_waiting(lambda: _call(args, M, N, size)):
        assert torch.equal(again, y)


@pytest.mark.parametrize("M,K,N,R,parts", HANDED_CODES)
def test_four_bit_values(M, K, N, R, parts):
    import paper_2601_16991_amd as salr
    args, _, nnz = _layer(M, K, N, R)
    codes, scales = salr.nf4_quantize(args[2])
    w = oracle.decode(to_host_u32(args[1]), to_host_u16(salr.nf4_dequantize(codes, scales, nnz))[:nnz], to_host_u32(args[3]), N, K)
    ref = oracle.linear(to_host_u16(args[0]), w, to_host_u16(args[4]), to_host_u16(args[5]))
    print(f"[one launch] quantised M{M} K{K} N{N} R{R}", flush=True)

    def call():
        y = salr.qsalr_linear(args[0], args[1], codes, scales, args[3], nnz, args[4], args[5])
        torch.cuda.synchronize()
        return y

    y = call()
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    for again in _without_waiting(call):
        assert torch.equal(again, y)


@pytest.mark.parametrize("M,K,N,R,parts", REPLAYED)
@pytest.mark.parametrize("kind", ["plain", "codes"])
@pytest.mark.parametrize("polls", [-1, 0])
def test_graph_replays_with_new_inputs(kind, polls, M, K, N, R, parts):
    """A captured call has the same tag on every replay: the words are clear again after each, whoever came last, and eager calls on the same
    workspace come between."""
    import paper_2601_16991_amd as salr
    args, _, nnz = _layer(M, K, N, R)
    x = args[0].clone()
    y, other = (torch.empty((M, N), dtype=torch.int16, device=dev()) for _ in range(2))
    if kind == "codes":
        codes, scales = salr.nf4_quantize(args[2])
        rest = (args[1], codes, scales, args[3], nnz, args[4], args[5])
        fn, size, eager = salr.salr_qsalr_linear, salr.salr_qsalr_linear_workspace_bytes_fastest(M, K, N, R, nnz), salr.qsalr_linear
    else:
        rest = tuple(args[1:])
        fn, size, eager = salr.salr_sparse_lowrank_linear, salr.salr_linear_workspace_bytes_fastest(M, K, N, R), salr.linear
    ws = torch.full((size,), 0x5A, dtype=torch.uint8, device=dev())
    fn(x, *rest, other, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    salr.lib().salr_set_handover_polls(polls)
    try:
        with torch.cuda.graph(graph):
            fn(x, *rest, y, ws)
    finally:
        salr.lib().salr_set_handover_polls(-1)
    for turn in range(6):
        print(f"[one launch] {kind} M{M} K{K} N{N} R{R}: replay {turn}", flush=True)
        x.copy_(to_dev_u16(wl.gaussian_bf16((M, K), 1.0 + turn, turn)))
        y.zero_()
        graph.replay()
        if turn % 2:
            torch.cuda.synchronize()
            fn(args[0], *rest, other, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, eager(x, *rest))


@pytest.mark.parametrize("M,K,N,R,parts", REPLAYED)
def test_two_calls_at_once(M, K, N, R, parts):
    """Calls on two streams, each on a workspace of its own, share the CUs: whoever waits for T longer than it wants to does without."""
    import paper_2601_16991_amd as salr
    args, _, _ = _layer(M, K, N, R)
    size = salr.salr_linear_workspace_bytes_fastest(M, K, N, R)
    want = _call(args, M, N, size)
    streams = [torch.cuda.Stream() for _ in range(2)]
    ws = [torch.full((size,), 0x5A, dtype=torch.uint8, device=dev()) for _ in streams]
    ys = [[torch.empty((M, N), dtype=torch.int16, device=dev()) for _ in range(8)] for _ in streams]
    torch.cuda.synchronize()
    print(f"[one launch] M{M} K{K} N{N} R{R}: two streams", flush=True)
    for i in range(8):
        for stream, w, y in zip(streams, ws, ys):
            salr.salr_sparse_lowrank_linear(*args, y[i], w, stream=stream)
    torch.cuda.synchronize()
    assert all(torch.equal(y, want) for per_stream in ys for y in per_stream)
