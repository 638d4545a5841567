"""Decoding calls of the small-batch kernels whose first workgroups form T = X A_cat for all of them: against the fp64 oracle
(max |Y - Y_ref| <= 1e-2 * max |Y_ref|), and bit for bit where only who forms T and when is another."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import dev, to_dev_u16, to_dev_u32, to_host_u16, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2

# M, K, N, R and the share of nonzeros: which calls of these form T beside their own work and which in workgroups of its own tests/test_routes.py
# holds them to.  As many row groups as T has slices and one row more; 2, 3 and 4 chunks a wave, fewer chunks than waves, uneven slices, rows of
# more than 32 chunks (with a table: 64); tokens and ranks at the edges of the tiles of 16, 8 and 128 ranks, 4 pairs of rank tiles
BESIDE = [(1, 4096, 4096, 32, 0.5), (16, 4096, 4096, 32, 0.5), (16, 1024, 4096, 32, 0.5), (15, 2176, 8176, 16, 0.5), (7, 1152, 4100, 128, 0.7)]
OWN = [(16, 4096, 256, 32, 0.5), (5, 4096, 241, 8, 0.5), (16, 1152, 1024, 128, 0.5), (7, 128, 512, 40, 0.5), (9, 2048, 1040, 64, 0.3),
       (16, 2176, 800, 72, 0.5), (16, 4224, 2000, 96, 0.5), (3, 4224, 1025, 128, 0.5), (16, 3968, 2500, 64, 0.9), (2, 1280, 530, 24, 1.0)]
# formed so under 2:4 only: the row-tiled kernel takes the others
LARGE = [(15, 3072, 8176, 16, 0.5), (16, 8192, 512, 48, 0.5)]
KINDS = ("plain", "prepared", "codes", "2of4")
# (the 2:4 call passes N % 4 != 0 on few rows on to the plain one)
CALLS = [(kind, *c) for c in BESIDE + OWN + LARGE for kind in KINDS if kind != "2of4" or c[2] % 4 == 0]


class Call:
    """A layer, what its kind of call takes, and the oracle's result."""

    def __init__(self, kind, M, K, N, R, density):
        import paper_2601_16991_amd as salr
        rng = np.random.default_rng(M + K + N)
        x = wl.gaussian_bf16((M, K), 1.0, M + K + N)
        w = wl.gaussian_bf16((N, K), 0.02, M + K + N + 1)
        if kind == "2of4":
            w = oracle.mask_nm(w, 2, 4)
        else:
            w[rng.random((N, K)) >= density] = 0
        a, b = wl.gaussian_bf16((K, R), 0.05, 2), wl.gaussian_bf16((R, N), 0.05, 3)
        rb, rv, ro = oracle.encode(w)
        self.kind, self.shape, self.inputs = kind, (M, K, N, R), (x, w, a, b)
        self.x, self.a, self.b = to_dev_u16(x), to_dev_u16(a), to_dev_u16(b)
        bitmap, values, offsets = to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro)
        if kind == "codes":
            codes, scales = salr.nf4_quantize(values)
            w = oracle.decode(rb, to_host_u16(salr.nf4_dequantize(codes, scales, rv.size))[:rv.size], ro, N, K)
            self.inputs = (x, w, a, b)
            self.weight = (bitmap, codes, scales, offsets, rv.size)
            self.size = salr.salr_qsalr_linear_workspace_bytes(M, K, N, R, rv.size)
        else:
            self.weight = (bitmap, values, offsets) + ((salr.build_slice_table(bitmap, offsets, K),) if kind == "prepared" else ())
            self.size = (salr.salr_linear_2of4_workspace_bytes if kind == "2of4" else salr.salr_linear_workspace_bytes)(M, K, N, R)
        self.entry = {"plain": salr.salr_sparse_lowrank_linear, "prepared": salr.salr_sparse_lowrank_linear_prepared,
                      "codes": salr.salr_qsalr_linear, "2of4": salr.salr_sparse_lowrank_linear_2of4}[kind]

    def oracle(self):
        return oracle.linear(*self.inputs)

    def into(self, y, workspace, x=None, a=None, stream=None):
        self.entry(self.x if x is None else x, *self.weight, self.a if a is None else a, self.b, y, workspace, stream=stream)

    def out(self):
        return torch.empty((self.shape[0], self.shape[2]), dtype=torch.int16, device=dev())

    def __call__(self, fill=0x5A, **kwargs):
        """On exactly the told workspace, whose bytes hold `fill` before."""
        buf, y = torch.full((self.size + 4096,), fill, dtype=torch.uint8, device=dev()), self.out()
        self.into(y, buf[:self.size], **kwargs)
        torch.cuda.synchronize()
        assert bool((buf[self.size:] == fill).all())
        return y


@pytest.mark.parametrize("kind,M,K,N,R,density", CALLS)
def test_close_to_the_oracle_whoever_forms_t(kind, M, K, N, R, density):
    import paper_2601_16991_amd as salr
    call = Call(kind, M, K, N, R, density)
    ref = call.oracle()
    print(f"[shared t] {kind} M{M} K{K} N{N} R{R}", flush=True)
    y = call()
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    assert torch.equal(call(0xFF), y)   # what the workspace held before is of no account
    # A_cat that starts inside a vector: a launch in front
    assert torch.equal(call(a=torch.empty(K * R + 1, dtype=call.a.dtype, device=dev())[1:].view(K, R).copy_(call.a)), y)
    salr.lib().salr_set_handover_polls(0)   # workgroups that do not find T at once form it themselves
    try:
        for _ in range(3):
            assert torch.equal(call(), y)
    finally:
        salr.lib().salr_set_handover_polls(-1)


REPLAYED = [BESIDE[0], BESIDE[2], OWN[2]]


@pytest.mark.parametrize("polls", [-1, 0])
@pytest.mark.parametrize("kind", ["plain", "codes", "2of4"])
@pytest.mark.parametrize("M,K,N,R,density", REPLAYED)
def test_graph_replays_with_new_inputs(M, K, N, R, density, kind, polls):
    """A captured call has the same tag on every replay: the words are clear again after each, whoever came last."""
    import paper_2601_16991_amd as salr
    call = Call(kind, M, K, N, R, density)
    ws = torch.full((call.size,), 0x5A, dtype=torch.uint8, device=dev())
    y, other, x = call.out(), call.out(), call.x.clone()
    call.into(other, ws, x=x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    salr.lib().salr_set_handover_polls(polls)
    try:
        with torch.cuda.graph(graph):
            call.into(y, ws, x=x)
    finally:
        salr.lib().salr_set_handover_polls(-1)
    for turn in range(6):
        print(f"[shared t] {kind} M{M} K{K} N{N} R{R}: replay {turn}", flush=True)
        x.copy_(to_dev_u16(wl.gaussian_bf16((M, K), 1.0 + turn, turn)))
        y.zero_()
        graph.replay()
        if turn % 2:
            torch.cuda.synchronize()
            call.into(other, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, call(x=x))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("M,K,N,R,density", REPLAYED)
def test_two_calls_at_once(M, K, N, R, density, kind):
    """Calls on two streams, each on a workspace of its own, share the CUs: whoever waits for T longer than it wants to forms it itself."""
    call = Call(kind, M, K, N, R, density)
    want = call()
    streams = [torch.cuda.Stream() for _ in range(2)]
    ws = [torch.full((call.size,), 0x5A, dtype=torch.uint8, device=dev()) for _ in streams]
    ys = [[call.out() for _ in range(8)] for _ in streams]
    torch.cuda.synchronize()
    print(f"[shared t] {kind} M{M} K{K} N{N} R{R}: two streams", flush=True)
    for i in range(8):
        for stream, w, y in zip(streams, ws, ys):
            call.into(y[i], w, stream=stream)
    torch.cuda.synchronize()
    assert all(torch.equal(y, want) for per_stream in ys for y in per_stream)
