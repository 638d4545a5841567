"""The adapter gradients in workgroups beside the matrix stage of dX: against the fp64 oracle (max |G - G_ref| <= 1e-2 * max |G_ref|), and
against the call without dX, whose gradients have a launch of their own: the same T and T', fp32 sums over the rows that may be cut into
another number of slices.  Such sums differ by about 2^-24 of their terms' magnitude, so their bf16 roundings by one step (2^-7 of a
value at most) where one lies beside a rounding boundary, which is 2^-24 / 2^-8 times some tens of terms: below 1 in 500."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import dev, to_dev_u16, to_dev_u32, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2


def _layer(M, K, N, R, seed=0):
    x, dy = wl.gaussian_bf16((M, K), 1.0, seed + M), wl.gaussian_bf16((M, N), 1.0, seed + M + 1)
    w = oracle.mask_topk_rows(wl.gaussian_bf16((N, K), 0.02, seed + 2), K // 2)
    a, b = wl.gaussian_bf16((K, R), 0.05, seed + 3), wl.gaussian_bf16((R, N), 0.05, seed + 4)
    rb, rv, ro = oracle.encode(w)
    return (x, dy, w, a, b), [to_dev_u16(x), to_dev_u16(dy), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), to_dev_u16(a), to_dev_u16(b)]


def _out(*shape):
    return torch.full(shape, 0x7FC0, dtype=torch.int16, device=dev())


# M, K, N, R and the stage of dX that the gradients are beside (tests/test_routes.py holds them to it): its tile and its split of the contraction.  One step
# of 32 rows and a few, one to eight slices of them; 64-column blocks that end early; two and four rank tiles a pass, two passes
BESIDE = [(32, 96, 64, 8, 64, 64, 1), (64, 32, 128, 16, 64, 64, 1), (96, 160, 192, 40, 64, 64, 1), (256, 416, 320, 96, 64, 64, 1),
          (512, 1056, 576, 64, 64, 64, 1), (480, 2048, 1024, 32, 64, 64, 1), (544, 2080, 2112, 8, 64, 64, 1), (1024, 2048, 2048, 72, 64, 64, 1),
          (32, 32, 1408, 64, 64, 64, 4), (256, 256, 4096, 8, 64, 64, 16), (416, 2496, 64, 40, 64, 128, 1), (2048, 1024, 1024, 32, 64, 128, 1),
          (32, 2208, 1536, 64, 64, 128, 8), (512, 512, 8192, 32, 64, 128, 8), (1568, 2464, 512, 40, 64, 256, 1), (2048, 2048, 1024, 32, 64, 256, 1),
          (160, 1088, 9216, 64, 64, 256, 16), (512, 2048, 4096, 32, 64, 256, 4), (1120, 1856, 192, 64, 128, 128, 1), (1632, 1280, 128, 96, 128, 128, 1),
          (96, 1088, 6656, 40, 128, 128, 16), (96, 2112, 3328, 8, 128, 128, 8), (2144, 7328, 128, 8, 128, 256, 1), (2048, 4096, 4096, 32, 128, 256, 1),
          (1504, 352, 15872, 32, 128, 256, 8)]


@pytest.mark.parametrize("M,K,N,R", [c[:4] for c in BESIDE])
def test_same_gradients_beside_the_stage_and_alone(M, K, N, R):
    import paper_2601_16991_amd as salr
    host, args = _layer(M, K, N, R)
    refs = oracle.linear_backward(*host)
    print(f"[beside] M{M} K{K} N{N} R{R}", flush=True)
    dx, da, db = salr.linear_backward(*args)
    _, da_alone, db_alone = salr.linear_backward(*args, False, True)
    torch.cuda.synchronize()
    for g, ref in zip((dx, da, db), refs):
        assert float(np.max(np.abs(y_to_f64(g) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    for g, alone in ((da, da_alone), (db, db_alone)):
        g, alone = y_to_f64(g), y_to_f64(alone)
        d = np.abs(g - alone)
        assert np.all(d <= 2.0 ** -7 * np.abs(alone) + 1e-5 * np.max(np.abs(alone))) and np.count_nonzero(d) * 500 <= d.size


@pytest.mark.parametrize("M,K,N,R", [(96, 160, 192, 40), (512, 1056, 576, 64)])
def test_one_gradient_inside_the_told_workspace(M, K, N, R):
    """dX with one of the two; whatever the workspace holds before, and nothing behind it touched."""
    import paper_2601_16991_amd as salr
    _, args = _layer(M, K, N, R)
    dx, da, db = salr.linear_backward(*args)
    for fill in (0x00, 0x5A, 0xFF):
        for which in ("da", "db", "both"):
            print(f"[beside] M{M} K{K} N{N} R{R}: {which}, workspace of {fill:#x}", flush=True)
            size = salr.salr_linear_backward_workspace_bytes(M, K, N, R, True, True)
            buf = torch.full((size + 4096,), fill, dtype=torch.uint8, device=dev())
            gx, ga, gb = _out(M, K), _out(K, R) if which != "db" else None, _out(R, N) if which != "da" else None
            salr.salr_sparse_lowrank_linear_backward(*args, gx, ga, gb, buf[:size])
            torch.cuda.synchronize()
            assert torch.equal(gx, dx) and (ga is None or torch.equal(ga, da)) and (gb is None or torch.equal(gb, db))
            assert bool((buf[size:] == fill).all())


def test_graph_replays_with_new_inputs():
    """The slices' words are clear again after every replay, whose tag is the captured call's."""
    import paper_2601_16991_amd as salr
    M, K, N, R = 512, 1056, 576, 64
    _, args = _layer(M, K, N, R)
    ws = torch.full((salr.salr_linear_backward_workspace_bytes(M, K, N, R, True, True),), 0x5A, dtype=torch.uint8, device=dev())
    out = (_out(M, K), _out(K, R), _out(R, N))
    salr.salr_sparse_lowrank_linear_backward(*args, *out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        salr.salr_sparse_lowrank_linear_backward(*args, *out, ws)
    for turn in range(5):
        print(f"[beside] replay {turn}", flush=True)
        args[0].copy_(to_dev_u16(wl.gaussian_bf16((M, K), 1.0, 100 + turn)))
        args[1].copy_(to_dev_u16(wl.gaussian_bf16((M, N), 1.0, 200 + turn)))
        graph.replay()
        if turn % 2:
            torch.cuda.synchronize()
        want = salr.linear_backward(*args)
        torch.cuda.synchronize()
        assert all(torch.equal(g, r) for g, r in zip(out, want))
