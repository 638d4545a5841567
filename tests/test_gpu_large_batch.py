"""GPU parity of the large-batch path (decode into MFMA operand order, one dense MFMA stage) at the edges of its tiles, splits
and layouts, against the fp64 CPU oracle.  Bar: max |Y - Y_ref| <= 1e-2 * max |Y_ref|."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import dev, to_dev_u16, to_dev_u32, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2


def _check(M, K, N, R, density, quantised=False):
    import paper_2601_16991_amd as salr
    seed = M + 3 * K + 5 * N + R
    rng = np.random.default_rng(seed)
    x = wl.gaussian_bf16((M, K), 1.0, seed)
    w = wl.gaussian_bf16((N, K), 0.02, seed + 1)
    w[rng.random((N, K)) >= density] = 0
    a = wl.gaussian_bf16((K, R), 0.05, seed + 2) if R else None
    b = wl.gaussian_bf16((R, N), 0.05, seed + 3) if R else None
    rb, rv, ro = oracle.encode(w)
    dx, dbm, dro = to_dev_u16(x), to_dev_u32(rb), to_dev_u32(ro)
    da, db = (to_dev_u16(a), to_dev_u16(b)) if R else (None, None)
    print(f"[large batch] M{M} K{K} N{N} R{R} density {density} nf4 {quantised}", flush=True)
    if quantised:
        codes, scales = salr.nf4_quantize(to_dev_u16(rv))
        q = salr.nf4_dequantize(codes, scales, rv.size)
        w = oracle.decode(rb, q.cpu().numpy().view(np.uint16), ro, N, K)
        y = salr.qsalr_linear(dx, dbm, codes, scales, dro, rv.size, da, db)
    else:
        y = salr.linear(dx, dbm, to_dev_u16(rv), dro, da, db)
    torch.cuda.synchronize()
    ref = oracle.linear(x, w, a, b)
    err, scale = float(np.max(np.abs(y_to_f64(y) - ref))), float(np.max(np.abs(ref)))
    assert err <= REL_TOL * scale, f"{err} > {REL_TOL} * {scale}"


# contraction lengths: one half step, half steps after whole ones, pieces of 256 columns and their remainders; outputs that are
# no multiple of 2, 4, 8; row counts around tile edges; ranks that leave whole, half and several steps of the rank dimension
@pytest.mark.parametrize("M,K,N,R,density", [
    (65, 32, 33, 0, 0.5), (129, 96, 17, 5, 0.5), (300, 160, 1, 3, 0.5), (131, 2720, 267, 24, 0.5), (257, 480, 130, 33, 0.3),
    (200, 224, 1027, 64, 0.9), (1025, 288, 65, 65, 0.5), (130, 64, 2051, 8, 0.02), (513, 1056, 4, 96, 0.5), (70, 992, 255, 0, 1.0)])
def test_ragged(M, K, N, R, density):
    _check(M, K, N, R, density)


# layers that take each output tile, with and without a split of the contraction
@pytest.mark.parametrize("M,K,N,R", [
    (150, 1024, 700, 16),        # 64 x 64
    (150, 8192, 512, 16),        # 64 x 64 and 64 x 128, split sixteen ways
    (600, 4096, 1100, 32),       # 64 x 128, split
    (1100, 512, 2050, 130),      # 128 x 128
    (520, 2048, 4104, 40),       # 128 x 256
    (260, 4096, 4096, 32),       # split
    (2050, 1024, 7300, 8),       # 256-row tiles
    (1030, 96, 14400, 8)])
def test_tiles(M, K, N, R):
    _check(M, K, N, R, 0.5)


@pytest.mark.parametrize("M,K,R", [(2100, 8192, 64), (1500, 8224, 130), (4100, 4128, 33),
                                   (3662, 8192, 128), (3663, 8192, 128)])   # the last two: either side of the line to T beside the pass over the weight
def test_adapter_product_of_its_own(M, K, R):
    """T = X A_cat large enough for the split-K product on the MFMA stage's kernel."""
    _check(M, K, 96, R, 0.5)


# fewer steps of 64 columns than waves or slices, half steps, more steps than two rounds of the slices
@pytest.mark.parametrize("M,K,R", [(2100, 32, 72), (2050, 160, 96), (1030, 224, 256), (1360, 1056, 128), (4100, 2144, 40)])
def test_adapter_product_in_blocks_of_32_rows(M, K, R):
    """T = X A_cat beside the pass over the weight where blocks of 16 rows of X and 32 ranks would be more than one a CU."""
    _check(M, K, 80, R, 0.5)


@pytest.mark.parametrize("M,N,R,form", [(130, 96, 8, "linear"), (1040, 80, 40, "linear"), (2100, 64, 72, "linear"), (300, 64, 96, "qsalr"), (2048, 6144, 40, "2of4")])
def test_sums_of_the_adapter_product(M, N, R, form):
    """T = X A_cat beside the pass over the weight: sixteen fp32 sums over every sixteenth step of 64 columns, added up in order.  2^24
    and -2^24 sixteen steps apart cancel in a sum of their own and leave the 1 of another one, which a sum that takes every
    fourth step would lose to the 2^24 before it."""
    import paper_2601_16991_amd as salr
    K = 1088
    x, a, b = np.zeros((M, K), np.float32), np.zeros((K, R), np.float32), np.zeros((R, N), np.float32)
    x[:, 0], x[:, 256], x[:, 1024] = 4096.0, 1.0, -4096.0
    a[0], a[256], a[1024] = 4096.0, 1.0, 4096.0
    b[:] = (1 + np.arange(N) % 7) / 8
    w = np.zeros((N, K), np.uint16)
    w[:, 1::4] = w[:, 2::4] = 0x3F80   # met by zeros only
    rb, rv, ro = oracle.encode(w)
    bf = wl.f32_to_bf16_bits
    dx, dbm, dv, dro, da, db = to_dev_u16(bf(x)), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), to_dev_u16(bf(a)), to_dev_u16(bf(b))
    if form == "qsalr":
        codes, scales = salr.nf4_quantize(dv)
        y = salr.qsalr_linear(dx, dbm, codes, scales, dro, rv.size, da, db)
    else:
        y = (salr.linear_2of4 if form == "2of4" else salr.linear)(dx, dbm, dv, dro, da, db)
    torch.cuda.synchronize()
    assert np.array_equal(y_to_f64(y), np.repeat(b[:1].astype(np.float64) * R, M, axis=0))


@pytest.mark.parametrize("M,K,N,R,density", [(129, 96, 40, 8, 0.8), (300, 2720, 130, 0, 0.8), (600, 512, 257, 32, 0.5), (129, 288, 64, 8, 1.0)])
def test_quantised(M, K, N, R, density):
    _check(M, K, N, R, density, quantised=True)


def test_empty_and_full_rows():
    """Rows without a single value next to full ones (a piece of 256 values spans 33 vectors off a vector boundary)."""
    import paper_2601_16991_amd as salr
    M, K, N = 140, 1280, 100
    x = wl.gaussian_bf16((M, K), 1.0, 5)
    w = wl.gaussian_bf16((N, K), 0.02, 6)
    w[::3] = 0
    w[1::3, :7] = 0
    rb, rv, ro = oracle.encode(w)
    y = salr.linear(to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), None, None)
    torch.cuda.synchronize()
    ref = oracle.linear(x, w, None, None)
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    w[:] = 0
    rb, rv, ro = oracle.encode(w)
    y = salr.linear(to_dev_u16(x), to_dev_u32(rb), torch.zeros(8, dtype=torch.int16, device=dev())[:0], to_dev_u32(ro), None, None)
    torch.cuda.synchronize()
    assert float(np.max(np.abs(y_to_f64(y)))) == 0.0


@pytest.mark.parametrize("M,K,N,R", [(130, 256, 4096, 32), (300, 512, 528, 8), (150, 96, 300, 8), (129, 4096, 256, 16), (520, 2048, 4104, 0)])
def test_every_workspace_size(M, K, N, R):
    """The least workspace, the one the query tells and one with room for everything: each takes its own path through the
    boundary, with the same result; bytes behind the size that was given stay as they were."""
    import paper_2601_16991_amd as salr
    seed = M + K + N
    x, w = wl.gaussian_bf16((M, K), 1.0, seed), wl.gaussian_bf16((N, K), 0.02, seed + 1)
    w[np.random.default_rng(seed).random((N, K)) >= 0.5] = 0
    a, b = (wl.gaussian_bf16((K, R), 0.05, seed + 2), wl.gaussian_bf16((R, N), 0.05, seed + 3)) if R else (None, None)
    rb, rv, ro = oracle.encode(w)
    args = [to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), None if a is None else to_dev_u16(a),
            None if b is None else to_dev_u16(b)]
    ref = oracle.linear(x, w, a, b)
    told = salr.salr_linear_workspace_bytes(M, K, N, R)
    for size in (salr.salr_linear_workspace_bytes_min(M, K, N, R), told, 2 * told + 64 * M * N + (4 << 20)):
        buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device=dev())
        y = torch.empty((M, N), dtype=torch.int16, device=dev())
        salr.salr_sparse_lowrank_linear(*args, y, buf[:size] if size else None)
        torch.cuda.synchronize()
        err = float(np.max(np.abs(y_to_f64(y) - ref)))
        print(f"[large batch] M{M} K{K} N{N} R{R} workspace {size}: max|d| {err:.3e}", flush=True)
        assert err <= REL_TOL * float(np.max(np.abs(ref)))
        assert bool((buf[size:] == 0x5A).all())
        y2 = salr.linear(*args, buf[:size] if size else None)
        torch.cuda.synchronize()
        assert float(np.max(np.abs(y_to_f64(y2) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
