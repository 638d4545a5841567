"""Where a slice of the row-tiled kernel starts in the packed values: the bitmap words left of it are counted sixteen chunks of four rows at a
time, 112 chunks in flight.  Against the fp64 oracle (max |Y - Y_ref| <= 1e-2 * max |Y_ref|), and the same bits from a slice table where its starts
are the slices'."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import to_dev_u16, to_dev_u32, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2


# slices that start below, at and past 16 and 112 chunks, rows of 32, 64 and 96 columns past whole chunks, a last tile of few rows, empty and full rows
@pytest.mark.parametrize("M,K,N,R,density", [(8, 14336, 256, 8, 0.5), (16, 28672, 160, 16, 0.5), (3, 31744, 131, 8, 0.3), (33, 6176, 260, 8, 0.5),
                                             (128, 16448, 129, 32, 0.5), (40, 14432, 500, 24, 0.7), (16, 8192, 1024, 8, 0.05), (64, 20480, 144, 8, 1.0)])
def test_slices_start_where_the_words_left_of_them_say(M, K, N, R, density):
    import paper_2601_16991_amd as salr
    rng = np.random.default_rng(M + K + N)
    x = wl.gaussian_bf16((M, K), 1.0, M + K)
    w = wl.gaussian_bf16((N, K), 0.02, K + N)
    w[rng.random((N, K)) >= density] = 0
    w[5], w[17, : K // 2] = 0, 0
    a, b = wl.gaussian_bf16((K, R), 0.05, 2), wl.gaussian_bf16((R, N), 0.05, 3)
    rb, rv, ro = oracle.encode(w)
    ref = oracle.linear(x, w, a, b)
    args = [to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro)]
    ab = [to_dev_u16(a), to_dev_u16(b)]
    print(f"[slice start] M{M} K{K} N{N} R{R} {density}", flush=True)
    y = salr.linear(*args, *ab)
    assert float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))
    table = salr.build_slice_table(args[1], args[3], K)
    assert torch.equal(salr.linear_prepared(*args, table, *ab), y)
