"""Which memory a call uses: the size that the query for the fastest path tells is all it needs, through the boundary and in
Python, and a Python call whose caller brings less still runs where torch's allocator has no more to give.  Results against the fp64
CPU oracle (max |Y - Y_ref| <= 1e-2 * max |Y_ref|); calls on the same path bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import salr_workloads as wl
from gpu_util import dev, to_dev_u16, to_dev_u32, y_to_f64

pytestmark = pytest.mark.gpu

REL_TOL = 1e-2


def _layer(M, K, N, R):
    seed = M + K + N
    x, w = wl.gaussian_bf16((M, K), 1.0, seed), wl.gaussian_bf16((N, K), 0.02, seed + 1)
    w[np.random.default_rng(seed).random((N, K)) >= 0.5] = 0
    a, b = (wl.gaussian_bf16((K, R), 0.05, seed + 2), wl.gaussian_bf16((R, N), 0.05, seed + 3)) if R else (None, None)
    rb, rv, ro = oracle.encode(w)
    args = [to_dev_u16(x), to_dev_u32(rb), to_dev_u16(rv), to_dev_u32(ro), None if a is None else to_dev_u16(a),
            None if b is None else to_dev_u16(b)]
    return args, oracle.linear(x, w, a, b), rv.size


def _ok(y, ref):
    return float(np.max(np.abs(y_to_f64(y) - ref))) <= REL_TOL * float(np.max(np.abs(ref)))


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device=dev())


# rows that end in half a step of 64 columns, outputs that are no multiple of 16, both, neither
@pytest.mark.parametrize("M,K,N,R", [(300, 2720, 267, 24), (130, 96, 300, 0), (200, 4096, 267, 0), (300, 544, 100, 65), (300, 512, 528, 8)])
def test_fastest_size_is_enough(M, K, N, R):
    """Through the boundary it gives what a call without a workspace gives, bit for bit, and nothing behind it is touched; in
    Python the call then allocates its result and nothing else."""
    import paper_2601_16991_amd as salr
    args, ref, nnz = _layer(M, K, N, R)
    size = salr.salr_linear_workspace_bytes_fastest(M, K, N, R)
    print(f"[workspace] M{M} K{K} N{N} R{R}: told {salr.salr_linear_workspace_bytes(M, K, N, R)}, fastest {size}", flush=True)
    alone = salr.linear(*args)
    buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    salr.salr_sparse_lowrank_linear(*args, y, buf[:size])
    torch.cuda.synchronize()
    assert torch.equal(y, alone) and _ok(y, ref) and bool((buf[size:] == 0x5A).all())
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    y = salr.linear(*args, buf[:size])
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before + 1
    torch.cuda.synchronize()
    assert torch.equal(y, alone)


@pytest.mark.parametrize("M,K,N,R", [(300, 2720, 267, 24), (200, 4096, 267, 0), (300, 544, 100, 8)])
def test_fastest_size_is_enough_for_four_bit_values(M, K, N, R):
    import paper_2601_16991_amd as salr
    args, _, nnz = _layer(M, K, N, R)
    codes, scales = salr.nf4_quantize(args[2])
    qargs = [args[0], args[1], codes, scales, args[3], nnz, args[4], args[5]]
    size = salr.salr_qsalr_linear_workspace_bytes_fastest(M, K, N, R, nnz)
    print(f"[workspace] quantised M{M} K{K} N{N} R{R}: fastest {size}", flush=True)
    alone = salr.qsalr_linear(*qargs)
    buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    salr.salr_qsalr_linear(*qargs, y, buf[:size])
    torch.cuda.synchronize()
    assert torch.equal(y, alone) and bool((buf[size:] == 0x5A).all())


# N no multiple of 4 on many rows: split over K with the fastest size only; rows of no whole chunks, where the told size is for other
# kernels; the plan within the told size, with T in the same launch and (17 x 512 x 8320) without room for that
ROW_TILED = [(16, 1152, 8193, 8), (40, 640, 8195, 33), (65, 512, 8198, 0), (5, 5408, 1131, 8), (20, 9120, 333, 24), (100, 992, 133, 5),
             (64, 2048, 260, 5), (128, 4224, 388, 33), (17, 512, 8320, 16)]


@pytest.mark.parametrize("M,K,N,R", ROW_TILED)
@pytest.mark.parametrize("size_of", ["salr_linear_workspace_bytes", "salr_linear_workspace_bytes_fastest"])
def test_row_tiled_calls_stay_inside_their_workspace(M, K, N, R, size_of):
    """At either size: close to the oracle, nothing behind the workspace touched, and what it held before of no account."""
    import paper_2601_16991_amd as salr
    args, ref, _ = _layer(M, K, N, R)
    size = getattr(salr, size_of)(M, K, N, R)
    print(f"[workspace] M{M} K{K} N{N} R{R}: {size_of} {size}", flush=True)
    buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device=dev())
    y = torch.empty((M, N), dtype=torch.int16, device=dev())
    salr.salr_sparse_lowrank_linear(*args, y, buf[:size] if size else None)
    torch.cuda.synchronize()
    assert _ok(y, ref) and bool((buf[size:] == 0x5A).all())
    buf[:size] = 0xFF   # NaN as fp32 and as bf16
    again = torch.empty_like(y)
    salr.salr_sparse_lowrank_linear(*args, again, buf[:size] if size else None)
    torch.cuda.synchronize()
    assert torch.equal(again, y)


# (65 to 128 tokens: at the told size the values are dequantised first)
@pytest.mark.parametrize("M,K,N,R", ROW_TILED + [(66, 160, 130, 0), (96, 4096, 515, 16), (128, 1152, 2050, 40)])
@pytest.mark.parametrize("size_of", ["salr_qsalr_linear_workspace_bytes", "salr_qsalr_linear_workspace_bytes_fastest"])
def test_row_tiled_calls_on_four_bit_values_stay_inside_their_workspace(M, K, N, R, size_of):
    import paper_2601_16991_amd as salr
    args, _, nnz = _layer(M, K, N, R)
    codes, scales = salr.nf4_quantize(args[2])
    w = oracle.decode(args[1].cpu().numpy().view(np.uint32), salr.nf4_dequantize(codes, scales, nnz).cpu().numpy().view(np.uint16)[:nnz],
                      args[3].cpu().numpy().view(np.uint32), N, K)
    ref = oracle.linear(args[0].cpu().numpy().view(np.uint16), w, *(None if t is None else t.cpu().numpy().view(np.uint16) for t in args[4:]))
    size = getattr(salr, size_of)(M, K, N, R, nnz)
    print(f"[workspace] quantised M{M} K{K} N{N} R{R}: {size_of} {size}", flush=True)
    buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device=dev())
    y, again = (torch.empty((M, N), dtype=torch.int16, device=dev()) for _ in range(2))
    qargs = (args[0], args[1], codes, scales, args[3], nnz, args[4], args[5])
    salr.salr_qsalr_linear(*qargs, y, buf[:size] if size else None)
    torch.cuda.synchronize()
    assert _ok(y, ref) and bool((buf[size:] == 0x5A).all())
    buf[:size] = 0xFF   # NaN as fp32 and as bf16
    salr.salr_qsalr_linear(*qargs, again, buf[:size] if size else None)
    torch.cuda.synchronize()
    assert torch.equal(again, y)


# the small-batch kernels with T from workgroups beside their own work and from workgroups of their own, the row-tiled kernel in one launch, and
# the gradients beside the matrix stage (tests/test_routes.py)
INSIDE_A_VECTOR = [("plain", 16, 1024, 4096, 32), ("plain", 5, 2048, 241, 8), ("prepared", 3, 2048, 1025, 64), ("codes", 16, 1024, 4096, 32),
                   ("2of4", 16, 1024, 4096, 32), ("plain", 24, 1120, 8384, 8), ("codes", 33, 1024, 8320, 16), ("backward", 96, 160, 192, 40)]


@pytest.mark.parametrize("kind,M,K,N,R", INSIDE_A_VECTOR)
@pytest.mark.parametrize("start", [4, 8])
def test_workspaces_that_start_inside_a_vector(kind, M, K, N, R, start):
    """A workspace is told to be aligned to 256 bytes, and one that is not ran slowly and still does: nothing in it is exchanged 64 bits at a
    time.  The same bits (of the backward pass: dX, the gradients being cut into other slices)."""
    import paper_2601_16991_amd as salr
    args, ref, nnz = _layer(M, K, N, R)
    extra = []
    if kind == "2of4":
        w = oracle.mask_nm(wl.gaussian_bf16((N, K), 0.02, 1), 2, 4)
        args[1:4] = [f(v) for f, v in zip((to_dev_u32, to_dev_u16, to_dev_u32), oracle.encode(w))]
    elif kind == "prepared":
        extra = [salr.build_slice_table(args[1], args[3], K)]
    elif kind == "codes":
        args[2:3], extra = salr.nf4_quantize(args[2]), [nnz]
    elif kind == "backward":
        dy = to_dev_u16(wl.gaussian_bf16((M, N), 1.0, 9))
    call = {"plain": salr.salr_sparse_lowrank_linear, "prepared": salr.salr_sparse_lowrank_linear_prepared, "codes": salr.salr_qsalr_linear,
            "2of4": salr.salr_sparse_lowrank_linear_2of4, "backward": salr.salr_sparse_lowrank_linear_backward}[kind]
    size = (salr.salr_linear_backward_workspace_bytes(M, K, N, R, True, True) if kind == "backward" else
            salr.salr_qsalr_linear_workspace_bytes_fastest(M, K, N, R, nnz) if kind == "codes" else
            salr.salr_linear_2of4_workspace_bytes(M, K, N, R) if kind == "2of4" else salr.salr_linear_workspace_bytes_fastest(M, K, N, R))
    out = []
    for at in (0, start):
        print(f"[workspace] {kind} M{M} K{K} N{N} R{R}: {size} bytes from {at} on", flush=True)
        buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device=dev())
        y = torch.empty((M, K if kind == "backward" else N), dtype=torch.int16, device=dev())
        grads = [torch.empty((K, R), dtype=torch.int16, device=dev()), torch.empty((R, N), dtype=torch.int16, device=dev())]
        if kind == "backward":
            call(args[0], dy, *args[1:], y, *grads, buf[at:at + size])
        else:
            call(*args[:-2], *extra, *args[-2:], y, buf[at:at + size])
        torch.cuda.synchronize()
        assert bool((buf[:at] == 0x5A).all()) and bool((buf[at + size:] == 0x5A).all())
        out.append((y, *(g.view(torch.bfloat16).float() for g in grads)))
    assert torch.equal(out[0][0], out[1][0])
    if kind == "backward":
        for g, h in zip(out[0][1:], out[1][1:]):
            assert float((g - h).abs().max()) <= 2.0 ** -7 * float(g.abs().max())
    elif kind in ("plain", "prepared"):
        assert _ok(out[1][0], ref)


@pytest.mark.parametrize("form", ["told", "none", "quantised"])
def test_runs_where_the_allocator_has_no_more(form):
    """The decoded weight of this layer takes 34 MB and its split sums more; the allocator may hand out the result and little else (in
    the last form the told workspace as well, 17 MB of values)."""
    import paper_2601_16991_amd as salr
    M, K, N, R = 130, 4128, 4096, 16
    args, ref, nnz = _layer(M, K, N, R)
    told = salr.salr_linear_workspace_bytes(M, K, N, R)
    ws = _bytes(told)
    if form == "quantised":
        codes, scales = salr.nf4_quantize(args[2])
        q = salr.nf4_dequantize(codes, scales, nnz)
        plain = salr.linear(args[0], args[1], q, *args[3:])   # the same products on the dequantised values
        del q
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.mem_get_info()[1]
    more = 26 << 20   # (small allocations come in pieces of 2 and 20 MB)
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + more) / total)
    try:
        print(f"[workspace] {form} with {more >> 20} MB to allocate", flush=True)
        if form == "quantised":
            y = salr.qsalr_linear(args[0], args[1], codes, scales, args[3], nnz, args[4], args[5])
        else:
            y = salr.linear(*args, ws if form == "told" else None)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    if form == "quantised":
        scale = float(plain.view(torch.bfloat16).float().abs().max())
        assert float((y.view(torch.bfloat16).float() - plain.view(torch.bfloat16).float()).abs().max()) <= REL_TOL * scale
    else:
        assert _ok(y, ref)
