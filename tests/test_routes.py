"""That the GPU tests of one path reach that path: what the calls they list are planned to take, asked on the host of the code that decides it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2601_16991_amd")


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    """route(kind, M, K, N, R, nnz) -> what tests/routes/routes.cpp prints for it, as a dict."""
    if not os.path.exists(os.path.join(PACKAGE, "libsalr_hip.so")):
        from paper_2601_16991_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("routes") / "routes")
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-Wno-attributes", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PACKAGE, "csrc"), "-isystem", "/opt/rocm/include", "-o", exe, os.path.join(ROOT, "tests", "routes", "routes.cpp"),
                    "-L" + PACKAGE, "-lsalr_hip", "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + PACKAGE, "-Wl,-rpath,/opt/rocm/lib"], check=True)

    def ask(kind, M, K, N, R, nnz=0):
        out = subprocess.run([exe], input=f"{kind} {M} {K} {N} {R} {nnz}\n", text=True, capture_output=True, check=True).stdout
        return dict(field.split("=") for field in out.strip().split(" ") if "=" in field)
    return ask


def test_row_tiled_calls_hand_t_over_inside_the_launch(route):
    import test_gpu_one_launch as t
    for M, K, N, R, parts in t.HANDED:
        r = route("linear", M, K, N, R)
        assert (r["kernel"], r["handed"], r["parts"]) == ("rowtile", "1", str(parts)), (M, K, N, R, r)
    for M, K, N, R, parts in t.HANDED_CODES:
        r = route("codes", M, K, N, R, N * K // 2)
        assert (r["kernel"], r["handed"], r["parts"]) == ("rowtile", "1", str(parts)), (M, K, N, R, r)
    for M, K, N, R, parts in t.PARTS:
        r = route("linear", M, K, N, R)
        assert (r["kernel"], r["slices"], r["parts"]) == ("rowtile", "1", str(parts)), (M, K, N, R, r)
    assert set(t.REPLAYED) <= set(t.HANDED_CODES)
    # every variant of the kernel that does: parts by tokens
    tiers = {(min(p for p in (16, 32, 64, 128) if c[0] <= p), c[4]) for c in t.HANDED}
    assert tiers == {(m, q) for m in (16, 32, 64, 128) for q in (1, 2, 4) if q < 4 or m <= 32}


def test_small_batch_calls_form_t_inside_the_launch(route):
    import test_gpu_shared_t as t
    kernels = {"plain": ("linear", "stream"), "prepared": ("linear", "stream"), "codes": ("codes", "codes"), "2of4": ("2of4", "2of4")}
    shapes = [("beside", c) for c in t.BESIDE] + [("own", c) for c in t.OWN]
    for kind, M, K, N, R, density in t.CALLS:
        c = (M, K, N, R, density)
        how = [h for h, s in shapes if s == c]
        if not how and kind != "2of4" or kind == "codes" and K > 4096:
            continue
        asked, kernel = kernels[kind]
        r = route(asked, M, K, N, R, int(N * K * density))
        assert r["kernel"] == kernel and (r["shared"] == how[0] if how else r["shared"] != "no"), (kind, c, r)
    for kind in t.KINDS:   # both ways under each kind
        assert {h for h, s in shapes if (kind, *s) in t.CALLS} == {"beside", "own"}
    assert set(t.REPLAYED) <= set(t.BESIDE + t.OWN)


def test_gradients_are_beside_every_tile_of_the_stage(route):
    import test_gpu_backward_beside as t
    seen = set()
    for M, K, N, R, mt, nt, split in t.BESIDE:
        r = route("backward", M, K, N, R)
        assert (r["beside"], r["mt"], r["nt"], r["split"]) == ("1", str(mt), str(nt), str(split)), (M, K, N, R, r)
        four = -(-R // 32) * 32 % 64 == 0 and mt * nt <= 128 * 128
        seen.add((mt, nt, split > 1, four))
    tiles = [(64, 64), (64, 128), (64, 256), (128, 128)]
    assert seen == {(m, n, s, f) for m, n in tiles for s in (False, True) for f in (False, True)} | {(128, 256, s, False) for s in (False, True)}


# Three passes over the rows, longer than the stage: beside it only where all workgroups find a place with it, or it leaves half of them
@pytest.mark.parametrize("M,K,N,R,beside", [(768, 2048, 2048, 64, 1), (768, 2048, 2048, 65, 0), (1024, 2048, 2048, 96, 1), (1024, 3072, 768, 96, 0),
                                            (512, 4096, 1024, 96, 1), (800, 2080, 6720, 96, 1), (160, 2048, 2048, 97, 0)])
def test_gradients_that_would_start_behind_the_stage_are_launches_of_their_own(route, M, K, N, R, beside):
    assert route("backward", M, K, N, R)["beside"] == str(beside)


def test_calls_on_workspaces_that_start_inside_a_vector_would_hand_over(route):
    import test_gpu_workspace as t
    for kind, M, K, N, R in t.INSIDE_A_VECTOR:
        r = route({"plain": "linear", "prepared": "linear"}.get(kind, kind), M, K, N, R, N * K // 2)
        assert r.get("handed") == "1" or r.get("shared") in ("own", "beside") or r.get("beside") == "1", (kind, M, K, N, R, r)
