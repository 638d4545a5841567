"""Compile the HIP library for gfx950 into paper_2601_16991_amd/libsalr_hip.so (in-tree).

Every source is compiled to an object of its own (in parallel), then linked; `python build.py --changed` skips
objects that are newer than their source and every header (for quick rebuilds while working on one kernel).  The native
half of the Python binding (csrc/salr_binding.cpp, host code against torch's headers) becomes _salr_binding.so beside
the library and links to it."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsalr_hip.so")
BINDING_SRC = os.path.join(CSRC, "salr_binding.cpp")
BINDING = os.path.join(HERE, "_salr_binding.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # packed-fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",
    # the LDS-DMA loads are issued from inline assembly that sets m0 and says so in its clobber list; the compiler
    # remarks on every such statement that m0 is a reserved register
    "-Wno-inline-asm",
]


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _headers() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(ROOT, "include", "*.h")))


def _run(cmd: list[str]) -> str:
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("build failed: " + " ".join(cmd) + "\n" + out)
    return out


def _binding_commands() -> list[list[str]]:
    """Compile and link lines of the binding (host code only)."""
    from torch.utils import cpp_extension as ext
    import torch
    obj = os.path.join(OBJ_DIR, "salr_binding.o")
    includes = ext.include_paths("cuda") + [sysconfig.get_paths()["include"], os.path.join(ROOT, "include"), CSRC]
    cxx = os.environ.get("CXX", "g++")
    compile_ = [cxx, "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                *[f for i in includes for f in ("-isystem" if "dist-packages" in i or "rocm" in i else "-I", i)], "-c", "-o", obj, BINDING_SRC]
    link = [cxx, "-shared", "-o", BINDING, obj, *["-L" + p for p in ext.library_paths("cuda")[:1]], "-L" + HERE, "-lsalr_hip", "-lc10",
            "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    return [compile_, link]


def _compile_commands(only_changed: bool) -> tuple[list[list[str]], list[str]]:
    """Compile lines of everything, or of what is older than its source or any header; and the library's objects."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    newest_header = max(os.path.getmtime(h) for h in _headers())

    def needed(obj: str, src: str) -> bool:
        return not (only_changed and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header))

    todo, objects = [], []
    if needed(os.path.join(OBJ_DIR, "salr_binding.o"), BINDING_SRC):
        todo.append(_binding_commands()[0])   # the longest one first
    for src in sources():
        obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
        objects.append(obj)
        if needed(obj, src):
            todo.append([hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", "-o", obj, src])
    return todo, objects


def build(verbose: bool = False, only_changed: bool = False, jobs: int | None = None) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    todo, objects = _compile_commands(only_changed)
    if jobs is None:
        jobs = min(8, max(1, len(os.sched_getaffinity(0))))
    if verbose:
        for cmd in todo:
            print(" ".join(cmd), flush=True)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        outs = list(pool.map(_run, todo))
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objects]
    # The interpreter's own symbols keep the linker from refusing undefined ones in the binding: load it once, all symbols now.
    load_binding = [sys.executable, "-c", f"import ctypes, os, torch; ctypes.CDLL({BINDING!r}, mode=os.RTLD_NOW)"]
    for cmd in (link, _binding_commands()[1], load_binding):
        if verbose:
            print(" ".join(cmd), flush=True)
        outs.append(_run(cmd))
    text = "\n".join(o for o in outs if o.strip())
    if verbose and text:
        print(text)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, only_changed="--changed" in sys.argv[1:]))
    sys.exit(0)
