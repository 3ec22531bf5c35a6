"""Builds liblutkan.so (host LUT compiler + gfx950 kernels) in-tree with hipcc, and beside it the binding's forward calls as a
CPython module (_lutkan_call.*.so, host code against torch's headers), which the library does not need."""
from __future__ import annotations

import os
import subprocess
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.environ.get("LUTKAN_LIBRARY", os.path.join(HERE, "liblutkan.so"))
CALL_SOURCE = os.path.join(CSRC, "lutkan_call.cpp")
SOURCES = [os.path.join(CSRC, "lutkan_compile.cpp"), os.path.join(CSRC, "lutkan_kernels.hip"),
           os.path.join(CSRC, "bspline_kernels.hip"), os.path.join(CSRC, "lutkan_probes.hip"),
           os.path.join(CSRC, "lutkan_stats.hip"), os.path.join(CSRC, "lutkan_base_gemm.hip"),
           os.path.join(CSRC, "bspline_matrix.hip"), os.path.join(CSRC, "lutkan_narrow.hip"),
           os.path.join(CSRC, "lutkan_rows.hip")]
HEADERS = [os.path.join(CSRC, "lutkan_internal.h"), os.path.join(CSRC, "lutkan_device.h"), os.path.join(CSRC, "lutkan_pieces.h"),
           os.path.join(CSRC, "bspline_matrix.h"), os.path.join(CSRC, "lutkan_locate.h"), os.path.join(CSRC, "lutkan_narrow.h"), os.path.join(CSRC, "lutkan_rows.h"),
           os.path.join(ROOT, "include", "lutkan.h")]

# -ffp-contract=off: the index arithmetic of the locate kernel and the host quantiser must round once per
#   operation; fused multiply-adds in the edge kernels are written explicitly.
# -packed-fp32-ops is switched off: the packed fp32 VALU forms are not used by this library.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-Wno-inline-asm",      # the LDS-DMA helper names M0 in its clobber list on purpose (see lutkan_device.h)
]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(p) > t for p in SOURCES + HEADERS)


def call_module() -> str:
    """Where the CPython module of these sources for this interpreter and this torch lies, built or not: it reads structures of both, so
    that a module of other sources, another Python or another torch must not be taken for it."""
    import hashlib
    import sysconfig
    import torch
    digest = hashlib.sha256()
    for path in (CALL_SOURCE, os.path.join(ROOT, "include", "lutkan.h")):
        with open(path, "rb") as f:
            digest.update(f.read())
    return os.path.join(HERE, f"_lutkan_call.{digest.hexdigest()[:12]}.torch-{torch.__version__}{sysconfig.get_config_var('EXT_SUFFIX')}")


def build_call(verbose: bool = False) -> str:
    """The CPython module, complete under its name or not there at all.  torch's libraries are named, not searched for at run time: the
    binding imports torch before the module."""
    import sysconfig
    import tempfile
    import torch
    path, torch_dir = call_module(), os.path.dirname(torch.__file__)
    handle, unfinished = tempfile.mkstemp(prefix=".lutkan_call.", suffix=".so", dir=os.path.dirname(path))
    os.close(handle)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", os.path.join(ROOT, "include")]
    for include in (os.path.join(torch_dir, "include"), os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"]):
        cmd += ["-isystem", include]
    cmd += [CALL_SOURCE, "-o", unfinished, "-L" + os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        subprocess.run(cmd, check=True)
        os.chmod(unfinished, 0o755)
        os.replace(unfinished, path)
    finally:
        if os.path.exists(unfinished):
            os.unlink(unfinished)
    return path


def build(verbose: bool = False) -> str:
    """The library; then the module, without which (no torch, no g++) the binding works and says so."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def compile_one(src: str) -> str:
        obj = os.path.splitext(src)[0] + ".o"
        cmd = [hipcc] + HIPCC_FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
        if src.endswith(".hip"):
            cmd += ["-x", "hip"]
        cmd += ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    # the translation units are independent: one compiler process each (lutkan_kernels.hip is the long one)
    with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, os.cpu_count() or 1, 8)) as pool:
        call = pool.submit(build_call, verbose)
        objs = list(pool.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs + ["-lpthread"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    try:
        call.result()
    except Exception as error:
        warnings.warn(f"_lutkan_call was not built ({type(error).__name__}: {error}); {LIB} was", RuntimeWarning)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
