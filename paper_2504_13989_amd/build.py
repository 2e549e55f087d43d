"""Build librotq.so (HIP kernels + C ABI) for gfx950 and _pyrotq.so (its Python side) in-tree with hipcc.  The library
itself needs no torch; where torch is not installed the Python side is left out."""
from __future__ import annotations

import importlib.util
import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "librotq.so")
NATIVE_PATH = os.path.join(HERE, "_pyrotq.so")

SOURCES = ["hadamard.cpp", "rotq_api.cpp", "kernels_generic.hip", "kernels_wave.hip", "kernels_wgblock.hip", "kernels_wgrotate.hip", "kernels_wgpair.hip", "kernels_dense.hip", "kernels_ref.hip", "kernels_waveblock2.hip", "kernels_rotate.hip", "kernels_plainasym.hip", "kernels_dequant.hip", "kernels_f64.hip", "kernels_search.hip", "kernels_gridsearch.hip", "kernels_wggrid.hip", "noalloc.hip"]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
    # packed-fp32 VALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-core results go straight to VGPRs (no AGPR copies in the wave kernels)
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    # the first plain parameters of a kernel are in scalar registers when a wave starts (see RQ_WAVE_PARAMS)
    "-mllvm", "-amdgpu-kernarg-preload-count=8",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-attributes",
]


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; the rotq library cannot be built")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 feature; that is harmless
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose and res.stderr.strip():
        print(res.stderr)


def _native_compile(hipcc: str, obj: str):
    """Command that compiles the Python side (host code only) against the installed torch."""
    import sysconfig
    from torch.utils import cpp_extension
    inc = [f"-I{d}" for d in (*cpp_extension.include_paths("cuda"), sysconfig.get_paths()["include"])]
    return [hipcc, "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-DUSE_ROCM", *inc, "-Wno-unused-command-line-argument",
            "-c", "-x", "hip", "--cuda-host-only", os.path.join(CSRC, "pyrotq.cpp"), "-o", obj]


def _native_link(hipcc: str, obj: str, out: str):
    from torch.utils import cpp_extension
    dirs = [f"-L{d}" for d in cpp_extension.library_paths("cuda")]
    return [hipcc, "-shared", "-fPIC", obj, "-o", out, f"-L{HERE}", "-l:librotq.so", *dirs, "-ltorch_python", "-ltorch",
            "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]


def build_library(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source to an object (a few at a time), then link the library and the Python side."""
    hipcc = hipcc_path()
    compile_flags = [f for f in FLAGS if f != "-shared"]
    python_side = importlib.util.find_spec("torch") is not None
    with tempfile.TemporaryDirectory(prefix="rotq_build_") as tmpdir:
        objs = [os.path.join(tmpdir, os.path.splitext(s)[0] + ".o") for s in SOURCES]
        jobs = [[hipcc, *compile_flags, *extra_flags, "-c", "-x", "hip", os.path.join(CSRC, s), "-o", o]
                for s, o in zip(SOURCES, objs)]
        pyobj = os.path.join(tmpdir, "pyrotq.o")
        with ThreadPoolExecutor(max_workers=min(len(jobs) + 1, 6)) as pool:
            native = pool.submit(lambda: _run(_native_compile(hipcc, pyobj), verbose)) if python_side else None
            list(pool.map(lambda c: _run(c, verbose), jobs))
        tmp = LIB_PATH + ".tmp"
        _run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", tmp], verbose)
        os.replace(tmp, LIB_PATH)
        if native is None:
            print("torch is not installed: librotq.so built, its Python side (_pyrotq.so) left out")
            return LIB_PATH
        native.result()
        tmp = NATIVE_PATH + ".tmp"
        _run(_native_link(hipcc, pyobj, tmp), verbose)
        os.replace(tmp, NATIVE_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
