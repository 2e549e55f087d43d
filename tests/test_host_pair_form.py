"""CPU-only: the workgroup block kernel where the LDS of its pair form cannot be had (tests/host/pair_form_without_lds.cpp)."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2504_13989_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_block_kernel_does_not_need_the_lds_of_its_pair_form(tmp_path):
    # (an incomplete handle comes from the product's own sources, host side only)
    sources = [os.path.join(build.CSRC, s) for s in ("kernels_wgblock.hip", "kernels_wgpair.hip", "kernels_wgrotate.hip", "hadamard.cpp")]
    sources.append(os.path.join(HERE, "host", "pair_form_without_lds.cpp"))
    objs = [str(tmp_path / f"{i}.o") for i in range(len(sources))]
    hipcc = build.hipcc_path()

    def compile_one(pair):
        subprocess.run([hipcc, "-std=c++17", "-O1", "-w", "-fPIC", "--cuda-host-only", "-c", "-x", "hip", pair[0], "-o", pair[1]], check=True,
                       capture_output=True)
    with ThreadPoolExecutor(4) as pool:
        list(pool.map(compile_one, zip(sources, objs)))
    exe = str(tmp_path / "pair_form_without_lds")
    subprocess.run(["g++", *objs, "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True, capture_output=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
    assert run.stdout.split("\n")[:-1] == ["18944 1 1", "20480 1 1", "18944 1 0", "20480 1 0"], run.stdout
