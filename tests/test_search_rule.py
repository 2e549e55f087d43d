"""CPU-only: the rule that gives a clip search to its grid form (csrc/search_rule.h, tests/host/search_rule.cpp) against measured
times of both sides."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

# (order, rows, bits, steps the search can take, us without the grid form, us with it)
MEASURED = [
    (1024, 64, 3, 16, 32.5, 19.1), (1024, 64, 3, 0, 12.4, 17.1), (1024, 2048, 3, 16, 47.1, 38.3), (1024, 2048, 4, 12, 34, 43),
    (1024, 2048, 3, 3, 15.6, 36.3), (1024, 8192, 3, 16, 143, 107), (1024, 8192, 4, 12, 96, 127), (1024, 8192, 3, 0, 29, 104),
    (2048, 512, 4, 12, 28.5, 22.9), (2048, 32768, 3, 16, 590, 429), (2048, 32768, 4, 12, 418, 502), (2048, 32768, 3, 0, 75, 427),
    (4096, 1, 4, 3, 12.1, 18.7), (4096, 512, 3, 16, 46.8, 24.2), (4096, 512, 3, 2, 14, 22), (4096, 2048, 3, 0, 26, 44),
    (4096, 2048, 3, 7, 76, 45), (4096, 32768, 4, 16, 1034, 593), (4096, 32768, 4, 4, 233, 592), (4096, 32768, 3, 0, 121, 526),
    (8192, 32768, 3, 16, 2164, 795), (8192, 32768, 3, 3, 391, 796), (8192, 8192, 4, 0, 80, 218),
    (3584, 64, 4, 16, 37.8, 21.1), (3584, 2048, 4, 3, 24.7, 50.8), (3584, 8192, 3, 16, 301, 148), (3584, 8192, 3, 3, 62, 146),
    (1536, 2048, 3, 16, 61, 45), (1536, 2048, 3, 6, 28, 44), (896, 1, 3, 16, 61, 24), (896, 64, 4, 12, 44, 56), (896, 512, 4, 3, 22, 55),
    (896, 512, 3, 16, 70, 45), (896, 2048, 4, 16, 86, 98), (4864, 512, 3, 16, 84, 32), (4864, 32768, 4, 7, 775, 1093),
    (4864, 32768, 3, 16, 1429, 912), (5120, 512, 3, 16, 94, 29), (5120, 8192, 4, 4, 133, 302), (5120, 32768, 4, 16, 1758, 1174),
    (18944, 512, 3, 16, 169, 40), (18944, 512, 3, 0, 30.5, 37.5), (18944, 8192, 4, 16, 1447, 371), (18944, 8192, 4, 3, 264, 368),
    (28672, 8192, 3, 16, 2443, 484), (28672, 8192, 3, 0, 299, 482), (28672, 512, 4, 7, 117, 49),
]
# order: Sylvester or block, waves of a row held in registers; on the workgroup block kernel rows per pass and threads
SHAPE = {1024: (1, 1, 0, 0), 2048: (1, 2, 0, 0), 4096: (1, 4, 0, 0), 8192: (1, 4, 0, 0), 1536: (0, 1, 0, 0), 3584: (0, 2, 0, 0),
         896: (0, 0, 4, 128), 4864: (0, 0, 2, 320), 5120: (0, 0, 1, 192), 18944: (0, 0, 1, 640), 28672: (0, 0, 1, 896)}


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("rule") / "search_rule")
    subprocess.run([gxx, "-std=c++17", "-O1", os.path.join(HERE, "host", "search_rule.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


LDS = 160 * 1024


def _taken(threads):                                   # the workgroup block kernel's operand buffer
    return (threads // 64 + 1) // 2 * 8192


def _grid(program, cases, lds=LDS):
    lines = []
    for n, rows, bits, steps in cases:
        sylvester, waves, rpp, threads = SHAPE[n]
        lines.append(f"{rows} {n} {bits} {sylvester} {waves} {rpp} {threads} {steps} {lds} {_taken(threads)}")
    run = subprocess.run([program], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=60)
    grid = [int(v) for v in run.stdout.split()]
    assert run.returncode == 0 and len(grid) == len(cases)
    return grid


def test_a_search_takes_the_faster_form(program):
    """coarse or limited searches need one or two passes of a few clip ratios, where the grid form always pays for 511"""
    for case, g in zip(MEASURED, _grid(program, [c[:4] for c in MEASURED])):
        without, with_grid = case[4:]
        assert (with_grid if g else without) <= 1.1 * min(without, with_grid), (case, g)


def test_a_histogram_needs_its_lds(program):
    """a row's histogram takes 24.5 KB (b = 3) or 57 KB of LDS beside the operand buffer: where it does not fit, the other forms
    still do"""
    cases = [(n, 300, bits, 16) for n in (1024, 3584, 5120, 18944, 28672) for bits in (3, 4)]
    need = {(n, bits): {3: 3068, 4: 7156}[bits] * 8 + _taken(SHAPE[n][3]) + 1024 for n, _, bits, _ in cases}
    for lds in (32 * 1024, 64 * 1024, 96 * 1024, LDS):
        fits = [need[n, bits] <= lds for n, _, bits, _ in cases]
        grid = _grid(program, cases, lds)
        assert all(f or not g for f, g in zip(fits, grid)), lds
        if lds == LDS:
            assert all(grid)
    for n, bits in need:                               # to the byte
        assert _grid(program, [(n, 40, bits, 16)], need[n, bits]) == [1] and _grid(program, [(n, 40, bits, 16)], need[n, bits] - 1) == [0]
