"""CPU-only: the rule that gives a clip search to its grid form (csrc/search_rule.h, tests/host/search_rule.cpp) against measured
times of both sides."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

# (order, rows, bits, steps the search can take, us without the grid form, us with it)
MEASURED = [
    (1024, 64, 3, 16, 32.9, 19.1), (1024, 64, 3, 0, 12.9, 19.1), (1024, 2048, 3, 16, 45.8, 37.2), (1024, 2048, 4, 12, 34.2, 41.7),
    (1024, 2048, 3, 3, 15.7, 37.2), (1024, 8192, 3, 16, 134, 103), (1024, 8192, 4, 12, 94, 120), (1024, 8192, 3, 0, 29.1, 103),
    (2048, 512, 4, 12, 28.6, 22.8), (2048, 32768, 3, 16, 576, 393), (2048, 32768, 4, 12, 417, 468), (2048, 32768, 3, 0, 75, 393),
    (4096, 1, 4, 3, 12.4, 19.7), (4096, 512, 3, 16, 45.3, 23), (4096, 512, 3, 2, 15.9, 23), (4096, 2048, 3, 0, 26.1, 44),
    (4096, 2048, 3, 7, 75, 44), (4096, 32768, 4, 16, 1030, 546), (4096, 32768, 4, 4, 232, 546), (4096, 32768, 3, 0, 123, 467),
    (8192, 32768, 3, 16, 2155, 703), (8192, 32768, 3, 3, 412, 703), (8192, 8192, 4, 0, 82, 206), (3584, 64, 4, 16, 38, 21.2),
    (3584, 2048, 4, 3, 25.8, 51), (3584, 8192, 3, 16, 291, 137), (3584, 8192, 3, 3, 62, 137), (1536, 2048, 3, 16, 58, 44.2),
    (1536, 2048, 3, 6, 27.3, 44.2), (896, 1, 3, 16, 54, 23.1), (896, 64, 4, 12, 43.1, 58), (896, 512, 4, 3, 21.6, 57),
    (896, 512, 3, 16, 59, 45.5), (896, 2048, 4, 16, 78, 95), (4864, 512, 3, 16, 75, 30.7), (4864, 32768, 4, 7, 775, 1103),
    (4864, 32768, 3, 16, 1429, 916), (5120, 512, 3, 16, 81, 27.9), (5120, 8192, 4, 4, 132, 300), (5120, 32768, 4, 16, 1738, 1178),
    (18944, 512, 3, 16, 153, 35), (18944, 512, 3, 0, 29.5, 35), (18944, 8192, 4, 16, 1459, 365), (18944, 8192, 4, 3, 263, 365),
    (28672, 8192, 3, 16, 2435, 488), (28672, 8192, 3, 0, 287, 488), (28672, 512, 4, 7, 118, 49),
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
