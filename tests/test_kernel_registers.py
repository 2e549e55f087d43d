"""CPU-only: registers of the built kernels, from the metadata in the library's own code objects."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2504_13989_amd import binding

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    """The gfx950 code objects embedded in librotq.so, one per source file."""
    data = open(binding.LIB_PATH, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, id_len = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + id_len]
            pos += 24 + id_len
            if b"gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """kernel symbol -> vector registers, of them spilled"""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not found")
    binding.lib()
    path = str(tmp_path_factory.mktemp("co") / "a.co")
    found = {}
    for obj in _code_objects():
        with open(path, "wb") as f:
            f.write(obj)
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.a", notes):
            name = re.search(r"\.symbol:\s+(\S+)\.kd", kernel)
            count = re.search(r"\.vgpr_count:\s+(\d+)", kernel)
            spilled = re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel)
            if name and count and spilled:
                found[name.group(1)] = int(count.group(1)), int(spilled.group(1))
    return found


@pytest.fixture(scope="module")
def spills(kernels):
    """kernel symbol -> vector registers spilled"""
    return {k: v[1] for k, v in kernels.items()}


def _waves(kernels, pattern):
    """template arguments of the kernels whose symbols match -> waves that a SIMD holds (512 registers a lane, in eights)"""
    found = {}
    for k, (count, spilled) in kernels.items():
        m = re.search(pattern, k)
        if m:
            assert spilled == 0, k
            found[tuple(map(int, m.groups()))] = min(8, 512 // (-(-count // 8) * 8))
    return found


def test_quantizing_workgroup_block_kernels_hold_their_registers(spills):
    """A spilled operand tile or accumulator is a trip to memory in every pass: with 23 registers spilled the kernel of
    8960-wide rows took 1.4 times as long as with 10.  The few spills there are (3 of 80) were measured as they are."""
    forms = {k: v for k, v in spills.items() if re.search(r"k_wg_blockILi\d+ELi[34]ELb[01]ELi0E", k)}
    assert len(forms) >= 100
    assert max(forms.values()) <= 3, sorted(forms.items(), key=lambda kv: -kv[1])[:8]


def test_pair_form_of_the_workgroup_block_kernel_holds_its_registers(spills):
    """128 registers with 64 accumulators: 10 to 14 spilled cost 28672-wide rows, b = 4, a twentieth of their time."""
    forms = {k: v for k, v in spills.items() if "k_wg_pair" in k}
    assert len(forms) == 7 * 2 * 2
    assert max(forms.values()) <= 1, sorted(forms.items(), key=lambda kv: -kv[1])[:8]


def test_rotating_workgroup_block_kernels_hold_their_registers(spills):
    """29 registers spilled made the rotation of 28672-wide rows to fp32 1.3 times as long.  (Blocks of 225 to 256 with fp32
    results spill 20 to 24, measured as they are.)"""
    forms = {k: v for k, v in spills.items() if re.search(r"k_wg_blockILi\d+ELi[34]ELb[01]ELi2E", k)}
    assert len(forms) >= 100
    for kk, most in ((range(1, 8), 4), (range(8, 9), 24)):
        some = {k: v for k, v in forms.items() if int(re.search(r"k_wg_blockILi(\d+)E", k).group(1)) in kk}
        assert max(some.values()) <= most, sorted(some.items(), key=lambda kv: -kv[1])[:8]


def test_grid_search_kernels_hold_their_registers(spills):
    """The clip search's grid kernels, which keep a row for the passes over its histogram.  Rows held by single waves and the passes
    of one row spill nothing; several rows per pass are measured as they are (with the operand tiles held for the whole launch they spill 17 - 35, and
    one row per pass 6 - 14 beyond blocks of 160: 512 rows of 28672 then take 55.2 us a search and not 51.3)."""
    rows = {k: v for k, v in spills.items() if "k_grid_rows" in k}
    assert len(rows) == 24 and max(rows.values()) == 0
    forms = {k: v for k, v in spills.items() if re.search(r"k_wg_blockILi\d+ELi[34]ELb0ELi3E", k)}
    assert len(forms) == 92
    for k, v in forms.items():
        kk, cb = map(int, re.search(r"k_wg_blockILi(\d+)ELi[34]ELb0ELi3ELi(\d)E", k).groups())
        assert v <= (0 if cb == 4 else 28 if kk == 1 else 10), (k, v)


def test_row_kernels_of_block_orders_hold_their_waves(kernels):
    """One wave a row, so the waves on a SIMD are the rows in flight: with two and not three of them 33600 rows of 5120, b = 4,
    took 83.6 us and not 76.0, with four and not six 67200 rows of 2560 74.7 and not 69.9."""
    waves = _waves(kernels, r"k_wave_blockILi([34])ELb([01])ELi(\d+)ELb([01])EE")
    assert len(waves) == 2 * 2 * 7 * 2
    for (bits, full, nv, f16), w in waves.items():
        want = {2: 7, 3: 7, 4: 7, 5: 6, 6: 5 if bits == 3 else 4, 7: 5 if bits == 3 else 4, 8: 4}[nv] if full else \
            {2: 6, 3: 6, 4: 6, 5: 6, 6: 5, 7: 4, 8: 4}[nv]
        assert w >= want, (bits, full, nv, f16, w)
    waves = _waves(kernels, r"k_wave_block2ILi([34])ELb([01])ELi(\d+)ELb([01])EE")
    assert len(waves) == 2 * 2 * 8 * 2
    for (bits, full, nv, f16), w in waves.items():
        assert w >= (3 if full and nv <= 12 else 2), (bits, full, nv, f16, w)


def test_short_row_kernels_hold_their_waves(kernels):
    """Several rows a wave.  655360 unrotated rows of 96 took 40.2 us with five waves a SIMD and 36.1 with six, 122880 of 512
    29.3 with four and 27.8 with five; of rotated rows of 128, b = 4, short launches have six and long ones five."""
    waves = _waves(kernels, r"k_plain_shortILi([34])ELi([012])ELi(\d+)ELi4EE")
    assert len(waves) == 2 * 3 * 3 and min(waves.values()) >= 6, waves
    waves = _waves(kernels, r"k_wave_shortILi([234])ELi([34])ELb([01])ELb[01]ELb([01])ELb([01])EE")
    assert len(waves) == 6 + 6 + 2 + 1, waves
    for (cb, bits, asym, plain, carried), w in waves.items():
        want = (5 if cb == 4 else 4) if plain else 6 if cb == 4 or (bits == 4 and cb == 2 and carried) else 5
        assert w >= want, (cb, bits, asym, plain, carried, w)
