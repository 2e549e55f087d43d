"""GPU parity of rq_rotate and rq_dequantize_rotate on the block orders (one-wave and workgroup kernels) against
the oracle: every number of contraction steps, symmetric and unsymmetric blocks, several rows per pass with a
ragged end, zero-padded input, narrowed output, every input / output type, both directions."""
import numpy as np
import pytest
import torch

import parity
import rotq_oracle as oracle
from paper_2504_13989_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

# (order, input width, output width, rows, kernel): blocks x columns 12 x 128, 28 x 128, 20 x 256 (40), 44 x 256 (88),
# 108 x 128, 148 x 128, 44 x 512 (176), 28 x 1024 (224), H_128 x 128; several rows per pass: 28 x 32, 76 x 64, 140 x 64
SHAPES = [(1536, 1536, 1536, 3, "wave_block"), (3584, 3584, 3000, 9, "wave_block"), (5120, 5000, 5120, 5, "wg_block"),
          (11264, 11008, 11008, 5, "wg_block"), (13824, 13824, 13824, 3, "wg_block"), (18944, 18944, 18944, 4, "wg_block"),
          (22528, 22528, 20000, 3, "wg_block"), (28672, 28672, 28672, 2, "wg_block"), (16384, 16384, 16384, 2, "wg_block"),
          (896, 896, 896, 9, "wg_block"), (4864, 4800, 4856, 5, "wg_block"), (8960, 8960, 8960, 3, "wg_block")]


def _close(got, want, out_dtype, what):
    amax = np.abs(want).max(axis=1, keepdims=True)
    # fp32 sums: 1e-5 of the row's maximum; one rounding to the output format on top
    step = {"f32": 0.0, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[out_dtype]
    err = np.abs(got.double().cpu().numpy() - want)
    assert np.all(err <= 1e-5 * amax + step * np.abs(want) + (6.2e-5 if out_dtype == "f16" else 0.0)), f"{what}: {err.max()}"


@pytest.mark.parametrize("n,d,d_out,rows,kernel", SHAPES)
def test_rotate(n, d, d_out, rows, kernel):
    import torch
    types = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
    rng = np.random.default_rng(n + rows)
    h = binding.hadamard_build(n)
    for i, (in_dtype, out_dtype) in enumerate([("bf16", "bf16"), ("f16", "f16"), ("bf16", "f32"), ("f16", "f32")]):
        xf = rng.standard_normal((rows, d + 8)).astype(np.float32)
        full = wl.f32_to_bf16_bits(xf) if in_dtype == "bf16" else xf.astype(np.float16)
        x = np.ascontiguousarray(full[:, :d])
        for transpose in (False, True):
            if transpose:
                xp = np.zeros((rows, n))
                xp[:, :d] = oracle.as_f64(x)
                want = oracle.rotate_back(xp, n)
            else:
                want = oracle.rotate(x, n)
            buf = torch.full((rows + 1, d_out + 8), 7.0, dtype=types[out_dtype], device="cuda")
            binding.rotate(h, parity.to_device(full)[:, :d], transpose=transpose, d_out=d_out, out=buf[:rows, :d_out])
            torch.cuda.synchronize()
            assert h.last_kernel == f"{kernel}_rotate"
            _close(buf[:rows, :d_out], want[:, :d_out], out_dtype, f"n={n} {in_dtype}->{out_dtype} transpose={transpose}")
            assert bool((buf[:, d_out:] == 7.0).all()) and bool((buf[rows:] == 7.0).all())


@pytest.mark.parametrize("b", [3, 4])
@pytest.mark.parametrize("n,d,d_out,rows,kernel", SHAPES)
def test_dequantize_rotate(n, d, d_out, rows, kernel, b):
    import torch
    types = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
    rng = np.random.default_rng(n + rows + b)
    h = binding.hadamard_build(n)
    q = rng.integers(-(2 ** (b - 1)), 2 ** (b - 1), size=(rows, n))
    scales = rng.uniform(0.5, 2.0, size=rows).astype(np.float32)
    packed = torch.from_numpy(oracle.pack_codes(q, b)).cuda()
    y = oracle.dequantize(q, scales.astype(np.float64))
    for transpose in (True, False):
        want = oracle.rotate_back(y, n) if transpose else oracle.rotate(y, n)
        for out_dtype in ("bf16", "f16", "f32"):
            buf = torch.full((rows + 1, d_out + 8), 7.0, dtype=types[out_dtype], device="cuda")
            binding.dequantize_rotate(h, packed, torch.from_numpy(scales).cuda(), b, transpose=transpose, d_out=d_out,
                                      out=buf[:rows, :d_out])
            torch.cuda.synchronize()
            assert h.last_kernel == f"{kernel}_dequant_rotate"
            _close(buf[:rows, :d_out], want[:, :d_out], out_dtype, f"n={n} b={b} ->{out_dtype} transpose={transpose}")
            assert bool((buf[:, d_out:] == 7.0).all()) and bool((buf[rows:] == 7.0).all())


@pytest.mark.parametrize("n", [896, 3584, 4864, 5120, 8960, 16384, 18944, 28672])
def test_fp32_results_are_rounded_once(n):
    """Error of fp32 results against 64 bits, 2-norm.  One rounding to nearest is uniform within 2^-24 of a value at most:
    2^-24 / sqrt(3).  From codes the sums are exact integers; from 16-bit rows the partial sums of a block stay within 24
    bits but for rare small terms.  With fp32 stages behind the block, rows have 3.7e-8 (896) to 7.4e-8 (13824)."""
    import torch
    rng = np.random.default_rng(n)
    h = binding.hadamard_build(n)
    bound = 2.0 ** -24 / 3 ** 0.5

    def rel(got, want):
        return np.linalg.norm(got.double().cpu().numpy() - want) / np.linalg.norm(want)

    q = rng.integers(-4, 4, size=(16, n))
    scales = rng.uniform(0.5, 2.0, size=16).astype(np.float32)
    got = binding.dequantize_rotate(h, torch.from_numpy(oracle.pack_codes(q, 3)).cuda(), torch.from_numpy(scales).cuda(), 3)
    assert rel(got, oracle.rotate_back(oracle.dequantize(q, scales.astype(np.float64)), n)) <= bound
    if n != 3584:                                       # (one-wave kernel: fp32 stages)
        x = rng.standard_normal((16, n)).astype(np.float16)
        for transpose in (False, True):
            want = oracle.rotate_back(oracle.as_f64(x), n) if transpose else oracle.rotate(x, n)
            assert rel(binding.rotate(h, parity.to_device(x), transpose=transpose), want) <= bound


@pytest.mark.parametrize("n", [3584, 4864, 18944])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_16_bit_results_of_codes_take_their_factor_rounded_once(n, dtype):
    """scale / sqrt(n) is formed in fp64 and rounded once.  Rows of a single code 1 have that factor as every result; the
    scales are ones for which 1 / sqrt(n) in fp32 times the scale in fp32 falls to the other side of a rounding boundary of
    the 16-bit type (a few in a million)"""
    inv = 1.0 / np.sqrt(np.float64(n))
    scales = torch.rand(1 << 24, generator=torch.Generator().manual_seed(n), dtype=torch.float32) + 0.5
    once = (scales.double() * inv).to(torch.float32).to(dtype)
    twice = (scales * torch.tensor(inv, dtype=torch.float32)).to(dtype)
    scales, want = scales[once != twice][:64], once[once != twice][:64]
    assert len(scales) >= 3
    h = binding.hadamard_build(n)
    for b in (3, 4):
        codes = torch.zeros((len(scales), n * b // 8), dtype=torch.uint8, device="cuda")
        codes[:, 0] = 1
        y = binding.dequantize_rotate(h, codes, scales.cuda(), b, out_dtype=dtype)
        assert h.last_kernel in ("wave_block_dequant_rotate", "wg_block_dequant_rotate")
        assert torch.equal(y.abs().cpu(), want[:, None].expand(-1, n))


@pytest.mark.parametrize("n", [896, 4864, 8960, 11264, 13824, 18944])
@pytest.mark.parametrize("out", [torch.float32, torch.bfloat16])
def test_infinities_of_the_last_block_rows(n, out):
    """one infinity in a row makes every result an infinity of its own sign, as on the general kernel; NaN makes every
    result NaN"""
    h = binding.hadamard_build(n)
    x = torch.randn((6, n), generator=torch.Generator().manual_seed(n)).to(torch.bfloat16)
    for i, at in enumerate((0, n // 2, n - 1, n - 130, n - 520)):
        x[i, at] = float("inf") if i % 2 else -float("inf")
    x[5, n - 1] = float("nan")
    x = x.cuda()
    y = binding.rotate(h, x, out_dtype=out)
    assert h.last_kernel == "wg_block_rotate"
    h.set_variant(1)
    want = binding.rotate(h, x, out_dtype=out)
    assert torch.isinf(want[:5]).all() and torch.isnan(y[5]).all()
    assert torch.equal(y[:5], want[:5])


@pytest.mark.parametrize("b", [3, 4])
@pytest.mark.parametrize("n", [1536, 2560, 3072, 3584, 8960, 11264, 14336])
def test_each_code_at_each_place_of_a_chunk(n, b):
    """Rows with a single code that is not 0, every code at every place of a chunk, in even and odd block rows: each result is
    code * scale / sqrt(n) up to its sign, with the factor formed in fp64 and rounded once - exactly, since the sums are integers."""
    columns = 128 if n != 8960 else 64
    h = binding.hadamard_build(n)
    places = [(0, 0), (1, 16), (2, 8), (n // columns - 1, columns - 8), (n // columns - 2, 0)]    # block row, first column of a chunk
    values = [c for c in range(-(2 ** (b - 1)), 2 ** (b - 1)) if c]
    rows = [(r * columns + c + i, v) for r, c in places for i in range(8) for v in values]
    q = np.zeros((len(rows), n), dtype=np.int64)
    for k, (at, v) in enumerate(rows):
        q[k, at] = v
    scales = torch.rand(len(rows), generator=torch.Generator().manual_seed(n + b), dtype=torch.float32) + 0.5
    packed = torch.from_numpy(oracle.pack_codes(q, b)).cuda()
    code = torch.tensor([v for _, v in rows], dtype=torch.float64)
    signs = torch.from_numpy(np.sign(oracle.rotate(np.eye(n)[[at for at, _ in rows[::len(values)]]], n))).repeat_interleave(len(values), 0)
    for dtype in (torch.bfloat16, torch.float16):
        k = (scales.double() / np.sqrt(np.float64(n))).to(torch.float32)
        want = (code.to(torch.float32) * k).to(dtype)
        got = binding.dequantize_rotate(h, packed, scales.cuda(), b, transpose=False, out_dtype=dtype).cpu()
        assert torch.equal(got, (want[:, None].double() * signs).to(dtype))
    want = (code * (scales.double() / np.sqrt(np.float64(n)))).to(torch.float32)
    got = binding.dequantize_rotate(h, packed, scales.cuda(), b, transpose=False, out_dtype=torch.float32).cpu()
    assert torch.equal(got, (want[:, None].double() * signs).to(torch.float32))
