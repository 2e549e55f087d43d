"""GPU: the grid form of the clip search (every probe down to a bracket of 1 / 256 evaluated at once, from a histogram of each
row): its values against quant_error's and against 64 bits, its steps against Algorithm 1 run on them, on every rotation it has;
the ends of its range; rows that are not finite, zero or tiny; many searches on two streams."""
import numpy as np
import pytest

import parity
import rotq_oracle as oracle
from paper_2504_13989_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


def _check(h, x, b, eps, result):
    clip, mse, trace = result
    seen = dict(trace)
    m, fm, otrace = oracle.gbs_search(lambda c: seen[np.float32(c)], eps)
    assert [np.float32(c) for c, _ in otrace] == [np.float32(c) for c, _ in trace]
    assert clip == np.float32(m) and mse == fm
    # both are sums of fp32 squares or better: a few 1e-7 apart
    want = binding.quant_error(h, x, b, [c for c, _ in trace]).cpu().numpy()
    assert np.allclose([v for _, v in trace], want, rtol=2e-6, atol=0.0)


# one wave a row, two, four, blocks of one and two waves; the workgroup block kernel's block rows of 128, 64 and 32 columns,
# one wave to sixteen; padded rows; one row, one more than the compute units, one more than two of each
@pytest.mark.parametrize("n,d,rows", [(1024, 1000, 257), (2048, 2048, 513), (4096, 4096, 1), (8192, 8192, 300), (1536, 1536, 70),
                                      (3584, 3584, 513), (3072, 3000, 31), (5120, 5120, 258), (18944, 18944, 3), (28672, 28672, 2),
                                      (8960, 8960, 515), (4864, 4864, 5), (896, 896, 1023), (896, 896, 1), (11264, 11008, 40),
                                      (384, 384, 2), (32768, 32768, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_grid_search_takes_the_steps_of_algorithm_1(n, d, rows, dtype):
    rng = np.random.default_rng(n + rows)
    xf = rng.standard_normal((rows, d)).astype(np.float32)
    xf[rows // 2] *= 20.0
    x = parity.to_device(wl.f32_to_bf16_bits(xf) if dtype == "bf16" else xf.astype(np.float16))
    h = binding.hadamard_build(n)
    for b in (3, 4):
        for eps in (1.0 / 256, 1.0 / 100):
            got = binding.gbs_search(h, x, b, eps)
            assert h.last_kernel == "grid_search"
            _check(h, x, b, float(np.float32(eps)), got)
            assert binding.gbs_search(h, x, b, eps) == got
        full = binding.gbs_search(h, x, b, 1.0 / 256)
        short = binding.gbs_search(h, x, b, 1.0 / 256, max_evals=14)
        assert h.last_kernel == "grid_search" and short[2] == full[2][:14]


def test_ends_of_the_grids_range():
    rng = np.random.default_rng(3)
    x = parity.to_device(wl.f32_to_bf16_bits(rng.standard_normal((300, 5120)).astype(np.float32)))
    h = binding.hadamard_build(5120)
    for eps, grid in ((1.0 / 256, True), (np.nextafter(np.float32(1.0 / 256), np.float32(0)), False), (1.0 / 128, True), (1e-6, False)):
        got = binding.gbs_search(h, x, 3, float(eps))
        assert (h.last_kernel == "grid_search") == grid
        _check(h, x, 3, float(eps), got)
    # without pinned memory the results are copied back
    want = binding.gbs_search(h, x, 3, 1.0 / 256)
    h.set_variant(7)
    assert binding.gbs_search(h, x, 3, 1.0 / 256) == want and h.last_kernel == "grid_search"


def _rows(kind, rows, d, rng):
    if kind == "constant":                             # one coefficient holds all of the energy
        return np.full((rows, d), 1.5, np.float32)
    if kind == "impulse":                              # every coefficient as large as the largest
        x = np.zeros((rows, d), np.float32)
        x[np.arange(rows), rng.integers(0, d, rows)] = 3.0
        return x
    if kind == "normal":
        return rng.standard_normal((rows, d)).astype(np.float32)
    x = rng.standard_t(3, (rows, d))                   # heavy tails, outlier channels, a row that outweighs the others
    x[:, rng.permutation(d)[:8]] *= 50.0
    x[rows // 2] *= 500.0
    return x.astype(np.float32)


@pytest.mark.parametrize("n,d,rows", [(1024, 1024, 40), (2048, 2000, 33), (4096, 4096, 300), (8192, 8192, 9), (1536, 1536, 20), (3584, 3584, 40),
                                      (896, 896, 70), (4864, 4864, 9), (5120, 5120, 20), (18944, 18944, 6)])
@pytest.mark.parametrize("kind", ["normal", "tails", "constant", "impulse"])
def test_values_against_64_bits(n, d, rows, kind):
    rng = np.random.default_rng(n + rows)
    xf = _rows(kind, rows, d, rng)
    bits = wl.f32_to_bf16_bits(xf)
    h = binding.hadamard_build(n)
    x = parity.to_device(bits)
    wide = parity.to_device(np.concatenate([bits, bits[:, ::-1], bits], axis=1))       # the middle of a wider tensor
    wide[:, d:2 * d] = x
    # log2 n fp32 additions lead to a value, each rounded by up to 2^-25 of it (uniform: over the square root of 3); where one value or
    # one row sets the error nothing averages that out, and the square doubles it; four standard deviations, and
    # the fp32 result's own rounding (measured: 4.3e-7 at most over these rows and others, rms 2e-8 - 2.1e-7)
    tol = 4 * 2 * 2.0 ** -25 * np.sqrt(np.log2(n) / 3) + 2.0 ** -24
    for b in (3, 4):
        got = binding.gbs_search(h, x, b, 1.0 / 256)
        assert h.last_kernel == "grid_search"
        assert binding.gbs_search(h, wide[:, d:2 * d], b, 1.0 / 256) == got and h.last_kernel == "grid_search"
        clips = np.array([c for c, _ in got[2]], np.float32)
        want = oracle.quant_error(bits, n, b, clips)
        rel = np.array([v for _, v in got[2]], np.float64) / want - 1.0
        assert np.abs(rel).max() <= tol, (b, np.abs(rel).max())


@pytest.mark.parametrize("n,rows,kernel", [(4096, 40, "gbs_resident"), (1024, 2048, "gbs_resident"), (4096, 2048, "wave_quant_error"),
                                           (3584, 2500, "wave_quant_error"), (896, 700, "wg_block_quant_error"),
                                           (4864, 1500, "wg_block_quant_error"), (18944, 600, "wg_block_quant_error")])
def test_searches_of_few_steps_evaluate_few_ratios(n, rows, kernel):
    """a coarse or limited search needs one or two passes of a few clip ratios: the form for that, with Algorithm 1's steps"""
    rng = np.random.default_rng(n)
    x = parity.to_device(wl.f32_to_bf16_bits(rng.standard_normal((rows, n)).astype(np.float32)))
    h = binding.hadamard_build(n)
    full = binding.gbs_search(h, x, 3, 1.0 / 256)
    assert h.last_kernel == "grid_search"
    for eps, limit in ((0.9, 64), (2.0, 64), (0.5, 64), (1.0 / 256, 1), (1.0 / 256, 3)):
        got = binding.gbs_search(h, x, 3, eps, max_evals=limit)
        assert h.last_kernel == kernel or (kernel == "gbs_resident" and h.last_kernel == "gbs_stepped")
        if eps < 0.5:
            assert [c for c, _ in got[2]] == [c for c, _ in full[2][:limit]]
            assert np.allclose([v for _, v in got[2]], [v for _, v in full[2][:limit]], rtol=2e-6, atol=0.0)
        else:
            _check(h, x, 3, eps, got)


@pytest.mark.parametrize("n", [4096, 1536, 5120, 896])
def test_rows_that_are_not_finite_zero_or_tiny(n):
    rng = np.random.default_rng(n)
    xf = rng.standard_normal((9, n)).astype(np.float32)
    h = binding.hadamard_build(n)
    base = xf.copy()
    for what in ("zero", "tiny", "inf", "nan", "over"):
        xf = base.copy()
        xf[4] = {"zero": 0.0, "tiny": xf[4] * np.float32(1e-36), "inf": xf[4], "nan": xf[4], "over": xf[4] * np.float32(5e37)}[what]
        if what in ("inf", "nan"):
            xf[4, 7] = np.inf if what == "inf" else np.nan
        x = parity.to_device(wl.f32_to_bf16_bits(xf))
        clip, mse, trace = got = binding.gbs_search(h, x, 4, 1.0 / 256)
        assert h.last_kernel == "grid_search"
        if what in ("zero", "tiny"):
            _check(h, x, 4, 1.0 / 256, got)
        else:
            want = binding.quant_error(h, x, 4, [c for c, _ in trace]).cpu().numpy()
            assert np.isnan(mse) and all(np.isnan(v) for _, v in trace) and np.isnan(want).all() and clip == 0.5


def test_many_searches_on_two_streams_in_turn():
    """nothing but the searches' own memory orders them"""
    import torch
    rng = np.random.default_rng(10)
    xs = [parity.to_device(wl.f32_to_bf16_bits(rng.standard_normal((r, 4096)).astype(np.float32))) for r in (900, 33)]
    h = binding.hadamard_build(4096)
    want = [binding.gbs_search(h, x, 3, 1.0 / 256) for x in xs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for i in range(300):
        assert binding.gbs_search(h, xs[i % 2], 3, 1.0 / 256, stream=streams[i % 3 % 2]) == want[i % 2], i
        assert h.last_kernel == "grid_search"
