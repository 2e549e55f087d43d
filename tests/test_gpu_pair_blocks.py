"""GPU: rows of the orders whose block splits into pairs of rows, enough of them for the form of the workgroup block kernel
that uses it, against the same rows a few at a time (the other form, which the oracle's tests cover) and against the oracle."""
import numpy as np
import pytest
import torch

import parity
from paper_2504_13989_amd import binding

pytestmark = pytest.mark.gpu

# five waves a row with and without a diagonal, six, four, seven with and without, eight
ORDERS = [148 * 128, 160 * 128, 192 * 128, 112 * 128, 128 * 128, 196 * 128, 204 * 128, 224 * 128, 256 * 128]


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n", ORDERS)
def test_many_rows_against_few(n, dtype, bits):
    # more than two rows a compute unit, in rounds that end unevenly; a padded width and a leading dimension beyond it
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows, d = 3 * cus + 5, n - 136 if bits == 3 else n
    gen = torch.Generator(device="cuda").manual_seed(n + bits)
    wide = torch.randn((rows, d + 40), generator=gen, device="cuda")
    wide[:, torch.randperm(d, generator=gen, device="cuda")[:5]] *= 40
    wide[3] = 0
    wide[rows - 2, d // 2] = float("inf")
    wide[7, 130] = -float("inf")
    wide[cus, 5] = float("nan")
    x = wide.to(dtype)[:, :d]
    h = binding.hadamard_build(n)
    codes, scales = binding.rotate_quantize(h, x, bits, 0.9)
    few = [binding.rotate_quantize(h, x[i:i + cus], bits, 0.9) for i in range(0, rows, cus)]
    want, wscales = (torch.cat([f[k] for f in few]) for k in (0, 1))
    odd = torch.tensor([3, 7, cus, rows - 2], device="cuda")
    assert torch.equal(codes[odd], want[odd]) and torch.equal(scales[odd].view(torch.int32), wscales[odd].view(torch.int32))
    # each form sums up to 256 values to a maximum of about 256^(1/2) times theirs, and adds for seven stages, in fp32: a few units of
    # 2^-24 of the largest value, which a code's boundary is as near as in one value of 10^5
    keep = torch.ones(rows, dtype=torch.bool, device="cuda")
    keep[odd] = False
    assert ((scales[keep] / wscales[keep] - 1).abs() < 16 * 2.0 ** -24).all()
    differ = codes[keep] != want[keep]
    assert differ.float().mean().item() < 2e-5
    # the oracle on a few rows
    some = [0, cus - 1, rows - 1]
    xs = x[some].contiguous()
    got = xs.view(torch.int16).cpu().numpy().view(np.uint16) if dtype == torch.bfloat16 else xs.cpu().numpy()
    if n <= 20480:                                       # (the dense matrix of the wider orders is too large here)
        parity.check_rotate_quantize(got, n, bits, 0.9, codes[some].cpu().numpy(), scales[some].cpu().numpy(), f"pairs n={n} b={bits}")


@pytest.mark.parametrize("d", [8, 1000, 1784, 1792])
@pytest.mark.parametrize("n", [148 * 128, 112 * 128, 224 * 128])
def test_many_narrow_rows(n, d):
    """Rows far narrower than the order, in a tensor whose other columns must not be seen: the rows' block rows from the first, the eighth
    and the fourteenth on lie beyond the width."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 3 * cus + 5
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    wide = torch.full((rows, d + 4096), 3e4, device="cuda", dtype=torch.bfloat16)
    wide[:, :d] = torch.randn((rows, d), generator=gen, device="cuda")
    h = binding.hadamard_build(n)
    codes, scales = binding.rotate_quantize(h, wide[:, :d], 4, 0.9)
    few = [binding.rotate_quantize(h, wide[i:i + cus, :d], 4, 0.9) for i in range(0, rows, cus)]
    want, wscales = (torch.cat([f[k] for f in few]) for k in (0, 1))
    assert ((scales / wscales - 1).abs() < 16 * 2.0 ** -24).all()
    assert (codes != want).float().mean().item() < 2e-5
    xs = wide[[0, rows - 1], :d].contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    if n <= 20480:
        parity.check_rotate_quantize(xs, n, 4, 0.9, codes[[0, rows - 1]].cpu().numpy(), scales[[0, rows - 1]].cpu().numpy(), f"narrow n={n} d={d}")


# (order, rows a compute unit up to which the workgroup block kernel takes it, 0: always)
FORMS = [(148 * 128, 2), (160 * 128, 2), (192 * 128, 1), (112 * 128, 2), (128 * 128, 2), (196 * 128, 1), (224 * 128, 1), (256 * 128, 1),
         (140 * 128, 0), (88 * 128, 0), (108 * 128, 0), (140 * 64, 0)]


@pytest.mark.parametrize("n,line", FORMS)
def test_which_form_runs(n, line):
    """By the number of rows; without it the comparisons above could be of a kernel with itself."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    h = binding.hadamard_build(n)
    x = torch.randn((3 * cus + 5, n), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").to(torch.bfloat16)
    for rows in (1, cus, cus + 1, 2 * cus, 2 * cus + 1, 3 * cus + 5):
        for bits in (3, 4):
            binding.rotate_quantize(h, x[:rows], bits, 0.9)
            assert h.last_kernel == ("wg_block_pair" if line and rows > line * cus else "wg_block"), rows
    if n <= 148 * 128:                                   # (the general kernel holds no wider row)
        binding.rotate_quantize(h, x[:, 1:n - 7], 4, 0.9)    # (rows off 16 bytes)
        assert h.last_kernel == "generic_lds"
        h.set_variant(1)
        binding.rotate_quantize(h, x, 4, 0.9)
        assert h.last_kernel == "generic_lds"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n", [148 * 128, 196 * 128, 204 * 128, 160 * 128, 224 * 128])
def test_rows_with_several_infinities(n, dtype):
    """The scale is infinite where the infinities of some value agree in sign and 0 where none do or the row has a NaN, as in the
    other form, also if every wave of the row has an infinity or all of the row is infinite."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows, pb = 3 * cus + 5, n // 128
    rng = np.random.default_rng(n)
    signs = np.zeros((rows, n), dtype=np.float32)
    for r in range(0, rows, 2):                          # (odd rows stay finite)
        kind = (r // 2) % 4
        if kind == 0:                                    # one in each wave's 32 block rows
            at = [128 * rng.integers(32 * w, min(pb, 32 * w + 32)) + rng.integers(128) for w in range((pb + 31) // 32)]
        else:
            at = rng.choice(n, [rng.integers(5, 10), rng.integers(10, 15), rng.integers(15, 60)][kind - 1], replace=False)
        signs[r, at] = rng.choice([-1.0, 1.0], len(at))
    signs[8] = 1.0                                       # (the first block row and column are of one sign)
    signs[10] = rng.choice([-1.0, 1.0], n)
    # a value whose infinities all agree: the largest sum of their signs is their number
    signs = torch.from_numpy(signs).cuda()
    h = binding.hadamard_build(n)
    sums = binding.rotate(h, signs.to(torch.bfloat16), out_dtype=torch.float32).abs().amax(1).double() * n ** 0.5
    count = signs.abs().sum(1).double()
    agree = (sums - count).abs() < 0.25
    x = torch.randn((rows, n), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").to(dtype)
    x[signs != 0] = signs[signs != 0].to(dtype) * float("inf")
    x[12, 77] = float("nan")
    x[14, torch.arange(60, n, 500, device="cuda")] = float("nan")
    agree[[12, 14]] = False
    nothing = count == 0
    nothing[[12, 14]] = False
    assert 20 < int((agree & ~nothing).sum()) and int((~agree).sum()) > 20
    for bits in (3, 4):
        codes, scales = binding.rotate_quantize(h, x, bits, 0.9)
        assert h.last_kernel == "wg_block_pair"
        few = [binding.rotate_quantize(h, x[i:i + cus], bits, 0.9) for i in range(0, rows, cus)]
        assert h.last_kernel == "wg_block"
        want, wscales = (torch.cat([f[k] for f in few]) for k in (0, 1))
        odd = ~nothing
        assert torch.equal(torch.isinf(wscales), agree & odd)
        assert torch.equal(scales[odd].view(torch.int32), wscales[odd].view(torch.int32))
        assert torch.equal(codes[odd], want[odd])
        assert ((scales[nothing] / wscales[nothing] - 1).abs() < 16 * 2.0 ** -24).all()
        assert (codes[nothing] != want[nothing]).float().mean().item() < 2e-5
