"""GPU: row counts at which one workgroup per row would be 2^32 threads or more in a grid dimension, of which the launch
keeps the remainder only: a few rows among millions of others against the same rows alone."""
import numpy as np
import pytest
import torch

from paper_2504_13989_amd import binding

pytestmark = pytest.mark.gpu


def _some(rows):
    return torch.tensor([0, 1, rows // 2, rows - 2, rows - 1], device="cuda")


def _need(gigabytes):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gigabytes * (1 << 30):
        pytest.skip(f"needs {gigabytes} GiB of device memory")


def _rows_alone(x, rows):
    g = torch.Generator(device="cuda").manual_seed(1)
    x[_some(rows)] = torch.randn((5, x.shape[1]), generator=g, device="cuda").to(x.dtype)
    return x[_some(rows)].contiguous()


def test_plain_quantizer_with_eight_waves_a_row():
    rows, d = (1 << 23) + 5, 8224
    _need(200)
    x = torch.empty((rows, d), dtype=torch.bfloat16, device="cuda")
    alone = _rows_alone(x, rows)
    codes, scales = binding.quantize(x, 3, 0.9)
    want = binding.quantize(alone, 3, 0.9)
    assert torch.equal(codes[_some(rows)], want[0]) and torch.equal(scales[_some(rows)], want[1])
    del x, codes, scales
    torch.cuda.empty_cache()


def test_fp32_rows():
    rows, d, n = (1 << 23) + 5, 8, 8192
    _need(40)
    x = torch.zeros((rows, d), dtype=torch.float32, device="cuda")
    alone = _rows_alone(x, rows)
    h = binding.hadamard_build(n)
    codes, scales = binding.rotate_quantize(h, x, 3, 0.9)
    assert h.last_kernel == "f64_rows"
    want = binding.rotate_quantize(h, alone, 3, 0.9)
    assert torch.equal(codes[_some(rows)], want[0]) and torch.equal(scales[_some(rows)], want[1])
    assert not codes[2:1000].any() and not scales[2:1000].any()
    del x, codes, scales
    torch.cuda.empty_cache()


def test_quant_error_of_rows_split_over_waves():
    rows, d, n = (1 << 24) + 5, 8, 8192
    _need(8)
    x = torch.zeros((rows, d), dtype=torch.bfloat16, device="cuda")
    alone = _rows_alone(x, rows)
    h = binding.hadamard_build(n)
    clips = [0.7, 1.0]
    got = binding.quant_error(h, x, 3, clips).cpu().numpy()
    assert h.last_kernel == "wave_quant_error"
    want = binding.quant_error(h, alone, 3, clips).cpu().numpy().astype(np.float64) * 5 / rows     # the others are zero
    assert np.allclose(got, want, rtol=1e-6, atol=0.0)


def _repeated(call, x, rows):
    """The sampled rows of a call on x against those of a call on them alone, and rows between them, which are zero."""
    alone = _rows_alone(x, rows)
    got = call(x)
    for g, want in zip(got, call(alone)):
        assert torch.equal(g[_some(rows)], want)
    for g in got[:1]:
        assert not g[2:1000].any() and not g[rows - 1000:rows - 2].any()


# Kernels of one-wave workgroups with a row, or a few rows, each: 2^24 workgroups at most, which take a second item from there on.
MOST = 1 << 24


@pytest.mark.parametrize("n,bits,kernel,gigabytes", [(1024, 4, "wave_sylvester", 20), (1536, 3, "wave_block", 25), (5120, 3, "wave_block", 50)],
                         ids=["orders of 2", "blocks to 32", "blocks to 64"])
def test_rows_of_one_wave_each(n, bits, kernel, gigabytes):
    rows = MOST + 5
    _need(gigabytes)
    x = torch.zeros((rows, 8), dtype=torch.bfloat16, device="cuda")
    h = binding.hadamard_build(n)
    _repeated(lambda v: binding.rotate_quantize(h, v, bits, 0.9), x, rows)
    assert h.last_kernel == kernel
    del x
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n,rows,gigabytes,kernel", [(1024, MOST + 5, 50, "wave_rotate"), (128, 16 * MOST + 5, 110, "wave_rotate"),
                                                     (1536, MOST + 5, 70, "wave_block_rotate")],
                         ids=["one row a wave", "16 rows a wave", "block order"])
def test_rotation_of_rows(n, rows, gigabytes, kernel):
    _need(gigabytes)
    x = torch.zeros((rows, 8), dtype=torch.bfloat16, device="cuda")
    h = binding.hadamard_build(n)
    _repeated(lambda v: (binding.rotate(h, v, out_dtype=torch.bfloat16),), x, rows)
    assert h.last_kernel == kernel
    del x
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d,rows,gigabytes", [(544, MOST + 5, 30), (32, 16 * MOST + 5, 30)], ids=["one row a wave", "16 rows a wave"])
def test_plain_quantizer_of_rows(d, rows, gigabytes):
    _need(gigabytes)
    x = torch.zeros((rows, d), dtype=torch.bfloat16, device="cuda")
    _repeated(lambda v: binding.quantize(v, 3, 0.9), x, rows)
    del x
    torch.cuda.empty_cache()


def test_plain_group_quantizer_of_rows():
    rows, d = 16 * MOST + 5, 128
    _need(110)
    x = torch.zeros((rows, d), dtype=torch.bfloat16, device="cuda")
    _repeated(lambda v: binding.quantize_asym(v, 3, 0.9), x, rows)
    del x
    torch.cuda.empty_cache()
