"""GPU parity of the rotation-free quantizer at the edges of its split of a row over waves: widths around 512, 1024,
4096, 8192, 12288 and 20480 values, row counts on either side of each rule."""
import numpy as np
import pytest

import parity
from paper_2504_13989_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,rows", [(544, 3), (1024, 512), (1024, 513), (1056, 7), (2048, 2049), (4096, 5), (4096, 2049),
                                    (4128, 513), (8192, 512), (8192, 513), (8224, 3), (12288, 5), (12320, 2), (20480, 3)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_plain_quantize_widths(d, rows, dtype):
    import torch
    rng = np.random.default_rng(d + rows)
    xf = rng.standard_t(3.0, size=(rows, d)).astype(np.float32)
    xf[rows // 2] = 0.0
    xf[0, d - 1] = 60.0                                   # the row's maximum in its last chunk
    x = wl.f32_to_bf16_bits(xf) if dtype == "bf16" else xf.astype(np.float16)
    for b in (3, 4):
        codes, scales = binding.quantize(parity.to_device(x), b, 0.9)
        torch.cuda.synchronize()
        parity.check_quantize_plain(x, b, 0.9, codes.cpu().numpy(), scales.cpu().numpy(), f"plain d={d} rows={rows} {dtype} b={b}")
