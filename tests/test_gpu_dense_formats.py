"""GPU parity of the dense-block kernel in both 16-bit formats: tiles per wave from one to twenty-five, one and two groups
of rows per workgroup."""
import numpy as np
import pytest

import parity
import rotq_oracle as oracle
from paper_2504_13989_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows", [(104, 17), (568, 5), (1040, 33), (1544, 1), (1544, 16), (1784, 19), (3088, 7),
                                    (568, 8193), (1544, 4097)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_dense_block(n, rows, dtype):
    import torch
    if oracle.factor_order(n) is None:
        pytest.skip(f"{n} is not a constructible order")
    rng = np.random.default_rng(n + rows)
    d = n - 8
    xf = rng.standard_t(3.0, size=(rows, d)).astype(np.float32)
    xf[rows // 2] = 0.0
    x = wl.f32_to_bf16_bits(xf) if dtype == "bf16" else xf.astype(np.float16)
    h = binding.hadamard_build(n)
    for b in (3, 4):
        codes, scales = binding.rotate_quantize(h, parity.to_device(x), b, 0.9)
        torch.cuda.synchronize()
        assert h.last_kernel == "dense_block"
        sel = np.unique(np.concatenate([np.arange(min(rows, 40)), [rows // 2], np.arange(max(0, rows - 24), rows)]))
        parity.check_rotate_quantize(x[sel], n, b, 0.9, codes.cpu().numpy()[sel], scales.cpu().numpy()[sel],
                                     f"dense n={n} rows={rows} {dtype} b={b}")
