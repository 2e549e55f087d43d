"""GPU parity of quant_error where a row's waves, or the workgroups of a pass, share the clip ratios: few rows, numbers of
ratios that do not divide evenly, both sides of the rules' row counts."""
import numpy as np
import pytest

import parity
from paper_2504_13989_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,rows,k", [(1024, 1024, 5, 33), (2048, 2000, 3, 33), (4096, 4096, 2, 64), (4096, 4096, 513, 5),
                                        (8192, 8192, 3, 7), (8192, 6000, 1100, 2), (896, 896, 5, 33), (4864, 4864, 2, 9),
                                        (5120, 5120, 3, 33), (8960, 8960, 1, 17), (18944, 18944, 2, 6), (128, 128, 3, 33), (256, 256, 9, 5),
                                        (128, 100, 5000, 7)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_quant_error_shares(n, d, rows, k, dtype):
    import torch
    rng = np.random.default_rng(n + rows + k)
    xf = rng.standard_t(4.0, size=(rows, d)).astype(np.float32)
    x = wl.f32_to_bf16_bits(xf) if dtype == "bf16" else xf.astype(np.float16)
    clips = np.linspace(0.4, 1.0, k).astype(np.float32)
    h = binding.hadamard_build(n)
    for b in (3, 4):
        mse = binding.quant_error(h, parity.to_device(x), b, clips)
        torch.cuda.synchronize()
        parity.check_quant_error(x, n, b, clips, mse.cpu().numpy(), what=f"n={n} rows={rows} clips={k} {dtype} b={b}")
    if n == 128:
        mse = binding.quant_error(h, parity.to_device(x), 3, clips, asym=True)
        torch.cuda.synchronize()
        parity.check_quant_error(x, n, 3, clips, mse.cpu().numpy(), what=f"asym rows={rows} clips={k} {dtype}", asym=True)
