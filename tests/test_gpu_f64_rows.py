"""GPU parity of the fp64 kernel of fp32 rows: every split of the stages over its passes (k = 5 .. 14), block orders with
one and several parts, rows that share a workgroup with a ragged end, zero-padded rows of odd width and pitch."""
import numpy as np
import pytest
import torch

import parity
from paper_2504_13989_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,rows", [(128, 128, 21), (256, 251, 9), (512, 512, 3), (1024, 1000, 2), (2048, 2048, 3),
                                      (4096, 4095, 3), (8192, 8192, 2), (16384, 16001, 2), (896, 896, 5), (1536, 1501, 3),
                                      (3584, 3584, 3), (5120, 5120, 2), (4864, 4800, 2), (8960, 8960, 2), (6144, 6144, 2)])
@pytest.mark.parametrize("b", [3, 4])
def test_fp32_rows(n, d, rows, b):
    rng = np.random.default_rng(n + d + b)
    full = rng.standard_t(3.0, size=(rows, d + 3)).astype(np.float32)
    full[0, 5] *= 300.0
    if rows > 2:
        full[1] = 0.0
    h = binding.hadamard_build(n)
    codes, scales = binding.rotate_quantize(h, torch.from_numpy(full).cuda()[:, :d], b, 0.9)
    torch.cuda.synchronize()
    assert h.last_kernel == "f64_rows"
    parity.check_rotate_quantize(np.ascontiguousarray(full[:, :d]), n, b, 0.9, codes.cpu().numpy(), scales.cpu().numpy(),
                                 f"fp32 n={n} d={d} b={b}")
