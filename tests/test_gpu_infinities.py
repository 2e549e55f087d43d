"""GPU: rows with infinities on the workgroup block kernel."""
import numpy as np
import pytest
import torch

from paper_2504_13989_amd import binding

pytestmark = pytest.mark.gpu


# full rows and padded ones; block rows of 32, 64 and 128 columns; blocks that do and do not fill the last wave's 16 rows
@pytest.mark.parametrize("n,d", [(896, 896), (4864, 4864), (4864, 4856), (8960, 8960), (11264, 11008), (13824, 13824),
                                 (14336, 14336), (18944, 18944), (18944, 18808), (26112, 26112), (28672, 28672)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_an_infinity_of_any_block_row_is_the_scale(n, d, dtype):
    """One infinity in a row makes every rotated value an infinity: the scale is infinite wherever it stands."""
    h = binding.hadamard_build(n)
    columns = [*range(0, d, max(1, d // 40)), *range(d - 600, d, 29), d - 1]
    x = torch.randn((len(columns), d), generator=torch.Generator().manual_seed(n)).to(dtype)
    x[torch.arange(len(columns)), columns] = torch.tensor([float("inf"), -float("inf")] * len(columns), dtype=dtype)[:len(columns)]
    for bits in (3, 4):
        codes, scales = binding.rotate_quantize(h, x.cuda(), bits, 0.9)
        assert h.last_kernel == "wg_block"
        lost = [c for c, s in zip(columns, scales.tolist()) if s != float("inf")]
        assert not lost, f"columns whose infinity is lost: {lost}"
        assert np.unique(codes.cpu().numpy()).size <= bits          # (the same code everywhere: as many patterns of bytes at most)
