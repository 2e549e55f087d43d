"""GPU: what the native marshalling has to get right - row geometry of views, caller's outputs and streams,
errors - against the same rows handed over as a plain contiguous matrix."""
import numpy as np
import pytest
import torch

from paper_2504_13989_amd import binding

pytestmark = pytest.mark.gpu


def _rows(rows, d, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(7)
    return torch.randn((rows, d), generator=g, device="cuda").to(dtype)


@pytest.mark.parametrize("view", ["4d", "slice", "one_row", "every_other", "empty"])
def test_views_give_the_rows_of_a_plain_matrix(view):
    h = binding.hadamard_build(256)
    wide = _rows(24, 768)
    x = {"4d": wide.view(2, 3, 12, 256), "slice": wide[:, 256:512], "one_row": wide[3:4, :256],
         "every_other": wide[::2, 512:], "empty": wide[:0, :256]}[view]
    plain = x.reshape(-1, 256).contiguous()
    codes, scales = binding.rotate_quantize(h, x, 4, 0.9)
    want, wscales = binding.rotate_quantize(h, plain, 4, 0.9)
    assert codes.shape == (plain.shape[0], 128) and scales.shape == (plain.shape[0],)
    assert torch.equal(codes, want) and torch.equal(scales, wscales)


def test_callers_outputs_and_stream():
    h = binding.hadamard_build(256)
    x = _rows(40, 256)
    want, wscales = binding.rotate_quantize(h, x, 3, 0.9)
    codes, scales = torch.zeros_like(want), torch.zeros_like(wscales)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    c, s = binding.rotate_quantize(h, x, np.int64(3), np.float32(0.9), codes=codes, scales=scales, stream=side)
    assert c is codes and s is scales
    side.synchronize()
    assert torch.equal(codes, want) and torch.equal(scales, wscales)
    wide = torch.zeros((40, 400), dtype=torch.float32, device="cuda")
    y = binding.rotate(h, x, d_out=200, out=wide[:, 100:300])
    assert y.data_ptr() == wide[:, 100:300].data_ptr()
    assert torch.equal(wide[:, 100:300], binding.rotate(h, x, d_out=200))
    assert not wide[:, :100].any() and not wide[:, 300:].any()
    clips = (0.5, 0.75, 1.0)
    assert torch.equal(binding.quant_error(h, x, 3, clips), binding.quant_error(h, x, 3, np.array(clips, np.float32)))


def test_errors():
    h = binding.hadamard_build(256)
    x = _rows(4, 256)
    with pytest.raises(ValueError, match="device tensor"):
        binding.rotate_quantize(h, x.cpu(), 4, 0.9)
    with pytest.raises(ValueError, match="contiguous"):
        binding.rotate_quantize(h, x.t(), 4, 0.9)
    with pytest.raises(ValueError, match="2-D"):
        binding.rotate_quantize(h, _rows(24, 512).view(2, 12, 512)[:, :, :256], 4, 0.9)
    with pytest.raises(TypeError, match="dtype"):
        binding.rotate_quantize(h, x.double(), 4, 0.9)
    with pytest.raises(ValueError, match="output dtype"):
        binding.rotate(h, x, out_dtype=torch.float64)
    for bits, clip in ((5, 0.9), (4, 1.5)):
        with pytest.raises(binding.RotqError) as e:
            binding.rotate_quantize(h, x, bits, clip)
        assert e.value.code == binding.RQ_ERR_ARG
    h.close()
    with pytest.raises(binding.RotqError):
        binding.rotate_quantize(h, x, 4, 0.9)


@pytest.mark.parametrize("rows", [16, 4096])
@pytest.mark.parametrize("call", ["rotate_quantize", "rotate_quantize_asym", "quantize", "quantize_asym"])
def test_results_are_saved_together_and_resized_apart(tmp_path, call, rows):
    """every result has a storage of its own, of its own size: torch.save takes them in one file, and resizing one
    leaves the others alone"""
    x = _rows(rows, 256)
    fn = getattr(binding, call)
    results = fn(binding.hadamard_build(256), x, 4, 0.9) if call.startswith("rotate") else fn(x, 4, 0.9)
    assert [r.untyped_storage().nbytes() for r in results] == [r.numel() * r.element_size() for r in results]
    assert len({r.untyped_storage().data_ptr() for r in results}) == len(results)
    torch.save(results, tmp_path / "results.pt")
    back = torch.load(tmp_path / "results.pt", weights_only=True)
    assert all(torch.equal(a, b) for a, b in zip(results, back))
    kept = [r.clone() for r in results[1:]]
    results[0].resize_(rows + 8, 128).fill_(255)
    assert all(torch.equal(a, b) for a, b in zip(results[1:], kept))
