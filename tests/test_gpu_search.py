"""GPU: the clip search against Algorithm 1 run on its own values and against quant_error, in its resident form (one launch),
its stepped form (the same values bit for bit) and its batched form: every waves-per-row form, one row to the most rows a
chip holds, ragged last workgroup, an evaluation limit; its memory, numbers and threads.  Brackets below 1 / 256, where the
search has these forms only; the grid form has tests of its own (test_gpu_grid_search.py)."""
import numpy as np
import pytest

import parity
import rotq_oracle as oracle
from paper_2504_13989_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


def _resident(h, x, *args, **kwargs):
    """a search that was taken in one launch (other work on the device may keep one from it: the result is the same then)"""
    got = binding.gbs_search(h, x, *args, **kwargs)
    for _ in range(3):
        if h.last_kernel == "gbs_resident":
            break
        assert h.last_kernel == "gbs_stepped" and binding.gbs_search(h, x, *args, **kwargs) == got
    assert h.last_kernel == "gbs_resident"
    return got


@pytest.mark.parametrize("n,d,rows", [(1024, 1024, 4096), (2048, 2000, 515), (4096, 4096, 1), (4096, 4096, 1023), (8192, 8192, 300),
                                      (1536, 1536, 257), (3584, 3584, 700), (3072, 3000, 2048), (4096, 4096, 1025)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_search_takes_the_steps_of_algorithm_1(n, d, rows, dtype):
    rng = np.random.default_rng(n + rows)
    xf = rng.standard_normal((rows, d)).astype(np.float32)
    xf[rows // 2] *= 20.0
    x = parity.to_device(wl.f32_to_bf16_bits(xf) if dtype == "bf16" else xf.astype(np.float16))
    h = binding.hadamard_build(n)
    most = {1024: 4096, 1536: 4096, 2048: 2048, 3072: 2048, 3584: 2048, 4096: 1024, 8192: 1024}[n]     # 256 compute units
    for b in (3, 4):
        if rows <= most:
            clip, mse, trace = _resident(h, x, b, 1.0 / 300)
        else:
            clip, mse, trace = binding.gbs_search(h, x, b, 1.0 / 300)
            assert h.last_kernel == "wave_quant_error"
        # Algorithm 1 with the values of the trace as its objective asks for the trace's probes, in its order
        seen = dict(trace)
        m, fm, otrace = oracle.gbs_search(lambda c: seen[np.float32(c)], 1.0 / 300)
        assert [np.float32(c) for c, _ in otrace] == [np.float32(c) for c, _ in trace]
        assert clip == np.float32(m) and mse == fm
        # and the values are quant_error's
        want = binding.quant_error(h, x, b, [c for c, _ in trace]).cpu().numpy()
        assert np.allclose([v for _, v in trace], want, rtol=2e-6, atol=0.0)
        _, _, short = binding.gbs_search(h, x, b, 1.0 / 300, max_evals=4)
        assert short == trace[:4]


@pytest.mark.parametrize("n,d,rows", [(1024, 1024, 4096), (2048, 2000, 515), (4096, 4096, 1), (4096, 4096, 1023), (8192, 8192, 300),
                                      (1536, 1536, 257), (3584, 3584, 700), (3072, 3000, 2048)])
def test_the_stepped_form_gives_the_resident_forms_bits(n, d, rows):
    """a launch per step (variant 5), and the resident form given up because nobody waits (variant 6)"""
    rng = np.random.default_rng(n + rows)
    x = parity.to_device(wl.f32_to_bf16_bits((rng.standard_normal((rows, d)) * 3).astype(np.float32)))
    h = binding.hadamard_build(n)
    for b, eps, limit in ((3, 1.0 / 300, 64), (4, 1.0 / 1000, 64), (4, 1e-30, 256), (3, 1.0 / 300, 1), (3, 1.0 / 300, 2), (4, 1.0 / 300, 7)):
        h.set_variant(0)
        want = _resident(h, x, b, eps, max_evals=limit)
        for variant in (5, 6, 7):
            h.set_variant(variant)
            for _ in range(2):
                assert binding.gbs_search(h, x, b, eps, max_evals=limit) == want, (b, eps, limit, variant)
                assert h.last_kernel == "gbs_stepped" or (variant == 6 and h.last_kernel == "gbs_resident")
    # the variants that name a form take it at every bracket, also where automatic has the grid form
    for b, eps, limit in ((3, 1.0 / 256, 64), (4, 1.0 / 64, 64), (3, 1.0 / 256, 2), (4, 0.9, 64)):
        h.set_variant(5)
        want = binding.gbs_search(h, x, b, eps, max_evals=limit)
        assert h.last_kernel == "gbs_stepped"
        seen = dict(want[2])
        m, fm, trace = oracle.gbs_search(lambda c: seen[np.float32(c)], float(np.float32(eps)), max_evals=limit)
        assert want[0] == np.float32(m) and want[1] == fm and [np.float32(c) for c, _ in trace] == [np.float32(c) for c, _ in want[2]]
        h.set_variant(6)
        assert binding.gbs_search(h, x, b, eps, max_evals=limit) == want
        assert h.last_kernel in ("gbs_stepped", "gbs_resident")
        h.set_variant(0)
        got = binding.gbs_search(h, x, b, eps, max_evals=limit)
        assert np.allclose([v for _, v in got[2]], [v for _, v in want[2]], rtol=2e-6, atol=0.0)
    h.set_variant(0)


def test_step_numbers_that_wrap():
    """the resident form's step numbers start again after 255 searches; two streams in turn, so that nothing but the
    exchange buffers orders the searches"""
    import torch
    rng = np.random.default_rng(10)
    xs = [parity.to_device(wl.f32_to_bf16_bits(rng.standard_normal((r, 4096)).astype(np.float32))) for r in (900, 33)]
    h = binding.hadamard_build(4096)
    want = [binding.gbs_search(h, x, 3, 1.0 / 300) for x in xs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    resident = 0
    for i in range(600):
        assert binding.gbs_search(h, xs[i % 2], 3, 1.0 / 300, stream=streams[i % 3 % 2]) == want[i % 2], i
        resident += h.last_kernel == "gbs_resident"
    assert resident > 540


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("eps", [1e-15, 1e-16, 1e-30])
def test_a_bracket_that_stops_shrinking(dtype, eps):
    """Below an ulp of the clip ratio the bracket no longer shrinks: the search ends at its limit of evaluations, in the
    batched form (fp32 rows) as in the resident one."""
    rng = np.random.default_rng(8)
    xf = rng.standard_normal((16, 1024)).astype(np.float32)
    x = parity.to_device(xf if dtype == "f32" else wl.f32_to_bf16_bits(xf))
    for limit in (128, 256):
        clip, mse, trace = binding.gbs_search(binding.hadamard_build(1024), x, 3, eps, max_evals=limit)
        seen = dict(trace)
        m, fm, otrace = oracle.gbs_search(lambda c: seen[np.float32(c)], float(np.float32(eps)), max_evals=limit)
        assert [np.float32(c) for c, _ in otrace] == [np.float32(c) for c, _ in trace]
        assert clip == np.float32(m) and mse == fm


@pytest.mark.parametrize("eps", [1.0 / 300, 1.0 / 256])
def test_searches_of_several_threads_and_streams(eps):
    """four at once: of the resident form (1 / 300) one has the turn and the others go step by step, the grid form (1 / 256) has
    no turns"""
    import threading
    import torch
    h = binding.hadamard_build(4096)
    rng = np.random.default_rng(5)
    xs = [parity.to_device(wl.f32_to_bf16_bits(rng.standard_normal((r, 4096)).astype(np.float32))) for r in (512, 300, 512, 40)]
    want = [binding.gbs_search(h, x, 3, eps) for x in xs]
    assert (h.last_kernel == "grid_search") == (eps > 1.0 / 300)
    torch.cuda.synchronize()
    got = [[] for _ in xs]

    def work(i):
        s = torch.cuda.Stream()
        for _ in range(10):
            got[i].append(binding.gbs_search(h, xs[i], 3, eps, stream=s))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(xs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i, (clip, mse, trace) in enumerate(want):
        assert len(got[i]) == 10
        for c, m, tr in got[i]:
            assert (c, m, tr) == (clip, mse, trace)


@pytest.mark.parametrize("eps", [1.0 / 300, 1.0 / 64])
def test_more_searches_at_once_than_slots_and_no_handle_left(eps):
    """More searches at once than a device has slots for, then none of the handles left, and again."""
    import gc
    import threading
    import torch
    rng = np.random.default_rng(6)
    x = parity.to_device(wl.f32_to_bf16_bits(rng.standard_normal((64, 1024)).astype(np.float32)))
    got = []
    for _ in range(2):
        h = binding.hadamard_build(1024)
        start = threading.Barrier(24)

        def work(h=h):
            s = torch.cuda.Stream()
            start.wait()
            for _ in range(4):
                got.append(binding.gbs_search(h, x, 4, eps, stream=s))

        threads = [threading.Thread(target=work) for _ in range(24)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        del threads, work, h
        gc.collect()
    assert len(got) == 2 * 24 * 4
    assert all(g == got[0] for g in got)


@pytest.mark.parametrize("eps", [1.0 / 300, 1.0 / 256])
def test_results_without_pinned_memory(eps):
    """where pinned host memory cannot be had, the results are copied back"""
    rng = np.random.default_rng(7)
    x = parity.to_device(wl.f32_to_bf16_bits(rng.standard_normal((200, 2048)).astype(np.float32)))
    for n_evals in (1, 64):
        for asym in (False, True):
            h = binding.hadamard_build(2048)
            want = binding.gbs_search(h, x, 3, eps, max_evals=n_evals, asym=asym)
            h.set_variant(7)
            for _ in range(3):
                assert binding.gbs_search(h, x, 3, eps, max_evals=n_evals, asym=asym) == want


def test_a_search_on_a_new_handle_allocates_nothing():
    """build, search, free costs what build, free and a search cost: device and pinned memory allocated and freed with
    every such search was 58 us more"""
    import statistics
    import time
    import torch
    x = parity.to_device(wl.f32_to_bf16_bits(np.random.default_rng(9).standard_normal((64, 4096)).astype(np.float32)))
    keep = binding.hadamard_build(256)
    first = binding.gbs_search(binding.hadamard_build(4096), x, 3, 1.0 / 256)
    del keep

    def median_us(fn):
        times = []
        for _ in range(25):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            fn()
            times.append((time.perf_counter() - t0) * 1e6)
        return statistics.median(times)

    def with_search():
        h = binding.hadamard_build(4096)
        assert binding.gbs_search(h, x, 3, 1.0 / 256) == first
        h.close()

    h = binding.hadamard_build(4096)
    search = median_us(lambda: binding.gbs_search(h, x, 3, 1.0 / 256))
    h.close()
    seen = []
    for _ in range(3):                                     # (a timing: the best of three)
        bare, full = median_us(lambda: binding.hadamard_build(4096).close()), median_us(with_search)
        seen.append(full - bare - search)
    assert min(seen) < 30.0, seen
