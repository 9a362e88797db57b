"""The extension module behind the package's functions refuses what it must before anything is
enqueued, and takes what stands for a number or a pointer."""
import pytest
import torch

import paper_1905_12334_amd as mp8


def test_every_call_refuses_tensors_that_are_not_on_the_gpu():
    f, u, h = torch.zeros((128, 128)), torch.zeros((128, 128), dtype=torch.uint8), torch.zeros(128 * 128, dtype=torch.float16)
    calls = [
        lambda: mp8.quantize_e5m2(f, u),
        lambda: mp8.gemm_fp8(mp8.FWD, 128, 128, 128, u, u, out8=u),
        lambda: mp8.gemm_fp8_static(mp8.FWD, 128, 128, 128, u, u, out8=u),
        lambda: mp8.quantize_gemm_fwd_fp8(128, 128, 128, f, u, u, out8=u),
        lambda: mp8.conv3x3_fp8(mp8.FWD, 1, 4, 4, 128, 128, u, u, out8=u),
        lambda: mp8.wgrad_update_fp16_sr(128, 128, 128, u, u, h, 0.1, 1.0),
        lambda: mp8.wgrad_momentum_fp16_sr(128, 128, 128, u, u, h, f, 0.1, 1.0, 0.9),
        lambda: mp8.wgrad_adam_fp16_sr(128, 128, 128, u, u, h, f, f, 0.1, 1.0, 1),
        lambda: mp8.conv3x3_wgrad_update_fp16_sr(1, 4, 4, 128, 128, u, u, h, 0.1, 1.0),
        lambda: mp8.conv3x3_wgrad_momentum_fp16_sr(1, 4, 4, 128, 128, u, u, h, f, 0.1, 1.0, 0.9),
        lambda: mp8.sgd_update_fp16_sr(h, u, 0.1, 1.0),
        lambda: mp8.sgd_momentum_fp16_sr(h, f, u, 0.1, 1.0, 0.9),
        lambda: mp8.adam_fp16_sr(h, f, f, u, 0.1, 1.0, 1),
    ]
    for call in calls:
        with pytest.raises(mp8.Mp8Error, match="must be a GPU tensor"):
            call()


def test_arguments_of_the_wrong_kind_raise():
    with pytest.raises(TypeError):
        mp8.gemm_fp8(mp8.FWD, 1, 1, 1, None, None)
    with pytest.raises(TypeError):
        mp8.quantize_e5m2([1.0], None)
    with pytest.raises(TypeError):
        mp8.gemm_fp8(mp8.FWD, "1", 1, 1, None, None)


def test_dimensions_and_operations_do_not_wrap():
    u = torch.zeros((128, 128), dtype=torch.uint8)
    for dims in ((2 ** 64 + 128, 128, 128), (128, 2 ** 64, 128), (128, 128, -2 ** 64 + 128)):
        with pytest.raises(mp8.Mp8Error, match="64 bits"):
            mp8.gemm_fp8(mp8.FWD, *dims, u, u, out8=u)
    for op in (3, -1, 2 ** 32):
        with pytest.raises(KeyError):
            mp8.gemm_fp8(op, 128, 128, 128, u, u, out8=u)
        with pytest.raises(KeyError):
            mp8.conv3x3_fp8(op, 1, 4, 4, 128, 128, u, u, out8=u)


@pytest.mark.gpu
def test_sizes_that_overflow_are_refused():
    """Products of dimensions and leading dimensions that exceed 64 bits are larger than any tensor."""
    u = torch.zeros((128, 128), dtype=torch.uint8, device="cuda")
    f, h = torch.zeros((128, 128), device="cuda"), torch.zeros((128, 128), dtype=torch.float16, device="cuda")
    e8, ef = torch.zeros(0, dtype=torch.uint8, device="cuda"), torch.zeros(0, device="cuda")
    big = 2 ** 62
    calls = [
        lambda: mp8.gemm_fp8(mp8.FWD, 128, 128, 128, u, u, out8=u, lda=big + 1),
        lambda: mp8.gemm_fp8(mp8.FWD, 128, 128, 128, u, u, out8=u, ldb=big),
        lambda: mp8.gemm_fp8(mp8.WGRAD, 128, 128, 128, u, u, out8=u, lda=big, flags=mp8.FLAG_CONTRACTION_MAJOR),
        lambda: mp8.gemm_fp8(mp8.FWD, 2 ** 32, 2 ** 32, 1, u, u, out8=u),
        lambda: mp8.quantize_gemm_fwd_fp8(128, 128, 128, f, u, u, out8=u, ldw=big),
        lambda: mp8.quantize_gemm_fwd_fp8(2 ** 32, 128, 2 ** 32, ef, e8, u, out8=u),
        lambda: mp8.conv3x3_fp8(mp8.FWD, 2 ** 62, 2, 2, 128, 128, e8, u, out8=u),
        lambda: mp8.conv3x3_fp8(mp8.FWD, 1, 4, 4, 128, 128, e8, u, out8=u, prows=2 ** 57),
        lambda: mp8.wgrad_update_fp16_sr(128, 128, 128, u, u, h, 0.1, 1.0, lda=big),
        lambda: mp8.wgrad_update_fp16_sr(128, 2 ** 32, 2 ** 32, u, u, h, 0.1, 1.0),
    ]
    for i, call in enumerate(calls):
        with pytest.raises(mp8.Mp8Error, match="smaller than|elements|sizes"):
            print("call", i, flush=True)
            call()
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_arguments_that_stand_for_numbers_and_pointers():
    """A step counter may be what optimizers keep (a float, a tensor); statistics, scratch and flags may be any
    object with a tensor's methods."""
    class Wrapped:
        def __init__(self, t):
            self.data_ptr, self.numel, self.element_size = t.data_ptr, t.numel, t.element_size

    n = 128 * 128
    x = torch.full((128, 128), 0x38, dtype=torch.uint8, device="cuda")
    results = []
    for step in (7, 7.0, torch.tensor(7.0), torch.tensor(7.0, device="cuda")):
        w, m, v = (torch.full((n,), 0.5, dtype=t, device="cuda") for t in (torch.float16, torch.float32, torch.float32))
        w2, m2, v2 = w.clone(), m.clone(), v.clone()
        mp8.adam_fp16_sr(w, m, v, x, torch.tensor(1e-2), 1.0, step)
        mp8.wgrad_adam_fp16_sr(128, 128, 128, x, x, w2, m2, v2, 1e-2, 1.0, step, g8_out=torch.empty_like(x),
                               workspace=Wrapped(torch.empty(4 * n, dtype=torch.uint8, device="cuda")))
        results.append((w, m, v, w2, m2, v2))
    assert all(torch.equal(p, q) for r in results[1:] for p, q in zip(results[0], r))
    src, out = torch.full((128, 128), float("inf"), device="cuda"), torch.zeros_like(x)
    stats = mp8.new_stats()
    mp8.quantize_e5m2(src, out, stats=Wrapped(stats))
    assert mp8.read_stats(stats)[1] == n
    before = results[0][0].clone()
    mp8.sgd_update_fp16_sr(results[0][0], x, 1.0, 1.0, skip_if_nonzero=Wrapped(stats[1:2]))
    assert torch.equal(before, results[0][0])


@pytest.mark.gpu
def test_dtype_errors_say_what_is_expected():
    u, d = torch.zeros((128, 128), dtype=torch.uint8, device="cuda"), torch.zeros((128, 128), dtype=torch.float64, device="cuda")
    with pytest.raises(mp8.Mp8Error, match=r"src has dtype torch.float64, expected \(torch.float32, torch.float16\)"):
        mp8.quantize_e5m2(d, u)
    with pytest.raises(mp8.Mp8Error, match="b has dtype torch.float64, expected torch.uint8"):
        mp8.gemm_fp8(mp8.FWD, 128, 128, 128, u, d, out8=u)
