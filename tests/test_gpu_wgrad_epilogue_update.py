"""GPU parity of the master-weight update inside the weight gradient's own epilogue (unsplit contractions on
64x64 tiles): equal, bit for bit, to the weight-gradient call followed by the stand-alone update."""
import numpy as np
import pytest

from gpu_util import gpu, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mp8():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_1905_12334_amd as m
    m.lib()
    return m


# both kernels (64x64s2 and the wave-split one), tiles at the edge of rows and columns, an incomplete stage
@pytest.mark.parametrize("dims", [(256, 64, 64), (384, 208, 80), (500, 272, 144), (2048, 1040, 976), (2100, 1024, 1008)])
@pytest.mark.parametrize("rule", ["sgd", "momentum", "adam"])
@pytest.mark.parametrize("contraction_major", [True, False])
def test_update_in_the_epilogue_equals_two_calls(mp8, dims, rule, contraction_major):
    import torch
    M, N, K = dims
    if not contraction_major and M % 16:
        M += 12
    rng = np.random.default_rng(M + N + K)
    x, e = ((rng.integers(0, 256, s).astype(np.uint8) & 0x83) | 0x38 for s in ((M, K), (M, N)))
    a, b = (gpu(t if contraction_major else np.ascontiguousarray(t.T)) for t in (x, e))
    n = K * N
    w0 = (rng.standard_normal(n) * 0.02).astype(np.float16)
    w0[:8] = np.float16(3e-6) * np.arange(8)                       # subnormal weights
    m0, v0 = rng.standard_normal(n).astype(np.float32) * 1e-3, rng.random(n).astype(np.float32) * 1e-6
    flags = mp8.FLAG_CONTRACTION_MAJOR if contraction_major else 0
    ws = torch.empty(max(16, n, mp8.gemm_fp8_workspace_bytes(mp8.WGRAD, M, N, K)), dtype=torch.uint8, device="cuda")
    for keep, skip, rounding in ((True, 0, mp8.SR), (False, 0, mp8.RNE), (True, 1, mp8.SR)):
        flag = torch.tensor([skip], dtype=torch.int32, device="cuda")
        st, st2 = mp8.new_stats(), mp8.new_stats()
        res = []
        for fused in (True, False):
            w, m, v = gpu(w0), gpu(m0), gpu(v0)
            w8 = torch.full((n + 16,), 0x55, dtype=torch.uint8, device="cuda")
            g = torch.full((n + 16,), 0xAA, dtype=torch.uint8, device="cuda")
            u = dict(skip_if_nonzero=flag, w8_out=w8[:n])
            if fused:
                kw = dict(g8_out=g[:n] if keep else None, alpha=0.25, g_round=rounding, flags=flags, g_seed=3, g_offset=1, stats=st,
                          w_round=rounding, w_seed=4, w_offset=2, workspace=ws, **u)
                if rule == "sgd":
                    mp8.wgrad_update_fp16_sr(M, N, K, a, b, w, 1e-3, 2.0 ** -8, **kw)
                elif rule == "momentum":
                    mp8.wgrad_momentum_fp16_sr(M, N, K, a, b, w, m, 1e-3, 2.0 ** -8, 0.9, weight_decay=1e-2, **kw)
                else:
                    mp8.wgrad_adam_fp16_sr(M, N, K, a, b, w, m, v, 1e-3, 2.0 ** -8, 7, weight_decay=1e-2, **kw)
            else:
                mp8.gemm_fp8(mp8.WGRAD, M, N, K, a, b, out8=g[:n], alpha=0.25, round=rounding, flags=flags, seed=3, offset=1,
                             stats=st2, workspace=ws)
                kw = dict(round=rounding, seed=4, offset=2, **u)
                if rule == "sgd":
                    mp8.sgd_update_fp16_sr(w, g[:n], 1e-3, 2.0 ** -8, **kw)
                elif rule == "momentum":
                    mp8.sgd_momentum_fp16_sr(w, m, g[:n], 1e-3, 2.0 ** -8, 0.9, 1e-2, **kw)
                else:
                    mp8.adam_fp16_sr(w, m, v, g[:n], 1e-3, 2.0 ** -8, 7, weight_decay=1e-2, **kw)
            torch.cuda.synchronize()
            assert bool((w8[n:] == 0x55).all()) and bool((g[n:] == 0xAA).all())
            res.append([host(t) for t in (w.view(torch.int16), m.view(torch.int32), v.view(torch.int32), w8)] + ([host(g)] if keep else []))
        assert all(np.array_equal(p, q) for p, q in zip(*res)), (keep, skip)
        assert mp8.read_stats(st) == mp8.read_stats(st2)


@pytest.mark.parametrize("dims,rule,own", [((256, 64, 64), "sgd", True), ((384, 208, 80), "momentum", True), ((2048, 1040, 976), "sgd", True),
                                           ((256, 64, 64), "adam", False), ((2048, 1040, 976), "adam", True),
                                           ((512, 1024, 512), "adam", True), ((512, 1024, 448), "adam", False)])
def test_which_calls_update_in_the_epilogue(mp8, dims, rule, own):
    """Only a kernel that applies the update in its own epilogue can do without a gradient buffer and a
    workspace where the contraction is whole stages: SGD and momentum on any number of 64x64 tiles,
    ADAM from 128 of them on."""
    import torch
    M, N, K = dims
    a, b = (torch.full(s, 0x38, dtype=torch.uint8, device="cuda") for s in ((M, K), (M, N)))
    w, m, v = (torch.zeros(K * N, dtype=t, device="cuda") for t in (torch.float16, torch.float32, torch.float32))
    kw = dict(flags=mp8.FLAG_CONTRACTION_MAJOR)
    call = {"sgd": lambda: mp8.wgrad_update_fp16_sr(M, N, K, a, b, w, 1e-3, 1.0, **kw),
            "momentum": lambda: mp8.wgrad_momentum_fp16_sr(M, N, K, a, b, w, m, 1e-3, 1.0, 0.9, **kw),
            "adam": lambda: mp8.wgrad_adam_fp16_sr(M, N, K, a, b, w, m, v, 1e-3, 1.0, 1, **kw)}[rule]
    if own:
        call()
        torch.cuda.synchronize()
        assert bool((w < 0).all())
    else:
        with pytest.raises(mp8.Mp8Error):
            call()


@pytest.mark.parametrize("dims", [(256, 64, 64), (400, 208, 80), (512, 1024, 448), (2048, 1024, 960), (2100, 1024, 1008)])   # 1 tile, 8, 112, 240, 256
@pytest.mark.parametrize("contraction_major", [True, False])
def test_adam_with_a_gradient_buffer_is_one_kernel(mp8, dims, contraction_major):
    """However few tiles there are, with whole and with incomplete stages, and with no workspace."""
    import torch

    from captured import launches
    M, N, K = dims
    M -= 0 if contraction_major else M % 16
    a, b = (torch.full(s, 0x38, dtype=torch.uint8, device="cuda") for s in ((M, K), (M, N)))
    w, m, v = (torch.zeros(K * N, dtype=t, device="cuda") for t in (torch.float16, torch.float32, torch.float32))
    g = torch.empty(K * N, dtype=torch.uint8, device="cuda")
    call = lambda: mp8.wgrad_adam_fp16_sr(M, N, K, a, b, w, m, v, 1e-3, 1.0, 1, g8_out=g,
                                          flags=mp8.FLAG_CONTRACTION_MAJOR if contraction_major else 0)
    call()
    torch.cuda.synchronize()
    names = launches(call)
    assert len(names) == 1 and "update" in names[0], names
