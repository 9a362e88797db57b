"""Which weight gradients of unaligned rows apply the update in their own epilogue."""
import numpy as np
import pytest

from captured import launches
from gpu_util import gpu, host
from test_gpu_gemm_ragged import TN, mp8  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu

RULES = ["sgd", "momentum", "adam"]


# tiles of 64 x 64: K by N; M leaves the contraction unsplit.  One kernel for SGD, momentum, ADAM -- without and with statistics of the gradient?
@pytest.mark.parametrize("dims,own,own_stats", [
    ((129, 24, 31 * 64), (0, 0, 0), (0, 0, 0)), ((129, 24, 32 * 64), (1, 1, 0), (1, 1, 0)), ((129, 36, 32 * 64), (0, 0, 0), (0, 0, 0)),  # 31 tiles, 32; no multiple of eight columns
    ((129, 520, 20 * 64), (1, 1, 0), (1, 1, 0)), ((129, 520, 9 * 64), (0, 0, 0), (0, 0, 0)), ((129, 536, 9 * 64), (1, 1, 0), (1, 1, 0)),  # a last column of tiles eight wide: 180 tiles, 81
    ((129, 1000, 16 * 64), (1, 1, 0), (1, 1, 0)), ((129, 1000, 17 * 64), (1, 1, 0), (0, 0, 0)), ((129, 1000, 32 * 64), (1, 1, 1), (0, 0, 0)),  # 256, 272, 512
    ((129, 1000, 33 * 64), (0, 0, 0), (0, 1, 0)), ((129, 1000, 40 * 64), (0, 0, 0), (0, 1, 0)), ((129, 1000, 41 * 64), (0, 1, 0), (0, 1, 1)),  # into the second round
    ((129, 1000, 43 * 64), (0, 1, 0), (0, 1, 1)), ((129, 1000, 44 * 64), (0, 1, 1), (0, 1, 1)), ((129, 1000, 55 * 64), (0, 1, 1), (0, 1, 1)),
    ((129, 1000, 56 * 64), (1, 1, 1), (1, 1, 1)), ((129, 1000, 64 * 64), (1, 1, 1), (1, 1, 1)), ((129, 1000, 65 * 64), (0, 1, 1), (0, 1, 1))])
@pytest.mark.parametrize("stats", [False, True])
def test_one_kernel_or_two(mp8, dims, own, own_stats, stats):  # noqa: F811
    import torch
    M, N, K = dims
    e8 = lambda *s: torch.zeros(s, dtype=torch.uint8, device="cuda")
    a, b, g8 = e8(M, K), e8(M, N), e8(K, N)
    w, m, v = (torch.zeros(K * N, dtype=t, device="cuda") for t in (torch.float16, torch.float32, torch.float32))
    for rule, one in zip(RULES, own_stats if stats else own):
        kw = dict(g8_out=g8, flags=TN, g_round=mp8.SR, w_round=mp8.SR, stats=mp8.new_stats() if stats else None)
        call = {"sgd": lambda: mp8.wgrad_update_fp16_sr(M, N, K, a, b, w, 1e-3, 1.0, **kw),
                "momentum": lambda: mp8.wgrad_momentum_fp16_sr(M, N, K, a, b, w, m, 1e-3, 1.0, 0.9, **kw),
                "adam": lambda: mp8.wgrad_adam_fp16_sr(M, N, K, a, b, w, m, v, 1e-3, 1.0, 1, **kw)}[rule]
        call()
        torch.cuda.synchronize()
        names = launches(call)
        assert len(names) == (1 if one else 2) and ("gemm_any_update" in names[0]) == bool(one), (rule, names)


@pytest.mark.parametrize("dims", [(129, 24, 2048), (300, 104, 1001), (65, 1000, 2047), (130, 1000, 2811), (200, 1016, 3585)])   # 32, 32, 512, 704, 912 tiles
@pytest.mark.parametrize("rounding", ["RNE", "SR"])
def test_without_statistics(mp8, dims, rounding):  # noqa: F811
    """Bit for bit the gradient and the update of the two calls."""
    import torch
    M, N, K = dims
    rng, mode = np.random.default_rng(sum(dims)), getattr(mp8, rounding)
    a, b = (gpu((rng.integers(0, 256, s).astype(np.uint8) & 0x83) | 0x38) for s in ((M, K), (M, N)))
    n = K * N
    w0, m0, v0 = (rng.standard_normal(n) * 0.02).astype(np.float16), rng.standard_normal(n).astype(np.float32) * 1e-3, rng.random(n).astype(np.float32) * 1e-6
    for rule in RULES:
        res = []
        for fused in (True, False):
            w, m, v, g, w8 = gpu(w0), gpu(m0), gpu(v0), *(torch.full((n + 16,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(2))
            state = [m][:rule != "sgd"] + [v][:rule == "adam"]
            u = dict(w_round=mode, w_seed=4, w_offset=2, w8_out=w8[:n])
            kw = dict(g8_out=g[:n], alpha=0.25, g_round=mode, flags=TN, g_seed=3, g_offset=1, **u)
            tail = {"sgd": (), "momentum": (0.9,), "adam": (7,)}[rule]
            if fused:
                call = getattr(mp8, {"sgd": "wgrad_update", "momentum": "wgrad_momentum", "adam": "wgrad_adam"}[rule] + "_fp16_sr")
                call(M, N, K, a, b, w, *state, 1e-3, 2.0 ** -8, *tail, **kw)
            else:
                mp8.gemm_fp8(mp8.WGRAD, M, N, K, a, b, out8=g[:n], alpha=0.25, round=mode, flags=TN, seed=3, offset=1)
                call = getattr(mp8, {"sgd": "sgd_update", "momentum": "sgd_momentum", "adam": "adam"}[rule] + "_fp16_sr")
                call(w, *state, g[:n], 1e-3, 2.0 ** -8, *tail, round=mode, seed=4, offset=2, w8_out=w8[:n])
            torch.cuda.synchronize()
            res.append([host(t) for t in (w.view(torch.int16), m.view(torch.int32), v.view(torch.int32), g, w8)])
        assert all(np.array_equal(p, q) for p, q in zip(*res)), rule
