"""Which forward calls quantise their activations inside the GEMM with several column tiles: only where the
two launches take longer."""
import numpy as np
import pytest

import oracle
from captured import launches
from test_gpu_fused_quantize_gemm import activations, finite_codes, mp8, run_fused, separate_calls  # noqa: F401  (mp8: fixture)

pytestmark = pytest.mark.gpu

X_SR, X_SAT, X_STATS = dict(x_round=oracle.SR), dict(x_flags=1), dict(x_stats=True)
OUT_SR, OUT_SAT, OUT_STATS, ACC1, ACC2, OUT_T = (dict(round=oracle.SR), dict(flags=1), dict(stats=True), dict(acc_mode=1),
                                                 dict(acc_mode=2), dict(out8_t=True))


@pytest.mark.parametrize("shape,options,kernels", [
    ((256, 256, 256), {}, 1), ((1, 256, 128), {}, 1), ((15, 256, 256), {}, 2), ((16, 256, 256), {}, 1),
    ((255, 256, 384), {}, 2), ((256, 256, 384), {}, 1), ((4096, 272, 128), {}, 2), ((256, 256, 640), {}, 2),
    # every column tile would draw the random numbers again, saturate again ...
    ((64, 16384, 256), X_SR, 2), ((4096, 256, 128), X_SR, 2), ((64, 1024, 128), X_SAT, 2), ((4096, 256, 256), X_SAT, 2),
    ((512, 256, 128), X_STATS, 2), ((1024, 256, 256), X_STATS, 1), ((4096, 256, 512), X_STATS, 2),
    # the complete epilogue
    ((64, 1024, 128), OUT_SR, 1), ((64, 1024, 128), OUT_SAT, 1), ((64, 1024, 128), ACC1, 1), ((64, 1024, 128), OUT_T, 1),
    ((4096, 256, 128), ACC2, 2), ((256, 256, 256), OUT_SR, 2), ((1024, 256, 256), OUT_STATS, 1), ((1024, 256, 512), ACC1, 2),
    ((2048, 256, 512), ACC1, 1), ((2048, 256, 512), OUT_T, 2), ((4096, 256, 512), OUT_T, 1), ((4096, 256, 512), OUT_SAT, 2),
    # one column tile: always
    ((64, 128, 256), X_SR, 1), ((64, 128, 1280), ACC2, 1)])
def test_one_kernel_or_two(mp8, shape, options, kernels):  # noqa: F811
    import torch
    M, N, K = shape
    empty = lambda *s: torch.zeros(s, dtype=torch.uint8, device="cuda")
    x, x8, w8, out = torch.zeros((M, K), device="cuda"), empty(M, K), empty(K, N), empty(M, N)
    kw = {k: mp8.new_stats() if k in ("stats", "x_stats") else empty(N, M) if k == "out8_t" else v for k, v in options.items()}
    if "acc_mode" in kw:
        kw["acc"] = torch.zeros((M, N), device="cuda")
    ws = empty(max(16, 4 * M * N, mp8.gemm_fp8_workspace_bytes(mp8.FWD, M, N, K)))
    call = lambda: mp8.quantize_gemm_fwd_fp8(M, N, K, x, x8, w8, out8=out, workspace=ws, **kw)
    call()
    torch.cuda.synchronize()
    names = launches(call)
    assert len(names) == kernels and ("gemm_qfwd" in names[0]) == (kernels == 1), names


@pytest.mark.parametrize("shape,x_stats,out", [((1024, 272, 256), True, {}), ((1025, 144, 128), True, dict(round=oracle.SR, seed=3)),
                                               ((130, 272, 128), False, dict(round=oracle.SR, seed=3)), ((2050, 144, 384), False, {})])
def test_column_tiles_with_statistics(mp8, shape, x_stats, out):  # noqa: F811
    """Statistics of both tensors and the complete epilogue, special values among the activations: bit for bit the two calls."""
    M, N, K = shape
    rng = np.random.default_rng(M + N + K)
    x, w8 = activations(rng, (M, K), specials=True), finite_codes(rng, (K, N))
    x8, _, out8, xst, st = run_fused(mp8, x, w8, want_acc=False, with_x_stats=x_stats, x_scale=2.0, alpha=0.25, **out)
    s8, sout, sxst, sst = separate_calls(mp8, x, w8, dict(scale=2.0), dict(alpha=0.25, **out))
    assert np.array_equal(s8, x8) and np.array_equal(sout, out8) and st == sst and (not x_stats or xst == sxst)
