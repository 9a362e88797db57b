"""Where FP32 and transposed results are made -- in the epilogue, by a finishing pass, by a pass over the codes --, and that
each route gives the same bits."""
import numpy as np
import pytest

import oracle
from captured import launches
from gpu_util import gpu, host
from test_gpu_gemm import mp8  # noqa: F401  (fixture)
from test_gpu_gemm_outputs import exact_operand

pytestmark = pytest.mark.gpu

NEAREST, SR = oracle.RNE, oracle.SR


def kernels(mp8, rows, cols, kc, acc_mode=0, want_t=True, rounding=NEAREST, km=False):  # noqa: F811
    """What a call launches: 'g'emm, 'f'inishing pass, pass over the codes 't'."""
    import torch
    e8 = lambda *s: torch.empty(s, dtype=torch.uint8, device="cuda")
    a, b = (e8(kc, rows), e8(kc, cols)) if km else (e8(rows, kc), e8(cols, kc))
    a.zero_(), b.zero_()
    op, dims = (mp8.WGRAD, (kc, cols, rows)) if km else (mp8.FWD, (rows, cols, kc))
    ws = e8(max(16, 4 * rows * cols, mp8.gemm_fp8_workspace_bytes(op, *dims)))
    kw = dict(out8=e8(rows, cols), out8_t=e8(cols, rows) if want_t else None, acc=torch.zeros((rows, cols), device="cuda") if acc_mode else None,
              acc_mode=acc_mode, round=rounding, flags=mp8.FLAG_CONTRACTION_MAJOR if km else 0, workspace=ws)
    call = lambda: mp8.gemm_fp8(op, *dims, a, b, **kw)
    call()
    torch.cuda.synchronize()
    return "".join("f" if "splitk_finish" in n else "t" if "transpose_codes" in n else "g" for n in launches(call))


@pytest.mark.parametrize("dims,options,expected", [
    # transposed copies of what a finishing pass rounds: large and filled ones by the pass over the codes
    ((64, 64, 16384), {}, "gf"), ((512, 512, 8192), {}, "gf"), ((600, 600, 256), {}, "gf"), ((1000, 1000, 256), {}, "gft"),
    ((20000, 60, 256), {}, "gf"), ((20000, 100, 256), {}, "gft"), ((1000, 48, 8192), {}, "gf"),
    # of the 256x256 tiles: always; of other aligned kernels: codes to nearest, large for the length of the contraction
    ((4096, 4096, 1024), {}, "gt"), ((4096, 4096, 1024), dict(rounding=SR), "gt"), ((2048, 2048, 1024), {}, "g"),
    ((4096, 4096, 256), {}, "g"), ((8192, 4096, 256), {}, "gt"), ((8192, 4096, 256), dict(rounding=SR), "g"), ((8192, 4096, 128), {}, "g"),
    ((8192, 4096, 128), dict(km=True), "gt"), ((4096, 4096, 144), {}, "g"), ((4096, 4096, 528), {}, "gt"), ((4096, 4096, 528), dict(rounding=SR), "g"),
    # never of the kernel for unaligned rows, which has one epilogue
    ((2900, 2900, 500), {}, "g"), ((4096, 4088, 200), dict(rounding=SR), "g"),
    # tiles mostly beyond the matrix
    ((65536, 48, 1024), dict(acc_mode=1, want_t=False), "gf"), ((65536, 112, 1024), dict(acc_mode=1, want_t=False), "g"),
    ((65536, 160, 1024), dict(acc_mode=2, want_t=False), "gf"), ((65536, 400, 1024), dict(acc_mode=2, want_t=False), "g"),
    ((65536, 48, 1024), dict(rounding=SR), "gf"), ((65536, 64, 1024), dict(rounding=SR), "g"), ((262144, 48, 1024), {}, "gt"),
    ((32768, 16, 512), dict(rounding=SR), "gf"), ((65536, 16, 512), dict(rounding=SR), "g"), ((65536, 16, 512), dict(acc_mode=2, want_t=False), "gf"),
    ((32768, 32, 2048), dict(acc_mode=2, want_t=False), "gf"), ((32768, 32, 512), dict(acc_mode=2, want_t=False), "g"),
    ((7, 40000, 256), {}, "gf"), ((16, 40000, 256), {}, "g"), ((16, 40000, 256), dict(acc_mode=2, want_t=False), "gf")])
def test_routes(mp8, dims, options, expected):  # noqa: F811
    assert kernels(mp8, *dims, **options) == expected


# the routes again on values: pass over the codes behind either kernel, with FP32 result beside it; finishing pass for poorly filled tiles
@pytest.mark.parametrize("rows,cols,kc,acc_mode,want_t,rounding", [
    (4096, 2112, 1024, 1, True, SR), (3584, 3600, 1024, 2, True, NEAREST), (1100, 720, 128, 0, True, SR), (20000, 100, 128, 1, True, NEAREST),
    (65536, 48, 1024, 2, True, SR), (65600, 48, 1024, 1, True, NEAREST), (32768, 16, 512, 2, True, SR), (7, 40000, 256, 1, True, SR), (524288, 16, 128, 0, True, NEAREST)])
def test_results_by_route(mp8, rows, cols, kc, acc_mode, want_t, rounding):  # noqa: F811
    """acc against exact sums on sampled rows, codes the oracle's rounding of acc, the transposed copy the codes'."""
    import torch
    rng = np.random.default_rng(rows + cols)
    a, b = exact_operand(rng, (rows, kc)), exact_operand(rng, (cols, kc))
    if kc > 256:
        a[:, rng.random(kc) < 0.75] = 0                       # keeps every partial sum exact in FP32
    acc0 = torch.full((rows, cols), 32.0, device="cuda")
    acc = acc0.clone()
    out, out_t = (torch.full(s, 0xAA, dtype=torch.uint8, device="cuda") for s in ((rows, cols), (cols, rows)))
    ws = torch.empty(max(4 * rows * cols, mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc)), dtype=torch.uint8, device="cuda")
    ad, bd = gpu(a), gpu(b)
    kw = dict(round=rounding, seed=3, offset=4, workspace=ws)
    mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ad, bd, out8=out, out8_t=out_t if want_t else None, acc=acc if acc_mode else None, acc_mode=acc_mode, **kw)
    plain = torch.empty_like(out)
    mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ad, bd, out8=plain, **kw)
    some = np.unique(np.concatenate([[0, rows - 1], rng.integers(0, rows, 30)]))
    ref = oracle.gemm_ref(a, b, row_idx=some, want_abs=False)[0]
    want = (ref + (32.0 if acc_mode == 2 else 0.0)).astype(np.float32)
    if acc_mode:
        assert np.array_equal(host(acc[some]), want)
        full = host(acc)
        if full.size <= 1 << 23:
            codes, _ = oracle.quantize_e5m2(full, mode=rounding, seed=3, offset=4)
            assert np.array_equal(host(out), codes)
    if acc_mode != 2:
        assert bool((out == plain).all())
    if rounding == NEAREST:
        assert np.array_equal(host(out[some]), oracle.round_ref_e5m2(want.astype(np.float64)))
    assert bool((out_t == out.t()).all())
