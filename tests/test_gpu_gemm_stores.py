"""Where a GEMM's results are stored past the L2 and where into it: the same numbers on both sides of each line."""
import pytest

from test_gpu_gemm_ragged import ROW, TN, mp8  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


def run(mp8, rows, cols, kc, layout, alpha, accumulate, stats):  # noqa: F811
    """FP32 sums and codes of one call, or of one and a second that adds to it; and the codes that the Q node gives for those sums."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(rows + cols + kc)
    a, b = ((torch.randn(n * kc, generator=gen, device="cuda") * 2).to(torch.float8_e5m2).view(torch.uint8) for n in (rows, cols))
    n = rows * cols
    out, want = (torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(2))
    acc = torch.full((n + 16,), 3.0, device="cuda")
    ws = torch.empty(max(16, mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc)), dtype=torch.uint8, device="cuda")
    st, st_want = (mp8.new_stats() if stats else None for _ in range(2))
    call = lambda mode, s: mp8.gemm_fp8(mp8.FWD, rows, cols, kc, a, b, out8=out[:n], acc=acc[:n], acc_mode=mode, alpha=alpha, flags=layout, workspace=ws, stats=s)
    call(1, None if accumulate else st)
    once = acc[:n].clone()
    if accumulate:
        call(2, st)
    mp8.quantize_e5m2(acc[:n].view(rows, cols), want[:n].view(rows, cols), scale=alpha, stats=st_want)
    torch.cuda.synchronize()
    assert torch.equal(out, want) and bool((acc[n:] == 3.0).all())
    assert torch.equal(acc[:n], once * 2 if accumulate else once)      # (twice the same sum is exact)
    if stats:
        assert mp8.read_stats(st) == mp8.read_stats(st_want)
    return once, a, b


# FP32 results of 32 MB and a little more; tiles of 64x64 and 128x128
@pytest.mark.parametrize("rows,cols", [(48, 32), (1024, 1040), (4096, 2048), (4112, 2048)])
@pytest.mark.parametrize("kc", [128, 384, 400])
@pytest.mark.parametrize("layout", [ROW, TN])
def test_added_to(mp8, rows, cols, kc, layout):  # noqa: F811
    run(mp8, rows, cols, kc, layout, 2.0 ** -4, True, False)


# one round of 64x64 tiles, and one tile more
@pytest.mark.parametrize("rows,cols,kc", [(64, 64, 128), (1024, 1024, 256), (1088, 1024, 256), (512, 496, 400), (1088, 976, 400)])
@pytest.mark.parametrize("accumulate,stats", [(False, False), (False, True), (True, False), (True, True)])
def test_codes_of_64x64_tiles(mp8, rows, cols, kc, accumulate, stats):  # noqa: F811
    import torch
    once, a, b = run(mp8, rows, cols, kc, TN, 2.0 ** -5, accumulate, stats)
    out, want = (torch.zeros(rows * cols, dtype=torch.uint8, device="cuda") for _ in range(2))
    kw = dict(round=mp8.SR, seed=3, offset=9)
    mp8.gemm_fp8(mp8.FWD, rows, cols, kc, a, b, out8=out, alpha=2.0 ** -5, flags=TN, stats=mp8.new_stats() if stats else None, **kw)
    mp8.quantize_e5m2(once.view(rows, cols), want.view(rows, cols), scale=2.0 ** -5, **kw)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
