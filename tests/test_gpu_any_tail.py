"""Unaligned GEMMs whose contraction ends inside a stage: contraction-major operands, whose last sixteen rows are read again and
put where they belong, give the bits that row-major ones give, whose rows end inside a chunk."""
import numpy as np
import pytest

from gpu_util import assert_as_precise_as_fp32, host
from test_gpu_gemm_ragged import BTN, ROW, TN, codes, mp8, oracle, stored  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


# one row of the last sixteen, all of them, and each side of that, in the first, the second and the sixth stage; slices; tiles at the edges
@pytest.mark.parametrize("kc", [16, 17, 31, 32, 33, 112, 113, 127, 129, 143, 144, 145, 255, 641, 655, 657, 5001])
@pytest.mark.parametrize("rows,cols", [(16, 17), (63, 65), (65, 127), (40, 71)])
def test_every_layout_gives_the_same_bits(mp8, rows, cols, kc):  # noqa: F811
    import torch
    rng = np.random.default_rng(kc * 131 + rows)
    a, b = codes(int(rng.integers(1 << 30)), (rows, kc)), codes(int(rng.integers(1 << 30)), (cols, kc))
    need, n, got = mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc), rows * cols, []
    for layout in (ROW, BTN, TN):
        ag, lda = stored(a, layout == TN, pad=3, shift=1)        # (NaN codes behind every row)
        bg, ldb = stored(b, layout != ROW, pad=5)
        for scratch in {0, need}:
            acc = torch.full((n + 16,), 7.0, device="cuda")
            ws = torch.empty(scratch, dtype=torch.uint8, device="cuda") if scratch else None
            mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, acc=acc[:n], acc_mode=1, flags=layout, lda=lda, ldb=ldb, workspace=ws)
            torch.cuda.synchronize()
            assert bool((acc[n:] == 7.0).all())
            got.append(host(acc[:n]))
    ref, _ = oracle.gemm_ref(a, b)
    assert_as_precise_as_fp32(got[0].reshape(rows, cols), a, b, ref, f"{rows} x {cols} x {kc}")
    assert all(np.array_equal(g.view(np.uint32), got[0].view(np.uint32)) for g in got[1:])


# one to two tiles of 64 x 64 for each CU: from 24 stages on (a contraction-major) and from 56 the loads are waited for
@pytest.mark.parametrize("kc", [23 * 128 + 127, 24 * 128, 55 * 128 + 127, 56 * 128 + 1])
@pytest.mark.parametrize("rows,cols", [(65, 8129), (1030, 1001)])
def test_operands_waited_for(mp8, rows, cols, kc):  # noqa: F811
    import torch
    a, b = codes(kc, (rows, kc)), codes(kc + 1, (cols, kc))
    got = []
    for layout in (ROW, BTN, TN):
        ag, lda = stored(a, layout == TN, pad=3, shift=1)
        bg, ldb = stored(b, layout != ROW, pad=5)
        acc = torch.full((rows * cols + 16,), 7.0, device="cuda")
        mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, acc=acc[:rows * cols], acc_mode=1, flags=layout, lda=lda, ldb=ldb)
        torch.cuda.synchronize()
        assert bool((acc[rows * cols:] == 7.0).all())
        got.append(host(acc[:rows * cols]).view(np.uint32))
    ref, _ = oracle.gemm_ref(a[:64], b[:64])
    assert_as_precise_as_fp32(got[0].view(np.float32).reshape(rows, cols)[:64, :64], a[:64], b[:64], ref, f"{rows} x {cols} x {kc}")
    assert all(np.array_equal(g, got[0]) for g in got[1:])
