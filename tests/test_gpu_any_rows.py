"""Unaligned GEMMs with few tiles run in tiles of 32 rows: the kernel that is chosen, and the same bits as tiles of 64 rows give."""
import numpy as np
import pytest

from captured import launches
from gpu_util import host
from test_gpu_gemm_ragged import BTN, ROW, TN, assert_as_precise_as_fp32, codes, mp8, oracle, stored  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


def call(mp8, ag, bg, lda, ldb, rows, cols, kc, layout, **kw):  # noqa: F811
    mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, flags=layout, lda=lda, ldb=ldb, **kw)


# tiles of 64 x 64: up to 128 always, up to 384 with three stages and less
@pytest.mark.parametrize("rows,cols,kc,small", [(8192, 65, 129, True), (8193, 65, 385, False), (8192, 63, 1000, True), (8256, 63, 1000, False),
                                                (12288, 65, 384, True), (12289, 65, 384, False), (33, 1000, 2047, True)])
@pytest.mark.parametrize("layout", [ROW, BTN])
def test_which_kernel(mp8, rows, cols, kc, small, layout):  # noqa: F811
    import torch
    u8 = lambda n: torch.zeros(n + 1, dtype=torch.uint8, device="cuda")[1:]
    a, b, out = u8(rows * kc), u8(cols * kc), torch.zeros(rows * cols, dtype=torch.uint8, device="cuda")
    names = launches(lambda: call(mp8, a, b, kc, cols if layout == BTN else kc, rows, cols, kc, layout, out8=out))
    assert len(names) == 1 and "gemm_any_kernel" in names[0] and ("Li32E" in names[0]) == small, names


# rows around 32, columns around 64, contractions around a chunk and a stage, more stages than waves
@pytest.mark.parametrize("layout", [ROW, BTN])
@pytest.mark.parametrize("kc", [16, 17, 31, 113, 127, 128, 129, 143, 145, 255, 257, 384, 385, 641, 1007])
def test_same_bits_as_64_rows(mp8, kc, layout):  # noqa: F811
    import torch
    rng = np.random.default_rng(kc)
    many = 64 * 385
    a = codes(int(rng.integers(1 << 30)), (many, kc))
    ag, lda = stored(a, False, pad=3, shift=1)
    for cols in (17, 63, 64, 65, 80):
        b = codes(int(rng.integers(1 << 30)), (cols, kc))
        bg, ldb = stored(b, layout == BTN, pad=5)
        whole = torch.empty((many, cols), device="cuda")
        call(mp8, ag, bg, lda, ldb, many, cols, kc, layout, acc=whole, acc_mode=1)      # tiles of 64 rows
        for rows in (1, 31, 32, 33, 64, 65, 97):
            n = rows * cols
            acc = torch.full((n + 16,), 7.0, device="cuda")
            out, out_t = (torch.full((n + 64,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(2))
            stats = mp8.new_stats()
            call(mp8, ag, bg, lda, ldb, rows, cols, kc, layout, acc=acc[:n], acc_mode=1, out8=out[:n], out8_t=out_t[:n], round=mp8.SR, seed=5, offset=6,
                 alpha=2.0 ** -24, stats=stats)
            torch.cuda.synchronize()
            assert torch.equal(acc[:n].view(rows, cols).view(torch.int32), whole[:rows].view(torch.int32)), (rows, cols)
            assert bool((acc[n:] == 7.0).all()) and bool((out[n:] == 0xAA).all()) and bool((out_t[n:] == 0xAA).all())
            full, st = host(acc[:n]).reshape(rows, cols), oracle.Stats()
            want, _ = oracle.quantize_e5m2(full, scale=2.0 ** -24, mode=oracle.SR, seed=5, offset=6, stats=st)
            assert np.array_equal(host(out[:n]).reshape(rows, cols), want) and np.array_equal(host(out_t[:n]).reshape(cols, rows), want.T)
            assert mp8.read_stats(stats) == st.as_tuple()
        ref, _ = oracle.gemm_ref(a[:97], b)
        assert_as_precise_as_fp32(host(whole[:97]), a[:97], b, ref, f"{kc} x {cols} layout {layout}")
