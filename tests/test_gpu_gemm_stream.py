"""Outputs of more 256x256 tiles than CUs, codes to nearest: the kernel whose workgroups take several tiles gives the bits of
the kernels that take one."""
import numpy as np
import pytest

from captured import launches
from test_gpu_gemm_ragged import BTN, ROW, TN, codes, mp8, oracle  # noqa: F401 (the fixture)
from gpu_util import host

pytestmark = pytest.mark.gpu


def gemm(mp8, a, b, rows, cols, kc, layout, **kw):  # noqa: F811
    return lambda: mp8.gemm_fp8(mp8.FWD, rows, cols, kc, a, b, **{"flags": layout, **kw})


@pytest.mark.parametrize("rows,cols,kc,layout,stream", [
    (16384, 1024, 1024, ROW, False), (16640, 1024, 1024, ROW, False),               # 256 tiles, 260: the second round nearly empty
    (16384, 1536, 2048, ROW, False),                                                # three quarters of two rounds
    (25088, 1024, 384, ROW, True), (24832, 1024, 384, ROW, False),                  # 392 tiles, 388
    (25088, 1024, 256, ROW, False), (25088, 1024, 256, BTN, True), (25088, 1024, 256, TN, True), (25088, 1024, 128, BTN, False),
    (16384, 3072, 256, ROW, False), (16384, 4096, 256, ROW, True)])                 # two stages, row-major: 768 tiles, 1024
def test_which_kernel(mp8, rows, cols, kc, layout, stream):  # noqa: F811
    import torch
    u8 = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")
    a, b, out = u8(rows * kc), u8(cols * kc), u8(rows * cols)
    plain = launches(gemm(mp8, a, b, rows, cols, kc, layout, out8=out))
    assert len(plain) == 1 and ("gemm_stream" in plain[0]) == stream
    for kw in (dict(round=mp8.SR), dict(stats=mp8.new_stats()), dict(flags=layout | mp8.FLAG_SATURATE)):
        assert not any("gemm_stream" in n for n in launches(gemm(mp8, a, b, rows, cols, kc, out8=out, **{"layout": layout, **kw})))


# tiles at the edges of the matrix, the fewest stages, odd and even numbers of them, two to five tiles per workgroup; alpha 1 and not
@pytest.mark.parametrize("layout", [ROW, BTN, TN])
@pytest.mark.parametrize("rows,cols,kc,alpha", [
    (4352, 4112, 256, 1.0), (16416, 4096, 384, 1.0), (5000, 4080, 640, 0.25), (257 * 256, 272, 1152, 0.03), (20464, 4096, 512, 1.0),
    (8192, 9216, 256, 2.0 ** -6)])
def test_same_bits_as_one_tile_per_workgroup(mp8, rows, cols, kc, alpha, layout):  # noqa: F811
    import torch
    rows = (rows + 15) // 16 * 16
    rng = np.random.default_rng(rows + cols + kc)
    draw = lambda n: torch.from_numpy(rng.integers(0, 0x44, n, dtype=np.uint8) | (rng.integers(0, 2, n, dtype=np.uint8) << 7)).cuda()
    a, b = draw(rows * kc), draw(cols * kc)
    a[::100003], b[::300007] = 0x7C, 0x7E                                          # infinities and NaN
    tile = 1
    assert mp8.gemm_fp8_plan(mp8.FWD, rows, cols, kc, layout, tile)[0] == "256x256x128s2"
    n = rows * cols
    out, one = (torch.full((n + 256,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(2))
    call = gemm(mp8, a, b, rows, cols, kc, layout, out8=out[:n], alpha=alpha, tile_config=tile, split_k=1)
    assert "gemm_stream" in launches(call)[0]
    stats = mp8.new_stats()
    gemm(mp8, a, b, rows, cols, kc, layout, out8=one[:n], alpha=alpha, tile_config=tile, split_k=1, stats=stats)()   # statistics: the other kernel
    for _ in range(3):
        out.fill_(0xAA)
        call()
        torch.cuda.synchronize()
        assert torch.equal(out, one)
    assert 0 < mp8.read_stats(stats)[1] < n // 2
    sub = rng.choice(rows, 3, replace=False)
    x = host(a).reshape((kc, rows) if layout == TN else (rows, kc))
    w = host(b).reshape((cols, kc) if layout == ROW else (kc, cols))
    ref, absref = oracle.gemm_ref(np.ascontiguousarray((x.T if layout == TN else x)[sub]), np.ascontiguousarray(w if layout == ROW else w.T))
    want, _ = oracle.quantize_e5m2(ref.astype(np.float32), scale=alpha)
    got = host(out[:n]).reshape(rows, cols)[sub]
    ok = np.isfinite(ref)
    assert (got[ok] != want[ok]).mean() < 1e-2 and np.array_equal(got[np.isnan(ref)], np.full(np.isnan(ref).sum(), 0x7F, np.uint8))
