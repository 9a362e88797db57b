"""GEMMs on tiles of 32x32, codes to nearest: equal, bit for bit, to the FP32 result of the same tiles rounded by the Q node."""
import numpy as np
import pytest

from gpu_util import gpu, host
from test_gpu_gemm_ragged import mp8  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


# rows and columns at the edge of a tile and inside one, few and many stages; codes that overflow, vanish, and are no numbers
@pytest.mark.parametrize("rows,cols,stages", [(32, 32, 16), (1, 16, 16), (33, 48, 17), (100, 240, 40), (127, 2032, 16), (128, 2048, 32)])
@pytest.mark.parametrize("alpha", [1.0, 2.0 ** -9, 2.0 ** 12, 2.0 ** -24])
@pytest.mark.parametrize("special", [False, True])
def test_codes_of_a_32x32_tile(mp8, rows, cols, stages, alpha, special):  # noqa: F811
    import torch
    rng = np.random.default_rng(rows + cols + stages)
    kc = 128 * stages
    a, b = ((rng.integers(0, 256, s).astype(np.uint8) & 0x83) | 0x38 for s in ((rows, kc), (cols, kc)))
    if special:
        a[rows // 2, 3], b[cols // 2, 5] = 0x7C, 0x7F
    a, b, n = gpu(a), gpu(b), rows * cols
    tile = next(i for i, t in enumerate(mp8.gemm_tile_configs(), 1) if t.startswith("32x32"))
    assert mp8.gemm_fp8_plan(mp8.FWD, rows, cols, kc, 0) == (mp8.gemm_tile_configs()[tile - 1], 1)
    out, want = (torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(2))
    acc = torch.empty(n, dtype=torch.float32, device="cuda")
    mp8.gemm_fp8(mp8.FWD, rows, cols, kc, a, b, out8=out[:n], alpha=alpha)
    mp8.gemm_fp8(mp8.FWD, rows, cols, kc, a, b, acc=acc, acc_mode=1)  # (the sums, without alpha)
    mp8.quantize_e5m2(acc.view(rows, cols), want[:n].view(rows, cols), scale=alpha)
    torch.cuda.synchronize()
    assert np.array_equal(host(out), host(want))
