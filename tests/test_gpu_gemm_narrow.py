"""GPU parity: FP32 tiles and FP32 results of outputs with few columns or rows, on each tile kernel."""
import numpy as np
import pytest

import oracle
from test_gpu_gemm import mp8  # noqa: F401  (fixture)
from test_gpu_gemm_outputs import exact_operand, run

pytestmark = pytest.mark.gpu

TILES = ["256x256x128s2", "256x128x128s3", "128x256x128s3", "128x128x128s2", "128x128x128s4", "64x128x128s3", "128x64x128s2", "64x64x128s2", "128x128x128k"]


# columns: FP32 tiles in rows of four lanes and more, and by a half / a whole band; rows: none, one, some of a band
@pytest.mark.parametrize("name", TILES)
@pytest.mark.parametrize("rows,cols", [(200, 1), (70, 4), (33, 7), (129, 13), (64, 16), (1, 17), (100, 30), (257, 32), (40, 33), (65, 62), (200, 80), (8, 130), (300, 259)])
def test_fp32_tiles_of_narrow_outputs(mp8, name, rows, cols):  # noqa: F811
    """FP32 result alone, and codes with it where it is stored and where it is added to: bit for bit (sums that FP32 holds exactly)."""
    rng = np.random.default_rng(rows * cols)
    a, b = exact_operand(rng, (rows, 256)), exact_operand(rng, (cols, 256))
    acc0 = rng.integers(-64, 65, (rows, cols)).astype(np.float32)
    ref = oracle.gemm_ref(a, b, want_abs=False)[0]
    tile = mp8.gemm_tile_configs().index(name) + 1
    for mode in (1, 2):
        want = ref + (acc0 if mode == 2 else 0)
        out, _, acc = run(mp8, a, b, acc_mode=mode, acc0=acc0, tile_config=tile, split_k=1)
        assert np.array_equal(acc.astype(np.float64), want) and np.array_equal(out, oracle.round_ref_e5m2(want))
    if "k" not in name:
        out, _, _ = run(mp8, a, b, tile_config=tile, split_k=2)
        assert np.array_equal(out, oracle.round_ref_e5m2(ref))


# more than half of the CUs with a tile: the FP32 result line by line; fewer, or rows that fill no tile of a half-precision kernel: with the codes
@pytest.mark.parametrize("rows,cols,kc", [(1024, 1024, 128), (1024, 512, 128), (1088, 528, 144), (640, 528, 144), (8320, 64, 80), (8320, 48, 80), (48, 8320, 80), (64, 8320, 80)])
@pytest.mark.parametrize("rounding", [oracle.RNE, oracle.SR])
def test_fp32_result_on_either_path(mp8, rows, cols, kc, rounding):  # noqa: F811
    rng = np.random.default_rng(rows + cols + kc)
    a, b = exact_operand(rng, (rows, kc)), exact_operand(rng, (cols, kc))
    acc0 = rng.integers(-64, 65, (rows, cols)).astype(np.float32)
    ref = oracle.gemm_ref(a, b, want_abs=False)[0]
    for mode in (1, 2):
        want = (ref + (acc0 if mode == 2 else 0)).astype(np.float32)
        out, _, acc = run(mp8, a, b, acc_mode=mode, acc0=acc0, round=rounding, seed=5, offset=6)
        codes, _ = oracle.quantize_e5m2(want, mode=rounding, seed=5, offset=6)
        assert np.array_equal(acc, want) and np.array_equal(out, codes)
