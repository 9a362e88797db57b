"""GPU parity: FP32 and transposed results beside the codes -- in the epilogue, by a finishing pass, and the transposing
pass over finished codes."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu, host
from test_gpu_gemm import mp8  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def exact_operand(rng, shape):
    """{1, 1.25, 1.5, 1.75} * 2^{0..3}, both signs: FP32 holds their sums exactly, in any order."""
    return ((rng.integers(0, 2, shape) << 7) | (rng.integers(15, 19, shape) << 2) | rng.integers(0, 4, shape)).astype(np.uint8)


def run(mp8, a, b, acc_mode=0, acc0=None, want_t=False, **kw):  # noqa: F811
    import torch
    rows, cols = a.shape[0], b.shape[0]
    out = torch.full((rows * cols + 64,), 0xAA, dtype=torch.uint8, device="cuda")
    out_t = torch.full((rows * cols + 64,), 0x55, dtype=torch.uint8, device="cuda")
    acc = gpu(acc0.reshape(-1)) if acc0 is not None else torch.zeros(rows * cols, device="cuda")
    ws = torch.empty(4 * 4 * rows * cols + 16, dtype=torch.uint8, device="cuda")
    mp8.gemm_fp8(mp8.FWD, rows, cols, a.shape[1], gpu(a), gpu(b), out8=out[: rows * cols], out8_t=out_t[: rows * cols] if want_t else None,
                 acc=acc if acc_mode else None, acc_mode=acc_mode, workspace=ws, **kw)
    torch.cuda.synchronize()
    assert bool((out[rows * cols:] == 0xAA).all()) and bool((out_t[rows * cols:] == 0x55).all()), "wrote past the end"
    return host(out[: rows * cols]).reshape(rows, cols), host(out_t[: rows * cols]).reshape(cols, rows), host(acc).reshape(rows, cols)


# split contractions: the transposing pass, in 16-byte pieces and in any; 3 columns: the finishing pass itself
@pytest.mark.parametrize("rows,cols", [(128, 128), (16, 144), (144, 16), (129, 131), (1, 4), (5, 133), (260, 7), (127, 64), (33, 3)])
def test_transposed_copy_of_a_split_contraction(mp8, rows, cols):  # noqa: F811
    rng = np.random.default_rng(rows + cols)
    a, b = exact_operand(rng, (rows, 256)), exact_operand(rng, (cols, 256))
    want = oracle.round_ref_e5m2(oracle.gemm_ref(a, b, want_abs=False)[0])
    tile = mp8.gemm_tile_configs().index("64x64x128s2") + 1
    out, out_t, _ = run(mp8, a, b, want_t=True, tile_config=tile, split_k=2)
    assert np.array_equal(out, want) and np.array_equal(out_t, want.T)


@pytest.mark.parametrize("rows,cols,kc", [(2912, 2896, 128), (2899, 2900, 144), (2048, 4096, 128)])
def test_transposed_copy_of_a_large_result(mp8, rows, cols, kc):  # noqa: F811
    """Around 2^23 outputs, where the copy becomes a pass of its own."""
    rng = np.random.default_rng(rows)
    a, b = exact_operand(rng, (rows, kc)), exact_operand(rng, (cols, kc))
    out, out_t, _ = run(mp8, a, b, want_t=True, round=mp8.SR, seed=3, offset=4)
    plain, _, _ = run(mp8, a, b, round=mp8.SR, seed=3, offset=4)
    assert np.array_equal(out, plain) and np.array_equal(out_t, out.T)


# the tile kernels by name; 200 rows and 144 columns leave a partial tile of each kind
@pytest.mark.parametrize("name", ["256x256x128s2", "256x128x128s3", "128x128x128s2", "64x128x128s3", "128x64x128s2", "64x64x128s2",
                                  "64x64x128w", "32x64x128w", "32x32x128w", "128x128x128p", "128x128x128k"])
@pytest.mark.parametrize("mode", [1, 2])
def test_fp32_result_beside_the_codes(mp8, name, mode):  # noqa: F811
    """acc stored or added to in the epilogue, codes of the sum, with and without a transposed copy: bit for bit."""
    rng = np.random.default_rng(mode)
    rows, cols, kc = 200, 144, 256
    a, b = exact_operand(rng, (rows, kc)), exact_operand(rng, (cols, kc))
    acc0 = rng.integers(-64, 65, (rows, cols)).astype(np.float32)
    ref = oracle.gemm_ref(a, b, want_abs=False)[0] + (acc0 if mode == 2 else 0)
    tile = mp8.gemm_tile_configs().index(name) + 1
    for want_t in (False, True):
        out, out_t, acc = run(mp8, a, b, acc_mode=mode, acc0=acc0, want_t=want_t, tile_config=tile, split_k=1)
        assert np.array_equal(acc.astype(np.float64), ref)
        want = oracle.round_ref_e5m2(ref)
        assert np.array_equal(out, want) and (not want_t or np.array_equal(out_t, want.T))
