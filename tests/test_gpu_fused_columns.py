"""GPU parity: the forward GEMM that quantises its activations with several column tiles (small layers)."""
import numpy as np
import pytest

import oracle
from gpu_util import check_outputs
from test_gpu_fused_quantize_gemm import activations, finite_codes, mp8, run_fused, separate_calls  # noqa: F401  (mp8: fixture)

pytestmark = pytest.mark.gpu


# last column tile of 16 columns and whole ones; one row, a ragged last row tile; one to four stages (four from 256
# rows on, else the two calls); the most tiles it takes (128) and one more
@pytest.mark.parametrize("shape", [(64, 144, 128), (1, 256, 256), (255, 272, 512), (256, 272, 512), (333, 1040, 384),
                                   (4096, 256, 128), (4033, 272, 128)])
def test_fused_forward_column_tiles(mp8, shape):  # noqa: F811
    """Every option at once, with special values, and the lean variant: bit for bit the two calls it stands for (x8,
    output, statistics of both), x8 the oracle's, the accumulator within tolerance of the oracle's product."""
    M, N, K = shape
    rng = np.random.default_rng(M + N + K)
    x, w8 = activations(rng, (M, K), specials=True), finite_codes(rng, (K, N))
    q = dict(round=mp8.SR, flags=1, seed=11, offset=5)
    g = dict(alpha=0.25, round=mp8.SR, seed=3, offset=9, flags=1)
    x8, _, out8, xst, st = run_fused(mp8, x, w8, want_acc=False, x_scale=2.0, x_round=mp8.SR, x_flags=1, x_seed=11, x_offset=5, **g)
    ost = oracle.Stats()
    want8, _ = oracle.quantize_e5m2(x, scale=2.0, mode=oracle.SR, flags=1, seed=11, offset=5, stats=ost)
    assert np.array_equal(x8, want8) and xst == ost.as_tuple()
    s8, sout, sxst, sst = separate_calls(mp8, x, w8, dict(scale=2.0, **q), dict(g))
    assert np.array_equal(s8, x8) and np.array_equal(sout, out8) and sxst == xst and sst == st
    x = activations(rng, (M, K), specials=False)
    want8, _ = oracle.quantize_e5m2(x)
    x8, acc, out8, _, _ = run_fused(mp8, x, w8, with_x_stats=False, with_stats=False)
    rows = np.unique(rng.integers(0, M, 64))
    ref, absref = oracle.gemm_ref(want8, np.ascontiguousarray(w8.T), row_idx=rows)
    assert np.array_equal(x8, want8)
    check_outputs(acc[rows], out8[rows], ref, absref, K)
    x8, _, lean, _, _ = run_fused(mp8, x, w8, want_acc=False, with_x_stats=False, with_stats=False)
    assert np.array_equal(x8, want8) and np.array_equal(lean, out8)
