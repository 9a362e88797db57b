"""GPU parity: forward and backward-data convolutions at the edges of the kernel that keeps a tile's pixel rows in
LDS -- halo widths, chunk counts, tile heights -- and the general kernels that wider images take."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu, host
from test_gpu_conv import exact_codes, interior, mp8, run_conv, to_padded  # noqa: F401  (mp8: fixture)

pytestmark = pytest.mark.gpu


# W = 29 / 30: without and with the last load of the halo; 61 / 62: the widest image it takes, the general kernels;
# 64 channels: one chunk, 128 and more: weights refilled; H such that rows are no multiple of a tile
@pytest.mark.parametrize("dims", [(1, 3, 29, 64, 64), (1, 3, 29, 192, 128), (2, 2, 30, 128, 64), (1, 5, 30, 64, 192),
                                  (1, 2, 61, 64, 128), (1, 3, 61, 256, 64), (1, 2, 62, 64, 128), (1, 3, 62, 192, 64),
                                  (1, 1, 1, 64, 64)])
def test_conv_rows_in_lds_exact_sums(mp8, dims):  # noqa: F811
    """Sums that FP32 holds exactly, in any order: accumulators and codes bit for bit, with the fused epilogue of
    each kind, padding rows zero."""
    import torch
    B, H, W, Ci, Co = dims
    rng = np.random.default_rng(sum(dims))
    x, w, e = exact_codes(rng, (B, H, W, Ci)), exact_codes(rng, (3, 3, Ci, Co)), exact_codes(rng, (B, H, W, Co))
    wd = gpu(w)
    for op, a_h, name in ((mp8.FWD, x, "fwd"), (mp8.BWD_DATA, e, "bwd_data")):
        ref, _ = oracle.conv3x3_ref(name, a_h, w, want_abs=False)
        a_dev = to_padded(mp8, a_h)
        acc, out8, _ = run_conv(mp8, op, dims, a_dev, wd)
        assert np.array_equal(interior(acc, B, H, W)[0].astype(np.float64), ref), name
        out_i, out_pad = interior(out8, B, H, W)
        assert np.array_equal(out_i, oracle.round_ref_e5m2(ref)) and not out_pad.any(), name
        _, out_b, _ = run_conv(mp8, op, dims, a_dev, wd, want_acc=False)     # with statistics
        assert np.array_equal(out_b, out8), name
        plain = torch.full(out8.shape, 0xAA, dtype=torch.uint8, device="cuda")
        mp8.conv3x3_fp8(op, *dims, a_dev, wd, out8=plain)                    # rounding to nearest alone
        assert np.array_equal(host(plain), out8), name


@pytest.mark.parametrize("Ci,Co", [(64, 64), (128, 64)])
def test_conv_tall_tiles_on_three_images(mp8, Ci, Co):  # noqa: F811
    """A grid of 256-row tiles (from 384 of them on); first, middle and last image against the oracle."""
    import torch
    B, H, W = 30, 56, 56
    rng = np.random.default_rng(Ci)
    x, w, e = exact_codes(rng, (B, H, W, Ci)), exact_codes(rng, (3, 3, Ci, Co)), exact_codes(rng, (B, H, W, Co))
    wd = gpu(w)
    for op, a_h, name, cols in ((mp8.FWD, x, "fwd", Co), (mp8.BWD_DATA, e, "bwd_data", Ci)):
        out = torch.full((mp8.conv_prows(B, H, W), cols), 0xAA, dtype=torch.uint8, device="cuda")
        mp8.conv3x3_fp8(op, B, H, W, Ci, Co, to_padded(mp8, a_h), wd, out8=out)
        out_i, out_pad = interior(host(out), B, H, W)
        assert not out_pad.any(), name
        for b in (0, B // 2, B - 1):
            ref, _ = oracle.conv3x3_ref(name, a_h[b:b + 1], w, want_abs=False)
            assert np.array_equal(out_i[b:b + 1], oracle.round_ref_e5m2(ref)), (name, b)
