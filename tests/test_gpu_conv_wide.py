"""GPU parity: forward and backward-data convolutions of images too wide for the kernel with the pixel rows in LDS, over
every tile and slicing of the general kernels; that kernel's 256-row tiles with each epilogue; row counts that no tile divides."""
import numpy as np
import pytest

import oracle
from captured import launches
from gpu_util import gpu, host
from test_gpu_conv import exact_codes, interior, mp8, run_conv, to_padded  # noqa: F401  (mp8: fixture)

pytestmark = pytest.mark.gpu


def operands(dims):
    B, H, W, Ci, Co = dims
    rng = np.random.default_rng(sum(dims))
    x, w, e = exact_codes(rng, (B, H, W, Ci)), exact_codes(rng, (3, 3, Ci, Co)), exact_codes(rng, (B, H, W, Co))
    return x, w, e


# 62: the narrowest image of the general kernels; contracted channels a multiple of 128 (a stage within one tap) in the
# forward, the backward or both directions; one and several contraction slices; 63, 70 columns: ragged last tiles
@pytest.mark.parametrize("dims", [(1, 3, 62, 128, 128), (1, 2, 62, 256, 64), (1, 2, 62, 64, 256), (2, 2, 63, 128, 192),
                                  (1, 2, 62, 256, 128), (1, 4, 70, 128, 384)])
def test_wide_images_exact_sums(mp8, dims):  # noqa: F811
    """Sums that FP32 holds exactly, in any order: accumulators and codes bit for bit, with the fused epilogue of
    each kind, padding rows zero."""
    import torch
    B, H, W, Ci, Co = dims
    x, w, e = operands(dims)
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
        ws = torch.empty(max(mp8.conv3x3_fp8_workspace_bytes(op, *dims), 16), dtype=torch.uint8, device="cuda")
        plain = torch.full(out8.shape, 0xAA, dtype=torch.uint8, device="cuda")
        mp8.conv3x3_fp8(op, *dims, a_dev, wd, out8=plain, workspace=ws)      # rounding to nearest alone
        assert np.array_equal(host(plain), out8), name


def test_wide_images_in_the_largest_tiles(mp8):  # noqa: F811
    """A grid that fills the GPU with 256x256 tiles, whole (forward) and half of each beyond the last column (backward
    data): strips of three rows -- first, middle and last image, top, middle and bottom -- against the oracle."""
    import torch
    dims = B, H, W, Ci, Co = 26, 62, 62, 128, 256
    x, w, e = operands(dims)
    wd = gpu(w)
    for op, a_h, name, cols in ((mp8.FWD, x, "fwd", Co), (mp8.BWD_DATA, e, "bwd_data", Ci)):
        a_dev = to_padded(mp8, a_h)
        plain = torch.full((mp8.conv_prows(B, H, W), cols), 0xAA, dtype=torch.uint8, device="cuda")
        ws = torch.empty(max(mp8.conv3x3_fp8_workspace_bytes(op, *dims), 16), dtype=torch.uint8, device="cuda")
        call = lambda: mp8.conv3x3_fp8(op, *dims, a_dev, wd, out8=plain, workspace=ws)
        kernels = launches(call)
        assert len(kernels) == 1 and "gemm_mfma_kernelILi256ELi256E" in kernels[0], kernels
        call()
        acc, out8, _ = run_conv(mp8, op, dims, a_dev, wd)
        assert np.array_equal(host(plain), out8), name
        (acc_i, _), (out_i, out_pad) = interior(acc, B, H, W), interior(out8, B, H, W)
        assert not out_pad.any(), name
        for b, y in ((0, 0), (0, 30), (B // 2, 17), (B - 1, H - 3)):
            y0, y1 = max(y - 1, 0), min(y + 4, H)
            ref, _ = oracle.conv3x3_ref(name, a_h[b:b + 1, y0:y1], w, want_abs=False)
            ref = ref[:, y - y0:y - y0 + 3]
            assert np.array_equal(acc_i[b:b + 1, y:y + 3].astype(np.float64), ref), (name, b, y)
            assert np.array_equal(out_i[b:b + 1, y:y + 3], oracle.round_ref_e5m2(ref)), (name, b, y)


def test_tall_tiles_with_every_epilogue(mp8):  # noqa: F811
    """256-row tiles of the kernel with the pixel rows in LDS: stochastic codes with statistics, an FP32 result beside them,
    added to, and alone; first, middle and last image against the oracle, codes and statistics of every pixel."""
    import torch
    dims = B, H, W, Ci, Co = 30, 56, 56, 64, 64
    x, w, e = operands(dims)
    wd, prows = gpu(w), mp8.conv_prows(B, H, W)
    row = np.zeros(prows, bool)
    row[:B * (H + 2) * (W + 2)].reshape(B, H + 2, W + 2)[:, 1:-1, 1:-1] = True
    for op, a_h, name in ((mp8.FWD, x, "fwd"), (mp8.BWD_DATA, e, "bwd_data")):
        a_dev = to_padded(mp8, a_h)
        ref = {b: oracle.conv3x3_ref(name, a_h[b:b + 1], w, want_abs=False)[0] for b in (0, B // 2, B - 1)}
        ws = torch.empty(max(mp8.conv3x3_fp8_workspace_bytes(op, *dims), 16), dtype=torch.uint8, device="cuda")

        def run(before, mode, sr, with_codes=True):
            out = torch.full((prows, 64), 0xAA, dtype=torch.uint8, device="cuda") if with_codes else None
            acc = torch.full((prows, 64), before, dtype=torch.float32, device="cuda") if mode else None
            st = mp8.new_stats() if sr else None
            call = lambda: mp8.conv3x3_fp8(op, *dims, a_dev, wd, out8=out, acc=acc, acc_mode=mode, round=oracle.SR if sr else oracle.RNE,
                                           seed=11, offset=5, stats=st, workspace=ws)
            assert "gemm_conv_kernelILi256E" in launches(call)[0]
            call()
            return acc, out, (mp8.read_stats(st) if sr else None)

        alone = interior(host(run(0.0, 1, False, False)[0]), B, H, W)[0]
        for b, r in ref.items():
            assert np.array_equal(alone[b:b + 1].astype(np.float64), r), (name, b)
        full = np.zeros((prows, 64), np.float32)
        full[row] = alone.reshape(-1, 64)
        for mode, sr in ((0, True), (1, True), (1, False), (2, True), (2, False)):
            total = np.where(row[:, None], full + np.float32(0.75 if mode == 2 else 0.0), np.float32(0))  # exact: multiples of 1/16
            stats = oracle.Stats()
            codes, _ = oracle.quantize_e5m2(total, mode=oracle.SR if sr else oracle.RNE, seed=11, offset=5)
            oracle.quantize_e5m2(np.ascontiguousarray(total[row]), mode=oracle.SR if sr else oracle.RNE, stats=stats)
            acc, out, got = run(0.75 if mode == 2 else float("nan"), mode, sr)
            assert np.array_equal(host(out), codes), (name, mode, sr)
            if mode:
                assert np.array_equal(host(acc)[row], total[row]), (name, mode, sr)
            if sr:
                assert got[:2] == tuple(stats.as_tuple())[:2], (name, mode)


@pytest.mark.parametrize("dims,prows", [((1, 3, 4, 64, 64), 30), ((1, 3, 4, 128, 64), 31), ((2, 9, 13, 64, 128), 333),
                                        ((3, 14, 14, 64, 64), 771)])
def test_row_counts_that_no_tile_divides(mp8, dims, prows):  # noqa: F811
    """Padded tensors with exactly the images' rows, or an odd number of them: nothing is written behind the last row, and no
    workspace is needed."""
    import torch
    B, H, W, Ci, Co = dims
    x, w, e = operands(dims)
    wd = gpu(w)
    n = B * (H + 2) * (W + 2)
    for op, a_h, name, cols in ((mp8.FWD, x, "fwd", Co), (mp8.BWD_DATA, e, "bwd_data", Ci)):
        ref, _ = oracle.conv3x3_ref(name, a_h, w, want_abs=False)
        xp = np.zeros((B, H + 2, W + 2, a_h.shape[3]), np.uint8)
        xp[:, 1:-1, 1:-1] = a_h
        a_dev = mp8.conv_buffer(prows, a_h.shape[3], W)
        a_dev[:n] = torch.from_numpy(xp.reshape(n, -1)).cuda()
        for kind in ("nearest", "statistics", "acc"):
            store = torch.full((prows + 256, cols), 0xAA, dtype=torch.uint8, device="cuda")
            acc = torch.full((prows + 256, cols), 7.5, dtype=torch.float32, device="cuda")
            st = mp8.new_stats() if kind != "nearest" else None
            mp8.conv3x3_fp8(op, *dims, a_dev, wd, out8=store[:prows], prows=prows, stats=st,
                            **({"acc": acc[:prows], "acc_mode": 1} if kind == "acc" else {}))
            out, beyond = host(store[:prows]), host(store[prows:])
            assert (beyond == 0xAA).all() and (host(acc[prows:]) == 7.5).all(), (name, kind)
            out_i, out_pad = interior(out, B, H, W)
            assert np.array_equal(out_i, oracle.round_ref_e5m2(ref)) and not out_pad.any(), (name, kind)
            if kind == "acc":
                assert np.array_equal(interior(host(acc[:prows]), B, H, W)[0].astype(np.float64), ref), name
