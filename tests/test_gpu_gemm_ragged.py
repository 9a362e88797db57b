"""GPU parity of GEMMs whose contraction is not a whole number of 128-byte stages, or whose rows
have no 16-byte alignment: the half-precision forms of the direct-to-LDS kernels, the kernel that fetches
operands through registers, its split contractions with and without a workspace, and the fallback for tiny shapes."""
import numpy as np
import pytest

import oracle
from paper_1905_12334_amd import workloads
from gpu_util import assert_as_precise_as_fp32, check_outputs, gpu, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mp8():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_1905_12334_amd as m
    m.lib()
    return m


ROW, BTN, TN = 0, 4, 6      # operand layouts (flags)

# rows, cols, contraction, layout
CASES = [
    # whole 16-byte chunks: one to eight of them in the incomplete stage
    (64, 64, 16, TN), (64, 64, 16, ROW), (100, 48, 112, BTN), (256, 256, 144, ROW), (256, 256, 144, BTN),
    (512, 384, 127, TN), (512, 384, 129, TN), (1024, 1024, 1, TN), (1536, 2048, 208, ROW), (2048, 1536, 240, BTN),
    (512, 512, 2049, TN), (512, 512, 2064, ROW), (128, 1024, 2096, BTN), (128, 512, 2160, ROW),
    (320, 128, 6007, TN), (64, 64, 9001, TN), (1536, 1408, 8200, TN), (1536, 1408, 8208, ROW), (1536, 1408, 8208, BTN),
    (3840, 4096, 1040, ROW), (3840, 4096, 1072, BTN), (3840, 4096, 1025, TN),
    # large outputs
    (1536, 2048, 2065, TN), (2032, 1936, 3100, TN), (2048, 2048, 3088, ROW), (2000, 1552, 2096, BTN), (2288, 1024, 4100, TN),
    (2304, 2032, 8208, BTN),
    # odd everything
    (17, 33, 16, ROW), (17, 33, 17, BTN), (17, 33, 31, TN), (16, 16, 100, TN), (63, 65, 127, ROW), (65, 63, 128, BTN),
    (129, 1000, 128, BTN), (256, 1000, 2048, BTN), (1000, 2048, 255, TN), (999, 1001, 333, ROW), (81, 79, 1000, TN),
    (40, 72, 5000, TN), (40, 72, 5000, ROW), (41, 71, 5001, BTN),
    # too short or too narrow for that kernel
    (5, 7, 15, ROW), (15, 40, 300, TN), (40, 15, 300, BTN), (1, 1, 1, TN),
]


def codes(seed, shape):
    """Uniform over the finite codes: every exponent, subnormals, zeros, both signs."""
    return workloads.random_e5m2_codes(seed, shape, finite_only=True)


def scale_for(kc):
    return float(2.0 ** -23 * (128.0 / kc) ** 0.5)      # most outputs inside the 8-bit range


def stored(x, km, pad=0, shift=0, fill=0x7E):
    """x in memory as its layout has it: contraction-major or not, `pad` NaN codes behind every row, the first
    byte `shift` bytes behind an aligned address.  Returns the tensor and its leading dimension."""
    x = np.ascontiguousarray(x.T) if km else x
    buf = np.full((x.shape[0], x.shape[1] + pad), fill, np.uint8)
    buf[:, : x.shape[1]] = x
    flat = gpu(np.concatenate([np.full(shift, fill, np.uint8), buf.reshape(-1)]))
    return flat[shift:], x.shape[1] + pad


@pytest.mark.parametrize("rows,cols,kc,layout", CASES)
def test_ragged_gemm(mp8, rows, cols, kc, layout):
    """FP32 accumulator as precise as FP32 multiply-adds on operands of the full range, 8-bit codes in both
    orientations, statistics, RNE and SR; the same bits with a workspace, a larger one and none; nothing
    read from the padding of the leading dimension (NaN codes there) or written out of bounds."""
    import torch
    rng = np.random.default_rng(rows * 7919 + cols * 31 + kc + layout)
    big = rows * cols * kc > 3e8
    a, b = codes(int(rng.integers(1 << 30)), (rows, kc)), codes(int(rng.integers(1 << 30)), (cols, kc))
    # aligned where the direct-to-LDS kernels can take it, any base address elsewhere
    direct = kc % 128 != 0 and (layout == TN or kc % 16 == 0) and (layout != TN or rows % 16 == 0) and (layout == ROW or cols % 16 == 0)
    pad, shift = 16 * int(rng.integers(0, 2)), 0 if direct else int(rng.integers(1, 16))
    ag, lda = stored(a, layout == TN, pad, shift)
    bg, ldb = stored(b, layout != ROW, pad)
    sub = rng.choice(rows, 24, replace=False) if big else np.arange(rows)     # rows that are checked
    ref, absref = oracle.gemm_ref(a[sub], b)
    need = mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc)
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    n, alpha = rows * cols, scale_for(kc)
    first = None
    for mode, workspace in ((oracle.RNE, ws), (oracle.SR, None), (oracle.SR, ws)):
        acc = torch.full((n + 16,), 7.0, dtype=torch.float32, device="cuda")
        o1, o1t, o2 = (torch.full((n + 64,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(3))
        s1, s2 = mp8.new_stats(), mp8.new_stats()
        kw = dict(round=mode, flags=layout, seed=11, offset=3, workspace=workspace, lda=lda, ldb=ldb, alpha=alpha)
        mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, out8=o1[:n], out8_t=o1t[:n], acc=acc[:n], acc_mode=1, stats=s1, **kw)
        mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, out8=o2[:n], stats=s2, **kw)
        torch.cuda.synchronize()
        assert bool((o1[n:] == 0xAA).all()) and bool((o1t[n:] == 0xAA).all()) and bool((o2[n:] == 0xAA).all())
        assert bool((acc[n:] == 7.0).all())
        full, out = host(acc[:n]).reshape(rows, cols), host(o1[:n]).reshape(rows, cols)
        if first is None:
            first = full
            assert_as_precise_as_fp32(full[sub], a[sub], b, ref, f"ragged {rows} x {cols} layout {layout}")
        assert np.array_equal(full, first), "the accumulator depends on the workspace"
        want, _ = oracle.quantize_e5m2(full, scale=alpha, mode=mode, seed=11, offset=3)
        assert np.array_equal(out, want)
        assert np.array_equal(host(o1t[:n]).reshape(cols, rows), out.T)
        check_outputs(full[sub], out[sub], ref, absref, kc, alpha=alpha, mode=mode, seed=11, offset=3,
                      first_index=sub.astype(np.int64) * cols if big else None, cols=cols)
        assert np.array_equal(host(o2[:n]).reshape(rows, cols), out)
        st = oracle.Stats()
        oracle.quantize_e5m2(full, scale=alpha, mode=mode, seed=11, offset=3, stats=st)
        assert mp8.read_stats(s1) == st.as_tuple() == mp8.read_stats(s2)


# operands through registers: unsplit, four slices; rows of a multiple of sixteen columns and others
SPECIAL = [(r, c, k, layout, False) for r, c, k in ((40, 72, 300), (100, 80, 301), (100, 80, 4100), (41, 71, 5001)) for layout in (ROW, BTN, TN)]
# direct to LDS: 64x64, wave-split and 128x128 tiles; rows of any number of columns where b is row-major
SPECIAL += [(r, c, k, layout, True) for r, c, k in ((112, 80, 304), (208, 1040, 2064), (2064, 1936, 272)) for layout in (ROW, BTN, TN)]
SPECIAL += [(99, 71, 304, ROW, True), (207, 1001, 2064, ROW, True), (2061, 1931, 272, ROW, True), (112, 80, 301, TN, True),
            (208, 1040, 2065, TN, True), (2064, 1936, 257, TN, True)]


@pytest.mark.parametrize("rows,cols,kc,layout,aligned", SPECIAL)
def test_ragged_gemm_special_codes_and_accumulation_across_calls(mp8, rows, cols, kc, layout, aligned):
    """Inf and NaN codes reach exactly the outputs they belong to, also from the last, partial chunk of a
    row; acc_mode 2 adds the accumulator of a call to what is there, once; a workspace changes no bit."""
    import torch
    rng = np.random.default_rng(rows + cols + kc)
    a, b = codes(int(rng.integers(1 << 30)), (rows, kc)), codes(int(rng.integers(1 << 30)), (cols, kc))
    plain, _ = oracle.gemm_ref(a, b)
    a[3, kc - 1], a[7, 0], a[rows - 1, kc // 2], b[5, kc - 2], b[cols - 1, 1] = 0x7C, 0xFC, 0x7D, 0x7F, 0x7C
    ref, _ = oracle.gemm_ref(a, b)
    assert np.isnan(ref).any() and np.isinf(ref).any() and np.isfinite(ref).any()
    ag, lda = stored(a, layout == TN, 0, 0 if aligned else 5)
    bg, ldb = stored(b, layout != ROW, 0 if aligned else 1)
    alpha = scale_for(kc)
    a0 = (rng.standard_normal((rows, cols)) * np.std(plain)).astype(np.float32)
    ws = torch.empty(max(16, mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc)), dtype=torch.uint8, device="cuda")
    results = []
    for workspace in (None, ws):
        one = torch.empty((rows, cols), dtype=torch.float32, device="cuda")
        two, o8 = gpu(a0), torch.zeros((rows, cols), dtype=torch.uint8, device="cuda")
        kw = dict(flags=layout, workspace=workspace, lda=lda, ldb=ldb, alpha=alpha)
        mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, acc=one, acc_mode=1, **kw)
        mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, acc=two, acc_mode=2, out8=o8, **kw)
        torch.cuda.synchronize()
        got, sums = host(one), host(two)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
        assert np.array_equal(np.sign(got[np.isinf(got)]), np.sign(ref[np.isinf(ref)]))
        assert np.array_equal(sums, a0 + got, equal_nan=True)
        assert np.array_equal(host(o8), oracle.quantize_e5m2(sums, scale=alpha)[0])
        results.append((got.view(np.uint32), sums.view(np.uint32)))
    fin = np.isfinite(ref)
    assert all(np.array_equal(x[fin], y[fin]) for x, y in zip(*results))


# Row-major operands of an odd leading dimension with a split contraction and whole stages; ragged token counts;
# row lengths that are not multiples of sixteen; 128x128 tiles.  `bare`: the rules that need neither a gradient
# buffer nor a workspace (the update in the GEMM's own epilogue); `scratch`: the queried workspace stands in for the
# buffer.
@pytest.mark.parametrize("layout,dims,odd,bare,scratch", [
    (ROW, (5120, 256, 256), 1, "", True), (TN, (1000, 128, 64), 0, "sgd momentum", True), (TN, (5001, 64, 192), 0, "sgd momentum", True),
    (ROW, (4000, 92, 77), 0, "", True), (BTN, (2049, 112, 80), 0, "", False), (TN, (300, 1008, 2048), 0, "sgd momentum adam", True),
    (ROW, (2064, 1024, 1008), 0, "sgd momentum adam", True), (TN, (300, 2064, 4096), 0, "", True)])
@pytest.mark.parametrize("rule", ["sgd", "momentum", "adam"])
def test_ragged_weight_gradient_with_update(mp8, layout, dims, odd, bare, scratch, rule):
    """Weight gradient and update in one call equal the two separate calls bit for bit, whatever workspace
    either of them is given, and with or without a buffer for the gradient."""
    import torch
    M, N, K = dims
    a, b = codes(1, (K, M)), codes(2, (N, M))
    (ag, lda), (bg, ldb) = stored(a, layout == TN, odd), stored(b, layout != ROW, odd)
    n = K * N
    rng = np.random.default_rng(3)
    w = (rng.standard_normal(n) * 0.05).astype(np.float16)
    m0, v0 = (rng.standard_normal(n) * 1e-3).astype(np.float32), (rng.random(n) * 1e-6).astype(np.float32)
    need = mp8.gemm_fp8_workspace_bytes(mp8.WGRAD, M, N, K)
    exact, large = (torch.empty(k, dtype=torch.uint8, device="cuda") for k in (max(need, 16), 8 * need + 4 * n))
    alpha, inv = scale_for(M), 2.0 ** -6
    grad = dict(flags=layout, lda=lda, ldb=ldb, alpha=alpha)

    def step(fused, workspace, keep=True):
        wt, mt, vt = gpu(w), gpu(m0), gpu(v0)
        g, w8 = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
        if fused:
            kw = dict(g8_out=g if keep else None, g_round=mp8.SR, g_seed=5, g_offset=1, w_round=mp8.SR, w_seed=6, w_offset=2,
                      w8_out=w8, workspace=workspace, **grad)
            if rule == "sgd":
                mp8.wgrad_update_fp16_sr(M, N, K, ag, bg, wt, 0.01, inv, **kw)
            elif rule == "momentum":
                mp8.wgrad_momentum_fp16_sr(M, N, K, ag, bg, wt, mt, 0.01, inv, 0.9, weight_decay=1e-2, **kw)
            else:
                mp8.wgrad_adam_fp16_sr(M, N, K, ag, bg, wt, mt, vt, 0.01, inv, 7, weight_decay=1e-2, **kw)
        else:
            mp8.gemm_fp8(mp8.WGRAD, M, N, K, ag, bg, out8=g, round=mp8.SR, seed=5, offset=1, workspace=workspace, **grad)
            kw = dict(round=mp8.SR, seed=6, offset=2, w8_out=w8)
            if rule == "sgd":
                mp8.sgd_update_fp16_sr(wt, g, 0.01, inv, **kw)
            elif rule == "momentum":
                mp8.sgd_momentum_fp16_sr(wt, mt, g, 0.01, inv, 0.9, 1e-2, **kw)
            else:
                mp8.adam_fp16_sr(wt, mt, vt, g, 0.01, inv, 7, weight_decay=1e-2, **kw)
        torch.cuda.synchronize()
        return [host(t) for t in (wt.view(torch.int16), mt.view(torch.int32), vt.view(torch.int32), w8)] + ([host(g)] if keep else [])

    want = step(False, exact)
    for fused in (False, True):
        for workspace in (None, exact, large):
            assert all(np.array_equal(x, y) for x, y in zip(want, step(fused, workspace))), (fused, workspace is None)
    for workspace, accepted in ((None, rule in bare.split()), (exact, scratch), (large, scratch)):
        if accepted:
            assert all(np.array_equal(x, y) for x, y in zip(want, step(True, workspace, keep=False)))
        else:
            with pytest.raises(mp8.Mp8Error):
                step(True, workspace, keep=False)
    acc = torch.empty((K, N), dtype=torch.float32, device="cuda")
    mp8.gemm_fp8(mp8.WGRAD, M, N, K, ag, bg, acc=acc, acc_mode=1, workspace=exact, **grad)
    ref, absref = oracle.gemm_ref(a, b)
    assert np.all(np.abs(host(acc) - ref) <= 1e-5 * np.sqrt(M) * absref)
    assert_as_precise_as_fp32(host(acc)[:24], a[:24], b, ref[:24], f"weight gradient {dims} layout {layout}")
    assert np.array_equal(want[4].reshape(K, N), oracle.quantize_e5m2(host(acc), scale=alpha, mode=oracle.SR, seed=5, offset=1)[0])
    if rule == "sgd":
        ow, ow8 = oracle.sgd_update_fp16(w.view(np.uint16), want[4], 0.01, inv, mode=oracle.SR, seed=6, offset=2, want_w8=True)
        assert np.array_equal(want[0].view(np.uint16), ow) and np.array_equal(want[3], ow8)
