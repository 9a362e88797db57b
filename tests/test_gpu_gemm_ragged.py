"""GPU parity of GEMMs whose contraction is not a whole number of 128-byte stages, or whose rows
have no 16-byte alignment: the incomplete stage of the direct-to-LDS kernels, and the kernel that
fetches operands through registers."""
import numpy as np
import pytest

import oracle
from paper_1905_12334_amd import workloads
from gpu_util import gpu, host, check_outputs

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
    # whole 16-byte chunks: one to eight of them in the incomplete stage, every kernel family
    (64, 64, 16, TN), (64, 64, 16, ROW), (100, 48, 112, BTN), (256, 256, 144, ROW), (256, 256, 144, BTN),
    (512, 384, 127, TN), (512, 384, 129, TN), (1024, 1024, 1, TN), (1536, 2048, 208, ROW), (2048, 1536, 240, BTN),
    (512, 512, 2049, TN), (512, 512, 2064, ROW), (128, 1024, 2096, BTN), (128, 512, 2160, ROW),
    (320, 128, 6007, TN), (64, 64, 9001, TN), (1536, 1408, 8200, TN), (1536, 1408, 8208, ROW), (1536, 1408, 8208, BTN),
    (3840, 4096, 1040, ROW), (3840, 4096, 1072, BTN), (3840, 4096, 1025, TN),
    # one 128x128 tile per CU on the four-stage ring, and two of the two-stage one
    (1536, 2048, 2065, TN), (2032, 1936, 3100, TN), (2048, 2048, 3088, ROW), (2000, 1552, 2096, BTN), (2288, 1024, 4100, TN),
    (2304, 2032, 8208, BTN),
    # odd everything
    (17, 33, 16, ROW), (17, 33, 17, BTN), (17, 33, 31, TN), (16, 16, 100, TN), (63, 65, 127, ROW), (65, 63, 128, BTN),
    (129, 1000, 128, BTN), (256, 1000, 2048, BTN), (1000, 2048, 255, TN), (999, 1001, 333, ROW), (81, 79, 1000, TN),
    (40, 72, 5000, TN), (40, 72, 5000, ROW), (41, 71, 5001, BTN),
    # too short or too narrow for that kernel
    (5, 7, 15, ROW), (15, 40, 300, TN), (40, 15, 300, BTN), (1, 1, 1, TN),
]


@pytest.mark.parametrize("rows,cols,kc,layout", CASES)
def test_ragged_gemm(mp8, rows, cols, kc, layout):
    """FP32 accumulator, 8-bit codes in both orientations, statistics, RNE and SR; with and without a
    workspace (the latter is what these shapes always accepted); nothing read from the padding of the
    leading dimension (NaN codes there) or written out of bounds."""
    import torch
    rng = np.random.default_rng(rows * 7919 + cols * 31 + kc + layout)
    big = rows * cols * kc > 3e8
    a = (workloads.random_e5m2_codes(int(rng.integers(1 << 30)), (rows, kc)) & 0x83) | 0x38
    b = (workloads.random_e5m2_codes(int(rng.integers(1 << 30)), (cols, kc)) & 0x83) | 0x38
    pad = 16 * int(rng.integers(0, 2))

    def stored(x, km):
        x = np.ascontiguousarray(x.T) if km else x
        buf = np.full((x.shape[0], x.shape[1] + pad), 0x7E, np.uint8)
        buf[:, : x.shape[1]] = x
        return gpu(buf), x.shape[1] + pad

    ag, lda = stored(a, layout == TN)
    bg, ldb = stored(b, layout != ROW)
    sub = rng.choice(rows, 24, replace=False) if big else np.arange(rows)     # rows that are checked
    ref, absref = oracle.gemm_ref(a[sub], b)
    ws = torch.empty(max(mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc), 4 * rows * cols), dtype=torch.uint8, device="cuda")
    n = rows * cols
    for mode, workspace in ((oracle.RNE, ws), (oracle.SR, None), (oracle.SR, ws)):
        if workspace is None and kc % 128 == 0:
            continue                                     # (whole stages may need one)
        acc = torch.full((n + 16,), 7.0, dtype=torch.float32, device="cuda")
        o1, o1t, o2 = (torch.full((n + 64,), 0xAA, dtype=torch.uint8, device="cuda") for _ in range(3))
        s1, s2 = mp8.new_stats(), mp8.new_stats()
        kw = dict(round=mode, flags=layout, seed=11, offset=3, workspace=workspace, lda=lda, ldb=ldb, alpha=0.37)
        mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, out8=o1[:n], out8_t=o1t[:n], acc=acc[:n], acc_mode=1, stats=s1, **kw)
        mp8.gemm_fp8(mp8.FWD, rows, cols, kc, ag, bg, out8=o2[:n], stats=s2, **kw)
        torch.cuda.synchronize()
        assert bool((o1[n:] == 0xAA).all()) and bool((o1t[n:] == 0xAA).all()) and bool((o2[n:] == 0xAA).all())
        assert bool((acc[n:] == 7.0).all())
        full, out = host(acc[:n]).reshape(rows, cols), host(o1[:n]).reshape(rows, cols)
        want, _ = oracle.quantize_e5m2(full, scale=0.37, mode=mode, seed=11, offset=3)
        assert np.array_equal(out, want)
        assert np.array_equal(host(o1t[:n]).reshape(cols, rows), out.T)
        check_outputs(full[sub], out[sub], ref, absref, kc, alpha=0.37, mode=mode, seed=11, offset=3,
                      first_index=sub.astype(np.int64) * cols if big else None, cols=cols)
        # without FP32 and transposed outputs another kernel may do it, in another order of additions
        other = host(o2[:n]).reshape(rows, cols)
        assert (other != out).mean() <= 2e-3
        st = oracle.Stats()
        oracle.quantize_e5m2(full, scale=0.37, mode=mode, seed=11, offset=3, stats=st)
        assert mp8.read_stats(s1) == st.as_tuple()


@pytest.mark.parametrize("layout,dims", [(TN, (1000, 128, 64)), (TN, (5001, 64, 192)), (ROW, (4000, 92, 77))])
def test_ragged_weight_gradient_with_update(mp8, layout, dims):
    """Weight gradient and update in one call on a ragged token count equal the two separate calls."""
    import torch
    M, N, K = dims
    a = (workloads.random_e5m2_codes(1, (M, K)) & 0x83) | 0x38
    b = (workloads.random_e5m2_codes(2, (M, N)) & 0x83) | 0x38
    ag, bg = (gpu(x if layout == TN else np.ascontiguousarray(x.T)) for x in (a, b))
    w = (np.random.default_rng(3).standard_normal(K * N) * 0.05).astype(np.float16)
    ws = torch.empty(max(mp8.gemm_fp8_workspace_bytes(mp8.WGRAD, M, N, K), 16), dtype=torch.uint8, device="cuda")
    for workspace in (ws, None):
        g, w8, w1 = torch.zeros(K * N, dtype=torch.uint8, device="cuda"), torch.zeros(K * N, dtype=torch.uint8, device="cuda"), gpu(w)
        mp8.wgrad_update_fp16_sr(M, N, K, ag, bg, w1, 0.01, 2.0 ** -6, g8_out=g, g_round=mp8.SR, flags=layout, g_seed=5,
                                 g_offset=1, w_round=mp8.SR, w_seed=6, w_offset=2, w8_out=w8, workspace=workspace)
        torch.cuda.synchronize()
        acc = torch.empty((K, N), dtype=torch.float32, device="cuda")
        mp8.gemm_fp8(mp8.WGRAD, M, N, K, ag, bg, acc=acc, acc_mode=1, flags=layout, workspace=ws)
        ref, absref = oracle.gemm_ref(np.ascontiguousarray(a.T), np.ascontiguousarray(b.T))
        assert np.all(np.abs(host(acc) - ref) <= 1e-5 * np.sqrt(M) * absref)
        want8, _ = oracle.quantize_e5m2(host(acc), mode=oracle.SR, seed=5, offset=1)
        assert (host(g).reshape(K, N) != want8).mean() <= 2e-3
        ow, ow8 = oracle.sgd_update_fp16(w.view(np.uint16), host(g), 0.01, 2.0 ** -6, mode=oracle.SR, seed=6, offset=2, want_w8=True)
        assert np.array_equal(host(w1).view(np.uint16), ow) and np.array_equal(host(w8), ow8)
