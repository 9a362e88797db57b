"""Statistics at the values that decide whether anything is counted: around the largest normal, the smallest subnormal and half of
it, zeros of both signs, FP32 subnormals, infinities, NaN -- one among values that count for nothing, and together."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu, host
from test_gpu_gemm import mp8  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

f = np.float32
up, down = lambda v: np.nextafter(f(v), f(np.inf)), lambda v: np.nextafter(f(v), f(0))
VALUES = [f(0), f(-0.0), f(2.0 ** -149), f(-2.0 ** -127), down(2.0 ** -17), f(2.0 ** -17), up(2.0 ** -17), down(2.0 ** -16), f(2.0 ** -16), up(2.0 ** -16), f(57344),
          up(57344), down(61440), f(61440), up(61440), f(65536), f(3e38), f(np.inf), f(-np.inf), f(np.nan), f(-np.nan)]


# flat kernels (workgroups of 256, of 1024, whole passes), transposing ones (element by element, guarded and whole tiles, teams)
@pytest.mark.parametrize("shape,transposed", [((33, 41), False), ((512, 1024), False), ((4096, 2048), False), ((100, 72), True), ((515, 517), True), ((1024, 1024), True),
                                              ((4096, 4096), True)])
@pytest.mark.parametrize("mode", [oracle.RNE, oracle.SR])
def test_q_node(mp8, shape, transposed, mode):  # noqa: F811
    import torch
    rng = np.random.default_rng(shape[0])
    n = shape[0] * shape[1]
    dst = torch.empty(shape, dtype=torch.uint8, device="cuda")
    dst_t = torch.empty(shape[::-1], dtype=torch.uint8, device="cuda") if transposed else None
    small = n <= 1 << 16
    cases = [[v] for v in VALUES] if small else []
    cases += [VALUES[:2], VALUES[2:10], VALUES[:10], VALUES[10:17], VALUES, []]  # zeros alone, flushed, both, overflowing, all, none
    for flags in (0, 1):
        for k, values in enumerate(cases):
            x = (rng.integers(1, 100, n) / 16).astype(np.float32)
            if values:
                at = rng.choice(n, 1 if len(values) == 1 else n // (2 if k % 2 else 500), replace=False)
                x[at] = np.resize(np.array(values, np.float32), at.size)
            want, st = oracle.Stats(), mp8.new_stats()
            codes, _ = oracle.quantize_e5m2(x.reshape(shape), mode=mode, flags=flags, seed=3, offset=k, stats=want)
            mp8.quantize_e5m2(gpu(x.reshape(shape)), dst, dst_t, round=mode, flags=flags, seed=3, offset=k, stats=st)
            assert mp8.read_stats(st) == want.as_tuple(), values
            assert np.array_equal(host(dst), codes) and (not transposed or np.array_equal(host(dst_t), codes.T))
    if not small:
        return
    halves = np.resize(np.array(VALUES, np.float32), n).astype(np.float16).reshape(shape)
    want, st = oracle.Stats(), mp8.new_stats()
    codes, _ = oracle.quantize_e5m2(halves, mode=mode, seed=3, offset=9, stats=want)
    mp8.quantize_e5m2(gpu(halves), dst, dst_t, round=mode, seed=3, offset=9, stats=st)
    assert mp8.read_stats(st) == want.as_tuple() and np.array_equal(host(dst), codes)


# few workgroups and more of them (where the running maximum is read before it is added to); sixteen columns at a time, ragged rows, a split contraction
@pytest.mark.parametrize("rows,cols,kc", [(64, 64, 128), (1024, 1024, 128), (65, 33, 128), (300, 200, 144), (100, 37, 130), (64, 64, 8192)])
@pytest.mark.parametrize("mode", [oracle.RNE, oracle.SR])
def test_gemm(mp8, rows, cols, kc, mode):  # noqa: F811
    """Rows of a that are zero but for one element, times a diagonal-like b: every output is one product, scaled to the values above."""
    import torch
    rng = np.random.default_rng(rows + cols)
    a, b = np.zeros((rows, kc), np.uint8), np.zeros((cols, kc), np.uint8)
    a[:, 0], b[:, 0] = rng.integers(0, 0x7C, rows), np.where(rng.random(cols) < 0.3, 0, rng.integers(0, 0x7C, cols))   # finite codes, zeros among them
    if kc % 128 == 0:
        a[::17, 0] = 0x7C
        a[5::29, 0] = 0x7E
    table = oracle.e5m2_decode_table().astype(np.float32)
    y = np.add(table[a[:, :1]] * table[b[:, :1]].T, f(0))     # exact in FP32; the sum starts at +0
    ws = torch.empty(max(16, mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc)), dtype=torch.uint8, device="cuda")
    for alpha in (1.0, 2.0 ** -8, 2.0 ** -20, 2.0 ** 10):
        want, st = oracle.Stats(), mp8.new_stats()
        codes, _ = oracle.quantize_e5m2(y, scale=alpha, mode=mode, seed=7, offset=1, stats=want)
        out = torch.empty((rows, cols), dtype=torch.uint8, device="cuda")
        for _ in range(2):                                     # into a cleared slot, then into one that holds the maximum
            mp8.gemm_fp8(mp8.FWD, rows, cols, kc, gpu(a), gpu(b), out8=out, alpha=alpha, round=mode, seed=7, offset=1, stats=st, workspace=ws)
        got = mp8.read_stats(st)
        assert np.array_equal(host(out), codes) and got == (want.as_tuple()[0], 2 * want.as_tuple()[1], 2 * want.as_tuple()[2])
