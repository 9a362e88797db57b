"""ADAM's bias corrections: a product with the double-precision reciprocal, rounded once, is the FP32 quotient."""
import numpy as np
import pytest

import oracle

BETAS = [(0.0, 0.0), (0.5, 0.75), (0.9, 0.999), (0.95, 0.9999999), (0.99999994, 0.99999994)]


@pytest.mark.parametrize("kind", ["any", "subnormal"])
@pytest.mark.parametrize("correction", ["any", "of the betas"])
def test_reciprocal_in_double_is_the_quotient(kind, correction):
    rng, n = np.random.default_rng(5), 1 << 20
    m = rng.integers(0, 1 << (32 if kind == "any" else 24), n, dtype=np.uint32).view(np.float32)
    if correction == "any":
        c = (rng.integers(1 << 23, (1 << 24) + 1, n) * np.exp2(-24.0 - rng.integers(0, 24, n))).astype(np.float32)
    else:
        beta = rng.choice(np.float32([b for pair in BETAS for b in pair]), n).astype(np.float64)
        c = (1.0 - beta ** rng.integers(1, 5000, n)).astype(np.float32)
    with np.errstate(all="ignore"):
        want, got = m / c, (m.astype(np.float64) * (1.0 / c.astype(np.float64))).astype(np.float32)
    ok = ~np.isnan(want)
    assert np.array_equal(np.isnan(got), ~ok) and np.array_equal(got[ok].view(np.uint32), want[ok].view(np.uint32))


@pytest.mark.gpu
@pytest.mark.parametrize("betas", BETAS)
@pytest.mark.parametrize("step", [1, 2, 1000, 2 ** 31 - 1])
def test_update_matches_oracle(betas, step):
    """Every class of moment, weights that show the quotients to their last bits (from zero, in several scales)."""
    import paper_1905_12334_amd as mp8
    from gpu_util import gpu, host
    import torch
    rng, n = np.random.default_rng(step % 97), 1 << 15
    w16, g8 = np.zeros(n, np.uint16), (rng.integers(0, 256, n) & 0x83).astype(np.uint8) | np.uint8(0x38)
    m0 = rng.integers(0, 1 << 32, n, dtype=np.uint32).view(np.float32)
    v0 = np.abs(rng.integers(0, 1 << 32, n, dtype=np.uint32).view(np.float32))
    m0[::2], v0[::2] = rng.standard_normal(n // 2), rng.random(n // 2)
    kw = dict(beta1=betas[0], beta2=betas[1], eps=1e-8)
    w, m, v = gpu(w16.view(np.int16)), gpu(m0), gpu(v0)
    mp8.adam_fp16_sr(w, m, v, gpu(g8), 0.125, 2.0 ** -8, step, round=mp8.RNE, **kw)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        ow, om, ov, _ = oracle.adam_fp16(w16, m0, v0, g8, 0.125, 2.0 ** -8, step, mode=oracle.RNE, **kw)
    for got, want in ((host(m), om), (host(v), ov), (host(w).view(np.float16), ow.view(np.float16))):
        ok = ~np.isnan(want)
        assert np.array_equal(np.isnan(got), ~ok) and np.array_equal(got[ok], want[ok])
