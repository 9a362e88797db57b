"""GPU parity of the Q node's launch forms where they change: how groups are dealt to the workgroups with
statistics, one group per thread for small tensors, and transposed copies of row and column counts that are not
multiples of four (both tile sizes)."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mp8():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_1905_12334_amd as m
    m.lib()
    return m


def check(mp8, x, rnd, want_t, with_stats, scale=1.0):
    import torch
    rows, cols = x.shape
    n = rows * cols
    d = torch.full((n + 64,), 0xAA, dtype=torch.uint8, device="cuda")
    t = torch.full((n + 64,), 0xAA, dtype=torch.uint8, device="cuda")
    st = mp8.new_stats() if with_stats else None
    mp8.quantize_e5m2(gpu(x), d[:n], t[:n] if want_t else None, scale=scale, round=rnd, seed=9, offset=4, stats=st)
    torch.cuda.synchronize()
    ost = oracle.Stats()
    want, _ = oracle.quantize_e5m2(x.astype(np.float32), scale=scale, mode=rnd, seed=9, offset=4, stats=ost)
    assert np.array_equal(host(d[:n]).reshape(rows, cols), want)
    assert bool((d[n:] == 0xAA).all()) and bool((t[n if want_t else 0:] == 0xAA).all())
    if want_t:
        assert np.array_equal(host(t[:n]).reshape(cols, rows), want.T)
    if with_stats:
        assert mp8.read_stats(st) == ost.as_tuple()


def data(seed, shape, half):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(shape) * np.exp2(rng.integers(-20, 8, shape))
    x[rng.random(shape) < 0.01] = 0
    x.reshape(-1)[rng.integers(0, x.size, 3)] = (np.inf, -np.inf, np.nan)
    return x.astype(np.float16 if half else np.float32)


# with statistics: runs of up to 512 groups for 256 threads, longer ones for 1024 threads, then whole rounds of 2^20
# groups over all workgroups and a rest (none, one group, several per thread)
@pytest.mark.parametrize("n", [4, 252, 4 * 256 * 256 - 4, 4 * 256 * 256 + 4, 4 * 256 * 512 + 260, 4 * 256 * 1024 + 1027,
                               4 * 256 * 3 * 1024 - 13, 4 * 256 * 5 * 1024 + 3, 4 * 256 * 9 * 1024 + 77,
                               4 * 32768, 4 * 32768 + 5, 4 * 2 ** 19, 4 * 2 ** 19 + 4, 4 * 2 ** 20, 4 * 2 ** 20 + 6, 4 * (2 ** 21 + 65000) + 1])
@pytest.mark.parametrize("rnd", [oracle.RNE, oracle.SR])
@pytest.mark.parametrize("with_stats", [False, True])
def test_flat_run_lengths(mp8, n, rnd, with_stats):
    check(mp8, data(n, (1, n), False), rnd, False, with_stats)


# to nearest without statistics the stores change at 7 * 2^19 and behind 13 * 2^19 elements
@pytest.mark.parametrize("n", [7 * 2 ** 19, 7 * 2 ** 19 + 1, 7 * 2 ** 19 + 1027, 13 * 2 ** 19, 13 * 2 ** 19 + 1])
@pytest.mark.parametrize("half", [False, True])
def test_flat_stores(mp8, n, half):
    check(mp8, data(n, (1, n), half), oracle.RNE, False, False)


# the guarded end of a run: one pass or two of 256 threads' groups, and of 1024 with statistics (runs of 64 r groups in 256 workgroups)
@pytest.mark.parametrize("n,with_stats", [(4 * (2 ** 18 + 256 + d), False) for d in (-1, 0, 1, 255, 256, 257, 511)] +
                         [(4 * 256 * 64 * r - 8, True) for r in (5, 7, 8, 9, 15, 16, 17, 31, 33, 47, 48, 49)])
def test_stochastic_ends_of_runs(mp8, n, with_stats):
    check(mp8, data(n, (1, n), False), oracle.SR, False, with_stats)


@pytest.mark.parametrize("shape", [(1, 1), (2, 3), (63, 65), (66, 127), (600, 450), (130, 2061), (517, 523), (2049, 2051), (2050, 2052), (2052, 2050)])
@pytest.mark.parametrize("rnd", [oracle.RNE, oracle.SR])
@pytest.mark.parametrize("half,with_stats", [(False, True), (True, False)])
def test_ragged_transposed_copies(mp8, shape, rnd, half, with_stats):
    check(mp8, data(shape[0], shape, half), rnd, True, with_stats)


@pytest.mark.parametrize("shape", [(128, 128), (1024, 2048), (2064, 2052), (2064, 2056), (8208, 8196)])
def test_transposed_copies_with_statistics_and_shared_random_blocks(mp8, shape):
    check(mp8, data(shape[1], shape, False), oracle.SR, True, True)


# with statistics: element by element in a capped grid, tiles of 64 up to 64 tiles of 128 (127 when stochastic)
@pytest.mark.parametrize("shape", [(256, 256), (256, 260), (256, 512), (255, 513), (512, 511), (1024, 1024), (1024, 1152), (1020, 1156), (1021, 1155),
                                   (1024, 1920), (1024, 2048)])
@pytest.mark.parametrize("rnd", [oracle.RNE, oracle.SR])
def test_transposed_copies_with_statistics_at_the_changes_of_form(mp8, shape, rnd):
    check(mp8, data(shape[1], shape, False), rnd, True, True)


# element by element, one tile of 64 across, tiles of 128
@pytest.mark.parametrize("shape", [(300001, 1), (20001, 15), (20000, 12), (20000, 16), (10001, 31), (10001, 32), (20000, 64), (6001, 65),
                                   (1, 300001), (15, 20001), (12, 20000), (16, 20000), (17, 20001), (63, 9001), (64, 9000), (66, 9002)])
@pytest.mark.parametrize("rnd", [oracle.RNE, oracle.SR])
@pytest.mark.parametrize("with_stats", [False, True])
def test_narrow_transposed_copies(mp8, shape, rnd, with_stats):
    check(mp8, data(shape[0] + shape[1], shape, True), rnd, True, with_stats)


@pytest.mark.parametrize("shape", [(2 ** 29 + 5, 1), (2 ** 27 + 64, 16)])
def test_narrow_transposed_copies_of_more_tiles_than_a_launch_takes(mp8, shape):
    """Tiles of 128 rows and 1024 threads each would be 2^32 threads and more; one tile of 64 x 64 more than the
    grid has workgroups."""
    import torch
    x = torch.arange(shape[0] * shape[1], device="cuda").remainder_(2039).to(torch.float16).view(shape)
    d, t, want = (torch.empty(x.numel(), dtype=torch.uint8, device="cuda") for _ in range(3))
    mp8.quantize_e5m2(x, d, t)
    mp8.quantize_e5m2(x, want)
    assert torch.equal(d, want)
    step = 2 ** 24
    for i in range(0, shape[0], step):
        part = want.view(shape)[i:i + step]
        assert torch.equal(t.view(shape[1], shape[0])[:, i:i + step], part.t())
