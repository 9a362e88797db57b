"""GPU parity of the master-weight update in the epilogue of the weight-gradient kernel that fetches operands
through registers (rows with no 16-byte alignment): the update and the gradient of the two calls, bit for bit."""
import numpy as np
import pytest

import test_gpu_wgrad_epilogue_update as epilogue_update

import test_gpu_gemm_ragged as ragged
from test_gpu_gemm_ragged import TN, mp8  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


# Tiles: 4, 32, 144 and 128, 512, 544, 1088; one stage, incomplete ones; rows and columns at the edge of a tile and of a pair of groups.  (With statistics
# of the gradient some of them take two launches; test_gpu_any_update_rule has calls without, and reads which call takes which.)
@pytest.mark.parametrize("dims", [(100, 72, 65), (300, 104, 1001), (129, 24, 2048), (257, 1000, 520), (1100, 1000, 500), (65, 1000, 2047),
                                  (1200, 2040, 1040), (130, 2040, 2113)])
@pytest.mark.parametrize("rule", ["sgd", "momentum", "adam"])
def test_update_in_the_epilogue(mp8, dims, rule):  # noqa: F811
    """Bit for bit the two calls, whatever is rounded how and with the step skipped (and refused without a gradient buffer)."""
    M, N, K = dims

    class Kept:
        """The library, with a gradient buffer where a call passes none: such calls are refused."""
        def __getattr__(self, name):
            f = getattr(mp8, name)
            if not name.startswith("wgrad_"):
                return f

            def call(*args, g8_out=None, **kw):
                import torch
                if g8_out is None:
                    with pytest.raises(mp8.Mp8Error):
                        f(*args, g8_out=None, **kw)
                    g8_out = torch.empty(N * K, dtype=torch.uint8, device="cuda")
                return f(*args, g8_out=g8_out, **kw)
            return call
    epilogue_update.test_update_in_the_epilogue_equals_two_calls(Kept(), dims, rule, True)


def test_update_in_the_epilogue_needs_no_workspace(mp8):  # noqa: F811
    import torch
    M, N, K = 300, 1000, 200
    rng = np.random.default_rng(3)
    a, b = (ragged.gpu(ragged.codes(int(rng.integers(1 << 30)), s)) for s in ((M, K), (M, N)))
    res = []
    for ws in (None, torch.empty(16, dtype=torch.uint8, device="cuda"), torch.empty(4 * N * K, dtype=torch.uint8, device="cuda")):
        w = torch.zeros(N * K, dtype=torch.float16, device="cuda")
        g = torch.empty(N * K, dtype=torch.uint8, device="cuda")
        mp8.wgrad_update_fp16_sr(M, N, K, a, b, w, 1e-3, 1.0, g8_out=g, alpha=2.0 ** -20, flags=TN, workspace=ws)
        torch.cuda.synchronize()
        res.append((ragged.host(w.view(torch.int16)), ragged.host(g)))
    assert all(np.array_equal(p, q) for r in res[1:] for p, q in zip(r, res[0]))
