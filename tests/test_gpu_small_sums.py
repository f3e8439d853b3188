"""Cycle kernel of small systems of up to 64 blocks: sums of every block's values.

A wave takes 64 / SLOTS blocks' values at once (SLOTS: 4, 8 or 16 by the
restart), up to eight such loads (fp64: four) together, fewer for a few blocks
in fp32.  Block counts at the edges of a load and of a pass, against the phases
launched one by one (the same bits) and the oracle.  Times: an fp64 iteration,
bound by the same exchanges as an fp32 one with values twice as long."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B

from gpu_common import say
from test_gpu_small_cycle import KINDS, banded, both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("blocks", [1, 4, 5, 8, 9, 16, 17, 32, 33, 63])
@pytest.mark.parametrize("inner,basis,m", [(*k, m) for k in KINDS for m in (28, 56, 112)])
def test_block_counts(inner, basis, m, blocks):
    say("small sums", inner, basis, m, blocks)
    n = 128 * blocks  # 128 rows a block
    both(banded(n, (-100, -1, 0, 1, 100), m), m, inner, basis, m + 3, oracle=m == 28)


def iteration_us(M, b, inner, m, iters):
    ws, x = B.Workspace(), torch.zeros_like(b)
    p = B.make_params(restart=m, inner=inner, basis=inner, rtol=1e-30, max_iters=iters, check_mode=0)
    best = 1e9
    for _ in range(9):
        x.zero_()
        torch.cuda.synchronize()
        t = time.perf_counter()
        _, info, _ = B.gmresir_solve(M, b, x, p, ws=ws)
        torch.cuda.synchronize()
        best = min(best, 1e6 * (time.perf_counter() - t))
        assert info["iters"] == iters
    return best / iters


@pytest.mark.parametrize("n,m", [(4900, 112), (15625, 56), (15625, 112)])
def test_fp64_time(n, m):
    """1.4 to 1.45 times an fp32 iteration.  Where each load of a sum was waited for
    before the next went out, 1.77 times it in the last case."""
    say("small sums, times", n, m)
    A = banded(n, (-300, -1, 0, 1, 300), m)
    A.vals[A.colidx == np.repeat(np.arange(n), np.diff(A.rowptr))] = 0.5  # far from converged in these steps
    M = B.Matrix.from_csr(A)
    b = torch.ones(n, dtype=torch.float64, device="cuda")
    t32, t64 = (iteration_us(M, b, inner, m, 4 * m) for inner in ("fp32", "fp64"))
    print(f"{t32:.1f} and {t64:.1f} us")
    assert t64 <= 1.55 * t32
