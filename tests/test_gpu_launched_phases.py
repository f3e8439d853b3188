"""Small systems whose cycles are launched kernel by kernel (gmresir_solve_noalloc,
profile = 1): not slower than the general kernels on the same cycles.

restart = 113 is past the small kernels' limit; with inner_cap = 50 it makes the
general kernels run cycles of 50 steps.  The wider bound covers the clock's
spread; sums taken group by group in every phase were at twice."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def best(M, b, **kw):
    p = B.make_params(rtol=1e-14, max_iters=200, check_mode=0, **kw)
    x = torch.zeros_like(b)
    t = []
    for _ in range(8):
        x.zero_()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, d, _ = B.gmresir_solve_noalloc(M, b, x, p)
        torch.cuda.synchronize()
        t.append((time.perf_counter() - t0) / d["iters"])
    return min(t)


@pytest.mark.parametrize("inner,basis", [("fp32", "fp32"), ("fp64", "fp64"), ("fp32", "bf16")])
@pytest.mark.parametrize("side", [64, 150, 250])
def test_not_slower_than_general(side, inner, basis):
    say("phases against general", side, inner, basis)
    A = P.convdiff2d_system(1, side).A
    M = B.Matrix.from_csr(A)
    b = torch.from_numpy(A.scipy() @ np.ones(A.n)).cuda()
    for ortho in (0, 1) if basis != "bf16" else (0,):
        phases = best(M, b, restart=50, inner=inner, basis=basis, ortho=ortho)
        general = best(M, b, restart=113, inner_cap=50, inner=inner, basis=basis, ortho=ortho)
        print(f"{side} {inner}/{basis} ortho {ortho}: {1e6 * phases:.1f} and {1e6 * general:.1f} us")
        assert phases <= 1.2 * general
    M.close()


def test_one_reduction_kernels_past_the_limit():
    """ortho = 1 launched one by one past 65536 rows is the one-reduction iteration again."""
    say("phases, ortho 1")
    A = P.convdiff2d_system(1, 260).A
    M = B.Matrix.from_csr(A)
    b = torch.from_numpy(A.scipy() @ np.ones(A.n)).cuda()
    kw = dict(restart=30, inner="fp32", rtol=1e-14, max_iters=30, hist_cap=30, profile=1)
    h1, h0 = (B.solve(M, b, ortho=o, **kw)[2] for o in (1, 0))
    assert not np.array_equal(h1, h0) and np.max(np.abs(h1 - h0)) <= 1e-5
    M.close()
