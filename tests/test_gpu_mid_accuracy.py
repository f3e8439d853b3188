"""Whole solves of large 7-point systems by the larger systems' cycle kernel.

The kernel sums in another order than the general ones, and where that ends a
refinement elsewhere the solution moves.  Anisotropic convection-diffusion of
729,000 and 1,030,301 rows to a residual of 1e-12, several right-hand sides,
against the exact solution: as accurate as the general kernels' solution, and no
further from it than either is from the exact one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import dev_tensor, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,inner,seeds", [(90, "fp32", 4), (101, "fp32", 2), (101, "fp64", 2)])
def test_aniso3d(side, inner, seeds):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    A = P.aniso3d_system(0, side).A
    S = A.scipy()
    M = B.Matrix.from_csr(A)
    for seed in range(seeds):
        say("mid accuracy", side, inner, seed)
        u = np.random.default_rng(seed).uniform(-1, 1, A.n)
        b = dev_tensor(S @ u)
        kw = dict(restart=50, inner=inner, rtol=1e-12, max_iters=20000)
        x, d, _ = B.solve(M, b, **kw)
        xp, dp, _ = B.solve(M, b, profile=1, **kw)
        assert d["status"] == dp["status"] == 0 and max(d["rel_resid_true"], dp["rel_resid_true"]) <= 1e-12
        x, xp = x.cpu().numpy(), xp.cpu().numpy()
        e, ep = rel(x, u), rel(xp, u)
        print(f"{side} {inner} {seed}: {e:.2e} and {ep:.2e}, apart {rel(x, xp):.2e}")
        assert e <= 2 * ep and rel(x, xp) <= max(e, ep)
    M.close()
