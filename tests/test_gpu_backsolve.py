"""The triangular solve at the end of a cycle, at the edges of its forms: up to
64 rows (one register of a lane), up to what fits LDS (100 rows in fp64, 142 in
fp32), the triangle read from memory past that, the longest restart.

One cycle of k steps on the 1D Laplacian, which does not converge in it; the
solution against the oracle's.  The triangle's condition is about (2k/pi)^2: 1e5
at 512, so 1e-9 holds a wide margin in fp64; 8e3 at 143, times fp32's 6e-8:
1e-3."""
import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

from oracle import linalg as L
from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import dev_tensor, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inner,k", [("fp64", k) for k in (1, 2, 63, 64, 65, 100, 101, 128, 129, 200, 512)] +
                         [("fp32", k) for k in (1, 64, 65, 128, 129, 142, 143)])
def test_cycle_of_k_steps(inner, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say("backsolve", inner, k)
    n = 3000
    S = sp.diags([np.full(n - 1, -1.0), np.full(n, 2.0), np.full(n - 1, -1.0)], (-1, 0, 1), format="csr")
    A = P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)
    b = S @ np.random.default_rng(k).uniform(-1, 1, n)
    M = B.Matrix.from_csr(A)
    x, d, _ = B.solve(M, dev_tensor(b), restart=k, inner=inner, rtol=1e-14, max_iters=k)
    ref = (L.gmres(A, b, m=k, rtol=1e-14, max_iters=k) if inner == "fp64" else
           L.gmres_ir(A, b, m=k, rtol=1e-14, inner="fp32", max_iters=k))
    assert d["iters"] == k
    assert np.linalg.norm(x.cpu().numpy() - ref.x) <= (1e-9 if inner == "fp64" else 1e-3) * np.linalg.norm(ref.x)
    M.close()
