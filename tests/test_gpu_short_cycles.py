"""Short cycles go to the kernels that make them faster.

Times against the general kernels on the same cycles: restart = 113 is past the
limits of the cycle kernels, inner_cap gives its cycles the same length.  The
larger systems' cycle kernel at the first lengths it takes, in every number of
steps per block: its histories against the general kernels' (profile = 1) at the
parity bars, and not their bits, so that it is what ran; at one step less they
are the same."""
import time

import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import bf16_hist_ok, dev_tensor, say

pytestmark = pytest.mark.gpu
SLICE = 256 * 64  # rows of one slice per block


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def banded(n, offsets=(-700, -30, -1, 0, 1, 30, 700)):
    rng = np.random.default_rng(n)
    d = [np.full(n - abs(o), 1.12 * len(offsets) ** 0.5) if o == 0 else rng.uniform(-1, 1, n - abs(o)) for o in offsets]
    S = sp.diags(d, offsets, shape=(n, n), format="csr")
    S.sort_indices()
    M = B.Matrix.from_csr(P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data))
    return M, dev_tensor(S @ np.random.default_rng(1).uniform(-1, 1, n))


@pytest.mark.parametrize("fam,side,inner,m", [
    ("laplace2d_5", 64, "fp32", 1), ("laplace2d_5", 500, "fp32", 1), ("box3d_27", 62, "fp32", 2),
    ("box3d_27", 45, "fp64", 1), ("laplace2d_5", 500, "fp64", 4), ("laplace3d_7", 81, "fp64", 5),
    ("laplace3d_7", 101, "fp32", 5), ("laplace3d_7", 101, "fp64", 20), ("laplace3d_7", 127, "fp32", 10)])
def test_not_slower_than_general(fam, side, inner, m):
    say("short cycles", fam, side, inner, m)
    A = P.stencil_matrix(fam, side)
    M = B.Matrix.from_csr(A)
    b = torch.from_numpy(np.random.default_rng(0).uniform(-1, 1, A.n)).cuda()

    def best(**kw):
        p = B.make_params(inner=inner, rtol=1e-14, max_iters=60, check_mode=0, **kw)
        x, ws, t = torch.zeros_like(b), B.Workspace(), []
        for _ in range(6):
            x.zero_()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, d, _ = B.gmresir_solve(M, b, x, p, ws=ws)
            torch.cuda.synchronize()
            t.append((time.perf_counter() - t0) / d["iters"])
        return 1e6 * min(t)

    short, capped, general = best(restart=m), best(restart=50, inner_cap=m), best(restart=113, inner_cap=m)
    print(f"{short:.1f}, {capped:.1f} and {general:.1f} us")
    assert max(short, capped) <= 1.08 * general
    M.close()


@pytest.mark.parametrize("inner,basis,m,n", [
    ("fp32", "fp32", 4, 20 * SLICE), ("fp32", "fp32", 8, 24 * SLICE + 1), ("fp32", "fp32", 14, 32 * SLICE + 65),
    ("fp32", "fp32", 25, 64 * SLICE), ("fp32", "fp32", 30, 128 * SLICE),
    ("fp32", "bf16", 8, 32 * SLICE), ("fp32", "bf16", 12, 40 * SLICE - 3), ("fp32", "bf16", 27, 48 * SLICE),
    ("fp32", "bf16", 27, 48 * SLICE + 2), ("fp32", "bf16", 36, 80 * SLICE - 5), ("fp32", "bf16", 36, 81 * SLICE),
    ("fp64", "fp64", 29, 15 * SLICE + 9), ("fp64", "fp64", 12, 20 * SLICE), ("fp64", "fp64", 22, 20 * SLICE + 63),
    ("fp64", "fp64", 26, 64 * SLICE)])
def test_first_lengths(inner, basis, m, n):
    say("mid first lengths", inner, basis, m, n)
    M, b = banded(n)

    def both(m):
        kw = dict(restart=m, inner=inner, basis=basis, rtol=1e-30, max_iters=m, hist_cap=m)
        (x, _, h), (xp, _, hp) = B.solve(M, b, **kw), B.solve(M, b, profile=1, **kw)
        return h, hp, torch.equal(x, xp)

    hc, hp, same = both(m)
    assert not same
    if basis == "bf16":
        ok, info = bf16_hist_ok(hc, hp)
        assert ok, info
    else:
        assert np.max(np.abs(hc - hp)) <= (1e-10 if inner == "fp64" else 1e-5)
    if m != 29:  # that one is the restart the smaller systems' kernel leaves to this one
        assert both(m - 1)[2]
    M.close()
