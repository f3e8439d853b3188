"""Small systems with wide rows: the cycle kernel where it is the faster one.

Bands and stencils of many entries a row keep their window of x in LDS whatever
their number of (slice, offset) pairs; scattered entries that do not fit a
window are gathered one by one up to a number of entries per lane and go to the
general kernels past it.  Bits: the cycle kernel's are those of profile = 1
(phases), the general kernels' too.  Times against the general kernels on the
same cycles (restart 113 is past the cycle kernel's limit, inner_cap = 50)."""
import time

import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import dev_tensor, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def system(n, offsets):
    rng = np.random.default_rng(n)
    offsets = sorted(o for o in offsets if abs(o) < n)
    d = [np.full(n - abs(o), 1.12 * len(offsets) ** 0.5) if o == 0 else rng.uniform(-1, 1, n - abs(o)) for o in offsets]
    S = sp.diags(d, offsets, shape=(n, n), format="csr")
    S.sort_indices()
    M = B.Matrix.from_csr(P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data))
    assert M.layout == 3
    return M, dev_tensor(S @ np.random.default_rng(1).uniform(-1, 1, n))


def band(w):
    return range(-w, w + 1)


def scattered(n, k):
    return [0] + [s * (n // (2 * k + 50) * i + 31) for i in range(1, k + 1) for s in (-1, 1)]


# pairs of a block: 512 and one slice more, the most that 16 rows a lane and 512 entries a row give;
# windows that do not fit, on both sides of the limit of entries per lane
@pytest.mark.parametrize("inner,basis", [("fp32", "fp32"), ("fp64", "fp64"), ("fp32", "bf16")])
@pytest.mark.parametrize("n,offsets", [
    (16385, range(-63, 65)), (16385, range(-64, 65)), (8192, band(128)), (5000, band(250)), (20000, band(255)),
    (70000, band(60)), (131072, band(40)), (100000, band(100)),
    (100000, scattered(100000, 20)), (100000, scattered(100000, 70)), (200000, scattered(200000, 40)),
    (262144, scattered(262144, 30)), (262144, band(70))])
def test_bits(n, offsets, inner, basis):
    say("wide rows", n, len(list(offsets)), inner, basis)
    if inner == "fp64" and n > 131072:
        pytest.skip("past the small kernel's limit in fp64")
    M, b = system(n, offsets)
    kw = dict(restart=50, inner=inner, basis=basis, rtol=1e-12, max_iters=53, hist_cap=53)
    (x, d, h), (xp, dp, hp) = B.solve(M, b, **kw), B.solve(M, b, profile=1, **kw)
    assert torch.isfinite(x).all() and torch.equal(x, xp) and np.array_equal(h, hp)
    M.close()


@pytest.mark.parametrize("inner", ["fp32", "fp64"])
@pytest.mark.parametrize("n,offsets", [
    (200000, band(40)), (100000, band(150)), (131072, scattered(131072, 60)), (262144, scattered(262144, 40))])
def test_not_slower_than_general(n, offsets, inner):
    say("wide rows against general", n, len(list(offsets)), inner)
    if inner == "fp64" and n > 131072:
        pytest.skip("past the small kernel's limit in fp64")
    M, b = system(n, offsets)

    def best(**kw):
        p = B.make_params(inner=inner, rtol=1e-14, max_iters=100, check_mode=0, **kw)
        x, ws, t = torch.zeros_like(b), B.Workspace(), []
        for _ in range(6):
            x.zero_()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, d, _ = B.gmresir_solve(M, b, x, p, ws=ws)
            torch.cuda.synchronize()
            t.append((time.perf_counter() - t0) / d["iters"])
        return 1e6 * min(t)

    one, general = best(restart=50), best(restart=113, inner_cap=50)
    print(f"{one:.1f} and {general:.1f} us")
    assert one <= 1.15 * general
    M.close()
