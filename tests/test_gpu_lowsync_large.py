"""The one-reduction CGS2 past the sizes whose cycle is one kernel, and on them.

Its kernels at every column-count class on 265225 rows (profile = 1 launches
them one by one), against two-pass CGS2's general kernels at the parity bars:
the cycles are equal in exact arithmetic.  Where a cycle is one kernel ortho 1
makes the passes of ortho 0: the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import dev_tensor, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def large():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    A = P.convdiff2d_system(3, 515).A
    M = B.Matrix.from_csr(A)
    yield M, dev_tensor(A.scipy() @ np.random.default_rng(1).uniform(-1, 1, A.n))
    M.close()


@pytest.mark.parametrize("inner", ["fp32", "fp64"])
@pytest.mark.parametrize("m", [1, 7, 16, 17, 33, 64, 65, 100, 128])
def test_restart_classes(large, m, inner):
    say("lowsync large", m, inner)
    kw = dict(restart=m, inner=inner, rtol=1e-14, max_iters=m, hist_cap=m, profile=1)
    (_, d, h), (_, d0, h0) = B.solve(*large, ortho="dcgs2", **kw), B.solve(*large, **kw)
    assert d["iters"] == d0["iters"] == m
    assert np.max(np.abs(h - h0)) <= (1e-10 if inner == "fp64" else 1e-5)
    if m > 64:  # the same kernels without profile
        x, _, h1 = B.solve(*large, ortho="dcgs2", **{**kw, "profile": 0})
        assert np.array_equal(h, h1) and torch.isfinite(x).all()


@pytest.mark.parametrize("inner", ["fp32", "fp64"])
@pytest.mark.parametrize("side", [16, 64, 200])
def test_one_kernel_cycles(side, inner):
    say("lowsync in one kernel", side, inner)
    A = P.convdiff2d_system(side, side).A
    M, b = B.Matrix.from_csr(A), dev_tensor(A.scipy() @ np.ones(A.n))
    kw = dict(restart=40, inner=inner, rtol=1e-11, max_iters=200, hist_cap=200)
    (x, _, h), (x0, _, h0) = B.solve(M, b, ortho="dcgs2", **kw), B.solve(M, b, **kw)
    assert torch.equal(x, x0) and np.array_equal(h, h0)
    M.close()


def test_mid_cycles(large):
    say("lowsync, part of the basis in registers")
    kw = dict(restart=40, inner="fp32", rtol=1e-11, max_iters=90, hist_cap=90)
    (x, _, h), (x0, _, h0) = B.solve(*large, ortho="dcgs2", **kw), B.solve(*large, **kw)
    assert torch.equal(x, x0) and np.array_equal(h, h0)
