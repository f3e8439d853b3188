"""Cycles of systems whose basis fits the compute units' registers in part.

The cycle kernel sums in another order than the general kernels (profile = 1),
which the oracle holds, so histories of a cycle agree to the parity bars of
the precision and solutions to their accuracy.  Sizes: the edges of the steps
per block (5, 6, 8, 10, 16 or 32 of 4 slices in fp32, 8 with a bf16 basis, 2
in fp64, for 256 blocks), a partial last slice, the smallest and the largest."""
import threading

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
    yield
    torch.cuda.synchronize()


def banded(n, offsets, seed=0):
    """n x n, constant offsets; no cycle here ends early: the residual of 64 steps stays over 1e-18"""
    rng = np.random.default_rng(seed)
    d = [np.full(n - abs(o), 1.12 * len(offsets) ** 0.5) if o == 0 else rng.uniform(-1, 1, n - abs(o)) for o in offsets]
    S = sp.diags(d, offsets, shape=(n, n), format="csr")
    S.sort_indices()
    return P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)


def system(A):
    M = B.Matrix.from_csr(A)
    return M, dev_tensor(A.scipy() @ np.random.default_rng(A.n).uniform(-1, 1, A.n))


def cycle(M, b, m, inner, basis, iters):
    kw = dict(restart=m, inner=inner, basis=basis, rtol=1e-30, max_iters=iters, hist_cap=iters, check_mode=1)
    (xc, dc, hc), (xp, dp, hp) = B.solve(M, b, **kw), B.solve(M, b, profile=1, **kw)
    torch.cuda.synchronize()
    assert dc["iters"] == dp["iters"] and torch.isfinite(xc).all()
    return xc, hc, xp, hp


@pytest.mark.parametrize("inner,basis,m,n", [
    ("fp32", "fp32", 50, (1 << 18) + 1025), ("fp32", "fp32", 1, 20 * SLICE), ("fp32", "fp32", 9, 20 * SLICE + 1),
    ("fp32", "fp32", 56, 24 * SLICE - 63), ("fp32", "fp32", 64, 32 * SLICE), ("fp32", "fp32", 8, 32 * SLICE + 65),
    ("fp32", "fp32", 30, 40 * SLICE + 5), ("fp32", "fp32", 50, 64 * SLICE + 2), ("fp32", "fp32", 17, 128 * SLICE),
    ("fp32", "fp32", 57, (1 << 17) + 1025), ("fp32", "fp32", 64, 16 * SLICE + 3),
    ("fp64", "fp64", 50, (1 << 17) + 1025), ("fp64", "fp64", 33, 10 * SLICE + 7), ("fp64", "fp64", 64, 12 * SLICE),
    ("fp64", "fp64", 50, 16 * SLICE + 1), ("fp64", "fp64", 20, 20 * SLICE + 63), ("fp64", "fp64", 25, 64 * SLICE),
    ("fp32", "bf16", 64, 32 * SLICE - 1), ("fp32", "bf16", 50, 40 * SLICE), ("fp32", "bf16", 20, 48 * SLICE + 2),
    ("fp32", "bf16", 50, 64 * SLICE + 7), ("fp32", "bf16", 30, 80 * SLICE - 5), ("fp32", "bf16", 50, 128 * SLICE)])
def test_steps(inner, basis, m, n):
    say("mid steps", inner, basis, m, n)
    M, b = system(banded(n, (-700, -30, -1, 0, 1, 30, 700), n))
    _, hc, _, hp = cycle(M, b, m, inner, basis, m)
    if basis == "bf16":
        ok, info = bf16_hist_ok(hc, hp)
        assert ok, info
    else:
        assert np.max(np.abs(hc - hp)) <= (1e-10 if inner == "fp64" else 1e-5)
    M.close()


@pytest.mark.parametrize("inner,basis,A", [
    ("fp32", "fp32", lambda: P.convdiff2d_system(1, 520).A), ("fp32", "bf16", lambda: P.varcoef27(65, 3)),
    ("fp64", "fp64", lambda: P.aniso3d_system(2, 52).A)])
def test_solves(inner, basis, A):
    """Whole solves, stencils with wide windows: the exact solution at the residual asked for."""
    A = A()
    say("mid solve", inner, basis, A.n)
    M = B.Matrix.from_csr(A)
    u = np.random.default_rng(4).uniform(-1, 1, A.n)
    x, d, _ = B.solve(M, dev_tensor(A.scipy() @ u), restart=50, inner=inner, basis=basis, rtol=1e-12, max_iters=6000)
    assert d["status"] == 0 and d["rel_resid_true"] <= 1e-12
    # the same accuracy as the general kernels' at the same residual
    xp, dp, _ = B.solve(M, dev_tensor(A.scipy() @ u), restart=50, inner=inner, basis=basis, rtol=1e-12, max_iters=6000,
                        profile=1)
    e, ep = (np.linalg.norm(v.cpu().numpy() - u) / np.linalg.norm(u) for v in (x, xp))
    assert e <= max(1e-8, 4 * ep)
    M.close()


@pytest.mark.parametrize("what", ["long restart", "window too wide", "rows of their own", "too large", "narrow rows"])
def test_general_kernels_still_take(what):
    """Systems the cycle kernel leaves to the general ones: their bits."""
    n, m = 300000, 20
    if what == "long restart":
        A, m = banded(n, (-1, 0, 1), 1), 65
    elif what == "window too wide":
        A = banded(n, sorted([0] + [s * (9000 * k + 31) for k in range(1, 14) for s in (-1, 1)]), 2)
    elif what == "too large":
        A = banded(128 * SLICE + 1, (-9, -2, -1, 0, 1, 2, 9), 3)
    elif what == "narrow rows":
        A = banded((1 << 19) + 1, (-700, -1, 0, 1, 700), 4)
    else:
        rng = np.random.default_rng(5)
        col = np.sort((np.arange(n)[:, None] + np.concatenate([[[0]] * n, rng.integers(1, 300, (n, 4))], 1)) % n, 1)
        S = sp.csr_matrix((np.ones(5 * n), (np.repeat(np.arange(n), 5), col.ravel())), shape=(n, n))
        S.setdiag(12.0)
        S.sort_indices()
        A = P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)
    say("mid not taken", what)
    M, b = system(A)
    xc, hc, xp, hp = cycle(M, b, m, "fp32", "fp32", m + 2)
    assert torch.equal(xc, xp) and np.array_equal(hc, hp)
    M.close()


def test_threads_and_streams():
    """Three threads solve systems of both cycle kernels at the same time: the bits of solving alone."""
    systems = [system(banded(n, (-40, -1, 0, 1, 40), n)) for n in (290000, 60000, 400001)]
    kw = dict(restart=30, inner="fp32", rtol=1e-12, max_iters=120)
    alone = [B.solve(M, b, **kw)[0] for M, b in systems]
    torch.cuda.synchronize()
    got, errors = [None] * 3, []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    got[i] = B.solve(*systems[i], **kw)[0]
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # reported by the assert below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not errors
    assert all(torch.equal(a, g) for a, g in zip(alone, got))
