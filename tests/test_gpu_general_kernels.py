"""The general kernels on small systems, where the cycle kernels take most calls.

The one-reduction CGS2 with a preconditioner (profile = 1 launches it: no cycle
kernel), and without the fused SpMV in every column-count class (matrices whose
rows share no offsets, under 65,536 rows), against the oracle's same mode.  HIP
graph replay, over several refinements and cycles, of systems that still record
one: restart lengths past the cycle kernels' and matrices without shared offsets.
Bars: fp64 histories within 1e-10, fp32 within 1e-5, solutions within 1e-8 at a
residual of 1e-12; replay and direct launches the same bits."""
import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

from oracle import linalg as L
from oracle import poly as PO
from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import bf16_hist_ok, dev_tensor, rel, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


def rhs(A, seed=0):
    return A.scipy() @ np.random.default_rng(seed).uniform(-1, 1, A.n)


def permuted(A, seed=3):
    """The same system in another order of its unknowns: no shared offsets, columns far from the row."""
    p = np.random.default_rng(seed).permutation(A.n)
    S = A.scipy()[p][:, p].tocsr()
    S.sort_indices()
    return P.CSR(A.n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)


def near(n, seed=5):
    """Rows of five entries within 300 columns, all different: 16-bit offsets."""
    rng = np.random.default_rng(seed)
    S = sp.csr_matrix((rng.uniform(-1, 1, 5 * n), (np.repeat(np.arange(n), 5),
                                                   np.clip(np.repeat(np.arange(n), 5) + rng.integers(-300, 301, 5 * n), 0, n - 1))),
                      shape=(n, n))
    S = S.tolil()
    S.setdiag(4.0)
    S = S.tocsr()
    S.sort_indices()
    return P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)


def compare(x, d, h, ref, tol):
    assert d["status"] == B.OK and ref.status == L.OK and d["rel_resid_true"] <= 1e-12
    k = ref.cycle_starts[1] if len(ref.cycle_starts) > 1 else len(ref.hist)
    assert np.max(np.abs(h[:k] - np.array(ref.hist[:k]))) <= tol
    assert rel(x.cpu().numpy(), ref.x) <= 1e-8


@pytest.mark.parametrize("side", [14, 42])  # 2744 rows: separate reduction, 74088: fused
def test_one_reduction_polynomial(side):
    A = P.conv_diff(3, side, 10.0, (1, 1, 1), (1, 1, 1e-2))
    bb = rhs(A)
    M, b = B.Matrix.from_csr(A), dev_tensor(bb)
    roots = PO.poly_roots(A, 10, start=PO.start_vector(A.n, 3), dtype=np.float32)
    say("one reduction, polynomial", side)
    x, d, h = B.solve(M, b, restart=30, inner="fp32", rtol=1e-12, poly_degree=10, poly_roots=roots, ortho="dcgs2",
                      hist_cap=5000, profile=1)
    ref = L.gmres_ir(A, bb, m=30, rtol=1e-12, inner="fp32", poly_roots=roots, check_mode=1, ortho="dcgs2")
    assert abs(d["iters"] - ref.iters) <= 30
    compare(x, d, h, ref, 1e-5)
    M.close()


@pytest.mark.parametrize("side", [64, 259])
def test_one_reduction_block_jacobi(side):
    A = P.conv_diff(2, side, 30.0, (1.0, -0.5))
    bb = rhs(A)
    M, b = B.Matrix.from_csr(A), dev_tensor(bb)
    say("one reduction, block Jacobi", side)
    x, d, h = B.solve(M, b, restart=50, inner="fp32", rtol=1e-12, bj_block=8, ortho="dcgs2", hist_cap=100000, profile=1)
    ref = L.gmres_ir(A, bb, m=50, rtol=1e-12, inner="fp32", bj_block=8, check_mode=1, ortho="dcgs2")
    compare(x, d, h, ref, 1e-5)
    M.close()


@pytest.mark.parametrize("inner", ["fp64", "fp32"])
@pytest.mark.parametrize("m", [1, 7, 16, 17, 33, 64, 65, 100, 128])
def test_one_reduction_column_classes(m, inner):
    A = permuted(P.conv_diff(2, 53, 20.0, (1.0, -0.5)))
    bb = rhs(A, m)
    M, b = B.Matrix.from_csr(A), dev_tensor(bb)
    assert M.layout in (1, 2)
    say("one reduction, no fused SpMV", m, inner)
    _, d, h = B.solve(M, b, restart=m, inner=inner, rtol=1e-12, check_mode=0, ortho="dcgs2", max_iters=m, hist_cap=m)
    ref = (L.gmres(A, bb, m=m, rtol=1e-12, ortho="dcgs2", max_iters=m) if inner == "fp64" else
           L.gmres_ir(A, bb, m=m, rtol=1e-12, inner="fp32", ortho="dcgs2", max_iters=m))
    assert d["iters"] == ref.iters == m
    assert np.max(np.abs(h - np.array(ref.hist[:m]))) <= (1e-10 if inner == "fp64" else 1e-5)
    M.close()


def test_one_and_two_reductions_agree():
    """Two different kernels here, unlike on systems whose cycle is one kernel."""
    A = permuted(P.conv_diff(2, 64, 30.0, (1.0, -0.5)))
    M, b = B.Matrix.from_csr(A), dev_tensor(rhs(A))
    say("one and two reductions")
    kw = dict(restart=50, inner="fp64", rtol=1e-12, max_iters=150, hist_cap=150)
    (x1, _, h1), (x0, _, h0) = B.solve(M, b, ortho="dcgs2", **kw), B.solve(M, b, **kw)
    assert not torch.equal(x1, x0) and np.max(np.abs(h1 - h0)) <= 1e-10
    M.close()


REPLAYED = {
    "restart 113": (lambda: P.conv_diff(2, 64, 30.0, (1.0, 0.3)), dict(restart=113)),
    "restart 120, bf16 basis": (lambda: P.conv_diff(2, 64, 30.0, (1.0, 0.3)), dict(restart=120, basis="bf16")),
    "restart 128, one reduction": (lambda: P.conv_diff(2, 64, 30.0, (1.0, 0.3)), dict(restart=128, ortho="dcgs2")),
    "far columns": (lambda: permuted(P.conv_diff(2, 64, 30.0, (1.0, 0.3))), dict(restart=30)),
    "far columns, fp64": (lambda: permuted(P.conv_diff(2, 64, 30.0, (1.0, 0.3))), dict(restart=30, inner="fp64")),
    "far columns, one reduction": (lambda: permuted(P.conv_diff(2, 64, 30.0, (1.0, 0.3))),
                                   dict(restart=30, ortho="dcgs2")),
    "far columns, several cycles": (lambda: permuted(P.conv_diff(2, 64, 30.0, (1.0, 0.3))),
                                    dict(restart=20, inner_cap=50)),
    "far columns, block Jacobi": (lambda: permuted(P.conv_diff(2, 64, 30.0, (1.0, 0.3))), dict(restart=30, bj_block=8)),
    "near columns": (lambda: near(20000), dict(restart=5)),
    "cycles of one step": (lambda: P.conv_diff(2, 20, 5.0, (1.0, 0.3)), dict(restart=1, max_iters=40)),
}


@pytest.mark.parametrize("case", sorted(REPLAYED))
def test_graph_replay(case):
    make, kw = REPLAYED[case]
    A = make()
    kw = dict(dict(inner="fp32", rtol=1e-10, hist_cap=20000), **kw)
    M, b = B.Matrix.from_csr(A), dev_tensor(rhs(A))
    say("graph replay", case)
    xg, dg, hg = B.solve(M, b, **kw)
    xg2, _, _ = B.solve(M, b, **kw)
    xd, dd, hd = B.solve(M, b, profile=1, **kw)
    assert dg["refinements"] >= 2 and dg["iters"] == dd["iters"] and dg["refinements"] == dd["refinements"]
    assert torch.equal(xg, xd) and torch.equal(xg, xg2) and np.array_equal(hg, hd)
    M.close()
