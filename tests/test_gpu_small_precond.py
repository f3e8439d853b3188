"""Preconditioned cycles of small systems in one kernel.

Against the general kernels (profile = 1: another order of sums), which the
oracle holds, at the parity bars of a cycle's history.  Sizes at the edges of
the slices, of one and two stages of the exchange and of the rows per lane;
block sizes that divide 64 and the whole slice; polynomials of one SpMV up to
many, with real and complex roots; matrices whose blocks read from one side
only.  Block sizes, windows and row counts the kernel leaves to the general
ones: their bits."""
import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import bf16_hist_ok, dev_tensor, say

pytestmark = pytest.mark.gpu
KINDS = [("fp32", "fp32"), ("fp64", "fp64"), ("fp32", "bf16")]
SIDES = (-300, -1, 0, 1, 300)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


def system(n, offsets):
    rng = np.random.default_rng(n)
    offsets = [o for o in offsets if abs(o) < n]
    d = [np.full(n - abs(o), 0.5 * len(offsets) + 0.5) if o == 0 else rng.uniform(-1, 1, n - abs(o)) for o in offsets]
    S = sp.diags(d, offsets, shape=(n, n), format="csr")
    S.sort_indices()
    M = B.Matrix.from_csr(P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data))
    return M, dev_tensor(S @ rng.uniform(-1, 1, n))


def compare(M, b, m, inner, basis, iters, same=False, **kw):
    kw = dict(restart=m, inner=inner, basis=basis, rtol=1e-9, max_iters=iters, hist_cap=iters, **kw)
    (x, d, h), (xp, dp, hp) = B.solve(M, b, **kw), B.solve(M, b, profile=1, **kw)
    torch.cuda.synchronize()
    assert torch.isfinite(x).all()
    if same:
        assert torch.equal(x, xp) and np.array_equal(h, hp)
        return
    # the first cycle: one that ends at rtol is followed by another from rounding noise
    k = min(d["iters"], dp["iters"], m)
    k = next((i for i in range(1, k) if hp[i] > 2 * hp[i - 1]), k)
    assert k >= min(4, iters) and abs(d["iters"] - dp["iters"]) <= max(2, iters // 8)
    if basis == "bf16":
        ok, info = bf16_hist_ok(h[:k], hp[:k])
        assert ok, info
    else:
        assert np.max(np.abs(h[:k] - hp[:k])) <= (1e-10 if inner == "fp64" else 1e-5)


def roots_of(count, pairs):
    """In the spectrum's half plane; `pairs` conjugate pairs, the others real."""
    r = []
    for i in range(pairs):
        r += [complex(2.0 + 0.1 * i, 0.9 - 0.05 * i), complex(2.0 + 0.1 * i, -(0.9 - 0.05 * i))]
    return np.array(r + [complex(2.2 + 0.15 * i) for i in range(count - 2 * pairs)])


@pytest.mark.parametrize("inner,basis", KINDS)
@pytest.mark.parametrize("n,bs", [(64, 1), (130, 2), (1000, 8), (4099, 16), (64 * 256, 32), (64 * 256 + 5, 64), (40001, 4),
                                  (65537, 8), (131072, 16)])
def test_block_jacobi(n, bs, inner, basis):
    say("small block Jacobi", n, bs, inner, basis)
    compare(*system(n, SIDES), 30, inner, basis, 30, bj_block=bs)


@pytest.mark.parametrize("inner,basis", KINDS)
@pytest.mark.parametrize("n,count,pairs", [(64, 2, 0), (129, 2, 1), (1000, 3, 1), (4099, 4, 2), (64 * 256, 5, 1),
                                           (64 * 256 + 5, 6, 3), (40001, 11, 2), (65537, 7, 0), (131072, 4, 1)])
def test_polynomial(n, count, pairs, inner, basis):
    say("small polynomial", n, count, pairs, inner, basis)
    compare(*system(n, SIDES), 30, inner, basis, 12, poly_degree=count - 1, poly_roots=roots_of(count, pairs))


@pytest.mark.parametrize("m", [28, 29, 56, 57, 112])
@pytest.mark.parametrize("inner", ["fp32", "fp64"])
def test_column_classes(m, inner):
    say("small precond classes", m, inner)
    M, b = system(20000, SIDES)
    compare(M, b, m, inner, inner, m, bj_block=8)
    compare(M, b, m, inner, inner, 10, poly_degree=2, poly_roots=roots_of(3, 1))


@pytest.mark.parametrize("offsets", [(0, 1, 700), (-700, -1, 0), (-2500, 0, 1)])
def test_one_sided(offsets):
    """Blocks that read from blocks that do not read from them."""
    say("small precond one-sided", offsets)
    M, b = system(30000, offsets)
    compare(M, b, 30, "fp32", "fp32", 8, poly_degree=8, poly_roots=roots_of(9, 2))
    compare(M, b, 30, "fp64", "fp64", 8, poly_degree=8, poly_roots=roots_of(9, 2))


@pytest.mark.parametrize("n,offsets,m,kw", [
    (5000, SIDES, 30, dict(bj_block=7)),                        # slices cut its blocks
    (30000, (-20000, 0, 20000), 30, dict(bj_block=8)),          # blocks too far apart
    (30000, (-20000, 0, 20000), 30, dict(poly_degree=2)),
    (20000, tuple(sorted([0] + [s * (197 * k + 31) for k in range(1, 41) for s in (-1, 1)])), 30, dict(bj_block=8)),  # window
    (5000, SIDES, 113, dict(bj_block=8)), (263000, SIDES, 30, dict(bj_block=8))])
def test_general_kernels_still_take(n, offsets, m, kw):
    say("small precond not taken", n, m, kw)
    if "poly_degree" in kw:
        kw = dict(kw, poly_roots=roots_of(3, 1))
    compare(*system(n, offsets), m, "fp32", "fp32", 10, same=True, **kw)


def test_whole_solves_in_threads():
    """Solves of all kinds at the same time, each on its own stream: the bits of solving alone."""
    import threading
    M, b = system(20000, SIDES)
    kws = [dict(restart=30, inner="fp32", rtol=1e-11, max_iters=400, **k) for k in
           (dict(bj_block=8), dict(poly_degree=4, poly_roots=roots_of(5, 2)), dict())]
    alone = [B.solve(M, b, **kw) for kw in kws]
    assert all(a[1]["status"] == 0 for a in alone)
    got = [None] * 3

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                got[i] = B.solve(M, b, **kws[i])[0]
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert all(torch.equal(a[0], g) for a, g in zip(alone, got))
