"""Cycles of systems whose basis fits the compute units' registers.

The cycle kernel (one cooperative launch, blocks exchanging their sums inside
it) and its phases launched one by one (profile = 1) do the same operations in
the same order, so their solutions and histories agree bit for bit; the
phases read the basis and the vector from memory and have no exchange to get
wrong.  Sizes sit at the edges of the slices and the blocks, in the ranges
of several numbers of rows per lane (the edges of those:
test_gpu_small_partitions.py) and at the largest system of the path; both are
held to the oracle's first cycle at the parity bars."""
import threading

import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

from oracle import linalg as L
from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import bf16_hist_ok, dev_tensor, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


def banded(n, offsets, seed=0):
    """n x n, constant offsets (entries that leave the matrix dropped), diagonally dominant."""
    rng = np.random.default_rng(seed)
    offsets = [o for o in offsets if abs(o) < n]
    d = [np.full(n - abs(o), 2.0 * len(offsets)) if o == 0 else rng.uniform(-1, 1, n - abs(o)) for o in offsets]
    S = sp.diags(d, offsets, shape=(n, n), format="csr")
    S.sort_indices()
    return P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)


def both(A, m, inner, basis, max_iters, oracle=True):
    M = B.Matrix.from_csr(A)
    assert M.layout == (3 if A.n >= 63 else 0)  # a slice of one or two rows is mostly padding: row tiles
    u = np.random.default_rng(A.n + m).uniform(-1, 1, A.n)
    bb = A.scipy() @ u
    b = dev_tensor(bb)
    kw = dict(restart=m, inner=inner, basis=basis, rtol=1e-11, max_iters=max_iters, hist_cap=max_iters)
    xc, dc, hc = B.solve(M, b, **kw)
    xp, dp, hp = B.solve(M, b, profile=1, **kw)
    assert dc["status"] == dp["status"] and dc["iters"] == dp["iters"]
    assert torch.equal(xc, xp) and np.array_equal(hc, hp)
    assert np.isfinite(xc.cpu().numpy()).all()
    if oracle:
        ref = (L.gmres(A, bb, m=m, rtol=1e-11, max_iters=m, check_mode=1) if inner == "fp64" else
               L.gmres_ir(A, bb, m=m, rtol=1e-11, inner="fp32", basis=basis, max_iters=m, check_mode=1))
        # the first cycle only: after an exact termination the next one starts from rounding noise
        k = min(len(hc), dc["iters"], m, ref.cycle_starts[1] if len(ref.cycle_starts) > 1 else len(ref.hist))
        if basis == "bf16":
            ok, info = bf16_hist_ok(hc[:k], ref.hist[:k])
            assert ok, info
        else:
            assert np.max(np.abs(hc[:k] - np.array(ref.hist[:k]))) <= (1e-10 if inner == "fp64" else 1e-5)
    M.close()


KINDS = [("fp32", "fp32"), ("fp64", "fp64"), ("fp32", "bf16")]


@pytest.mark.parametrize("inner,basis", KINDS)
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 1000, 4097, 8192])
def test_sizes(n, inner, basis):
    say("small sizes", n, inner, basis)
    both(banded(n, (-33, -1, 0, 1, 33), n), 20, inner, basis, 45)


# restart length (4, 8 or 16 columns a wave) and rows: 4, 8, 12 and 16 rows a lane
# in fp32, 4 to 16 in fp64, up to the most of each restart length
@pytest.mark.parametrize("inner,m,n", [
    ("fp32", 28, 128 * 192), ("fp32", 28, 128 * 768 + 1), ("fp32", 29, 128 * 256 + 1), ("fp32", 56, 128 * 512),
    ("fp32", 50, 128 * 1024 + 63), ("fp32", 50, 262144), ("fp32", 57, 128 * 128 + 1), ("fp32", 112, 131072),
    ("fp64", 28, 64 * 1024 + 1), ("fp64", 56, 64 * 384 + 1), ("fp64", 50, 131072), ("fp64", 112, 65536)])
def test_rows_per_lane(inner, m, n):
    say("small rows per lane", inner, m, n)
    both(banded(n, (-300, -1, 0, 1, 300), m), m, inner, inner, m + 3, oracle=False)


@pytest.mark.parametrize("inner,n", [("fp32", 262145), ("fp64", 131073)])
def test_past_the_largest(inner, n):
    """One row more than the path takes: the general kernels, same bars."""
    say("small past the largest", inner, n)
    both(banded(n, (-1, 0, 1), 3), 50, inner, inner, 8)


@pytest.mark.parametrize("inner,basis", KINDS)
def test_wide_rows_and_rows_gathered_one_by_one(inner, basis):
    """27-point rows (values too many for LDS in the larger fp64 blocks), rows
    of 40 scattered offsets (more 64-row chunks of x than a block keeps, so
    every row is gathered from memory), and slices without entries."""
    say("small wide rows", inner, basis)
    both(P.varcoef27(20, 5), 50, inner, basis, 53)
    far = [0] + [s * (97 * k + 31) for k in range(1, 21) for s in (-1, 1)]
    both(banded(5000, sorted(far), 1), 30, inner, basis, 33)
    A = banded(2000, (-64, 0, 64), 2)
    S = A.scipy().tolil()
    S[512:640, :] = 0
    S[512:640, 512:640] = 0
    S = S.tocsr()
    S.eliminate_zeros()
    H = P.CSR(2000, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)
    M = B.Matrix.from_csr(H)
    b = dev_tensor(H.scipy() @ np.ones(2000))
    kw = dict(restart=20, inner=inner, basis=basis, rtol=1e-6, max_iters=25, hist_cap=25)
    xc, dc, hc = B.solve(M, b, **kw)
    xp, dp, hp = B.solve(M, b, profile=1, **kw)
    assert dc["status"] == dp["status"] and torch.equal(xc, xp) and np.array_equal(hc, hp)


@pytest.mark.parametrize("inner,basis", KINDS)
@pytest.mark.parametrize("n", [64 * 256, 64 * 256 + 1, 72 * 256, 73 * 256 - 1, 128 * 256, 128 * 256 + 1, 200 * 256 + 3, 65537])
def test_exchange_in_one_and_two_stages(n, inner, basis):
    """64 blocks (every block reads every line), 65 and more (groups of up to
    16 blocks of a die first: one of nine blocks, full ones, a second per die
    of one block and of several)."""
    say("small stages", n, inner, basis)
    both(banded(n, (-600, -1, 0, 1, 600), n), 40, inner, basis, 43, oracle=False)


def test_threads_and_streams():
    """Four threads, each with its own stream and workspace, solve different
    systems at the same time: the bits of solving alone."""
    systems = [banded(n, (-40, -1, 0, 1, 40), n) for n in (3000, 20000, 60000, 200000)]
    mats = [B.Matrix.from_csr(A) for A in systems]
    rhs = [dev_tensor(A.scipy() @ np.ones(A.n)) for A in systems]
    kw = dict(restart=30, inner="fp32", rtol=1e-12, max_iters=120)
    alone = [B.solve(M, b, **kw)[0] for M, b in zip(mats, rhs)]
    torch.cuda.synchronize()
    got, errors = [None] * 4, []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(5):
                    got[i] = B.solve(mats[i], rhs[i], **kw)[0]
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # reported by the assert below
            errors.append(e)

    say("small threads")
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for a, g in zip(alone, got):
        assert torch.equal(a, g)
