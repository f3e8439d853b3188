"""Solves beside other work that holds compute units.

A cycle kernel's blocks wait for each other, so all of them have to be on the
GPU.  A running sum over two long rows occupies one compute unit for most of a
second: a cycle kernel that wants every one gives up after 0.1 s and the solve
goes on with kernels launched one by one, without waiting for the sum; where
those sum in another order its bits are the ones of profile = 1.  Two processes
whose cycle kernels want every compute unit at once both finish."""
import os
import subprocess
import sys
import time

import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import dev_tensor, say

pytestmark = pytest.mark.gpu
ROOTS = np.array([complex(2.0 + 0.11 * i) for i in range(21)])


def banded(n, offsets):
    rng = np.random.default_rng(n)
    d = [np.full(n - abs(o), 0.5 * len(offsets) + 0.5) if o == 0 else rng.uniform(-1, 1, n - abs(o)) for o in offsets]
    S = sp.diags(d, offsets, shape=(n, n), format="csr")
    S.sort_indices()
    return S


def system(n):
    S = banded(n, (-300, -30, -1, 0, 1, 30, 300))
    M = B.Matrix.from_csr(P.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data))
    return M, dev_tensor(S @ np.random.default_rng(1).uniform(-1, 1, n))


class Busy:
    """One compute unit busy for about `seconds` on a stream of its own."""

    def __init__(self, seconds):
        self.stream = torch.cuda.Stream()
        small = torch.ones(2, 1 << 20, device="cuda")
        torch.cumsum(small, 1)
        torch.cuda.synchronize()
        t = time.perf_counter()
        torch.cumsum(small, 1)
        torch.cuda.synchronize()
        n = int((1 << 20) * seconds / (time.perf_counter() - t))
        self.x = torch.ones(2, min(n, 1 << 28), device="cuda")
        self.out = torch.empty_like(self.x)
        torch.cuda.synchronize()

    def __enter__(self):
        with torch.cuda.stream(self.stream):
            torch.cumsum(self.x, 1, out=self.out)
            self.done = torch.cuda.Event()
            self.done.record()
        time.sleep(0.02)
        return self

    def running(self):
        return not self.done.query()

    def __exit__(self, *exc):
        torch.cuda.synchronize()


@pytest.fixture(scope="module")
def busy():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    return Busy(0.9)


@pytest.mark.parametrize("n,kw,same", [
    (300000, dict(), False), (300000, dict(inner_cap=75), False), (262144, dict(), True),
    (262144, dict(poly_degree=20, poly_roots=ROOTS), False), (262144, dict(bj_block=8), False)])
def test_solve_beside_a_long_kernel(busy, n, kw, same):
    say("beside a long kernel", n, {k: v for k, v in kw.items() if k != "poly_roots"})
    M, b = system(n)
    kw = dict(restart=30, inner="fp32", rtol=1e-11, max_iters=150, hist_cap=150, **kw)
    ws = B.Workspace()
    x, d, h = B.solve(M, b, ws=ws, **kw)
    xp, dp, hp = B.solve(M, b, ws=ws, profile=1, **kw)
    assert torch.equal(x, xp) == same  # together, the cycle kernel's order of sums
    torch.cuda.synchronize()
    with busy:
        xb, db, hb = B.solve(M, b, ws=ws, **kw)
        assert busy.running()
    assert db["status"] == dp["status"]
    assert all(db[k] == dp[k] for k in ("iters", "refinements", "cycles"))
    assert torch.equal(xb, xp) and np.array_equal(hb, hp)
    M.close()


def test_features_beside_a_long_kernel(busy):
    say("features beside a long kernel")
    M, b = system(262144)
    f = B.gmresir_features(M, b)
    with busy:
        fb = B.gmresir_features(M, b)
        assert busy.running()
    assert np.array_equal(f, fb)
    M.close()


CHILD = """
import sys, torch
sys.path[:0] = {paths!r}
from paper_2109_01232_amd import binding as B
from test_gpu_shared_device import system
M, b = system(300000)
kw = dict(restart=30, inner="fp32", rtol=1e-11, max_iters=150)
xs = [B.solve(M, b, profile=1, **kw)[0]]
for i in range(25):
    x, d, _ = B.solve(M, b, **kw)
    torch.cuda.synchronize()
    assert d["rel_resid_true"] <= 1e-11, d
    assert (x - xs[0]).norm() <= 1e-9 * x.norm()
    print("solve", i, flush=True)
print("ok", flush=True)
"""


def test_two_processes(busy):
    say("two processes")
    here = os.path.dirname(os.path.abspath(__file__))
    code = CHILD.format(paths=[os.path.dirname(here), here])
    procs = [subprocess.Popen([sys.executable, "-c", code], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
             for _ in range(2)]
    try:
        outs = [p.communicate(timeout=90)[0] for p in procs]
    finally:
        for p in procs:
            if p.poll() is None:
                p.kill()
    assert all(p.returncode == 0 and o.rstrip().endswith("ok") for p, o in zip(procs, outs)), outs
