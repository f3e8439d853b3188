"""The work this library is timed on: solves, products, matrix set-up, training.

Every case goes through the public entry points (`paper_2109_01232_amd.binding`
and the C ABI under it) as a user's program calls them: the matrix handle and
the workspace are made once, a pass is one call on them.  Inputs are made on
the GPU from the seed alone, with the stencils and distributions of
`paper_2109_01232_amd.problems` (the same formulas, drawn by torch so that the
large systems take a fraction of a second).

Solves run to a relative residual of 1e-12 from x0 = 0, the tolerance at which
the repository compares solutions, and return the whole fp64 solution; the
right-hand side is b = A u, so u is the exact answer.
"""

import ctypes
import math

import torch

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

RTOL = 1e-12
DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _solve(name, family, n, inner, basis, m, iters, ortho=0, degree=0, bj=0):
    return {"name": name, "kind": "solve", "family": family, "n": n, "inner": inner, "basis": basis, "m": m,
            "iters": iters, "ortho": ortho, "degree": degree, "bj": bj}


def listed():
    return [
        # the smallest systems: 64^2 = 4096 rows (the repository's parity system), bound by launches and latency
        _solve("solve_2d_64_fp32", "convdiff2d", 64, "fp32", "fp32", 50, 530),
        # small, odd-sized, plain fp64 GMRES: the method GMRES-IR is measured against
        _solve("solve_2d_171_fp64", "convdiff2d", 171, "fp64", "fp64", 50, 800),
        # middle of the parameter chooser's population (1e4 .. 2e6 rows), wide rows, bf16-stored basis
        _solve("solve_27pt_45_bf16", "varcoef27", 45, "fp32", "bf16", 50, 325),
        # the 2D benchmark system (10^6 rows, 5 nonzeros per row) with GMRES-IR
        _solve("solve_2d_1000_fp32", "convdiff2d", 1000, "fp32", "fp32", 50, 3000),
        # the headline benchmark: 27-point 128^3, GMRES-IR with an fp32 and a bf16 basis
        _solve("solve_27pt_128_fp32", "varcoef27", 128, "fp32", "fp32", 50, 285),
        _solve("solve_27pt_128_bf16", "varcoef27", 128, "fp32", "bf16", 50, 330),
        # fp64 GMRES on a large odd-sized system of the same family
        _solve("solve_27pt_101_fp64", "varcoef27", 101, "fp64", "fp64", 50, 280),
        # the 3D anisotropic system with a long restart and the one-reduction CGS2
        _solve("solve_3d_150_dcgs2", "aniso3d", 150, "fp32", "fp32", 100, 1930, ortho=1),
        # polynomial preconditioner, its set-up in the call as in every use of it
        _solve("solve_3d_101_poly10", "aniso3d", 101, "fp32", "fp32", 50, 205, degree=10),
        # matrix products alone, both precisions: the repository's SpMV study (13-point, 1500^2)
        {"name": "spmv_2d13_1500", "kind": "spmv", "family": "biharmonic2d_13", "n": 1500},
        # a new matrix: the handle with its copies from CSR arrays on the GPU, and the first products
        {"name": "setup_3d_150", "kind": "setup", "family": "laplace3d_7", "n": 150},
        # one step of the parameter chooser's training (forward, backward, Adam) at its batch size
        {"name": "train_256", "kind": "train", "batch": 256},
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["solve"] * 6 + ["spmv", "setup", "train"])
    if kind == "train":
        return {"kind": "train", "batch": logint(7, 1024)}
    if kind in ("spmv", "setup"):
        family = rng.choice(sorted(P.STENCILS))
        rows = logint(4e3, 2.25e6)
        n = max(8, int(round(rows ** (1.0 / P.STENCILS[family][0]))))
        return {"kind": kind, "family": family, "n": n}
    family = rng.choice(["convdiff2d", "aniso3d", "varcoef27", "varcoef27"])
    inner = rng.choice(["fp32", "fp32", "fp64"])
    basis = "bf16" if family == "varcoef27" and inner == "fp32" and rng.random() < 0.4 else inner
    option = rng.choice(["plain", "plain", "ortho", "poly", "bj"])
    if basis == "bf16" and option == "ortho":
        option = "plain"
    dim = 2 if family == "convdiff2d" else 3
    rows = logint(1e3, 1.6e5 if dim == 2 else 1.5e6)
    n = max(10, int(round(rows ** (1.0 / dim))))
    m = rng.choice([30, 50, 50, 75, 100])
    iters = {"convdiff2d": 4 * n, "aniso3d": 11 * n, "varcoef27": 280}[family]
    if option == "poly":
        iters = max(10, iters // 8)
    case = _solve(None, family, n, inner, basis, m, iters, ortho=1 if option == "ortho" else 0,
                  degree=rng.choice([5, 10, 20]) if option == "poly" else 0,
                  bj=rng.choice([8, 16]) if option == "bj" else 0)
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# inputs, on the GPU
# ---------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(g, n, dtype=torch.float64):
    return torch.rand(n, generator=g, device=DEV, dtype=dtype) * 2 - 1


class _Stencil:
    """A table of values [rows][entries] over sorted stencil offsets."""

    def __init__(self, dim, n, offsets):
        self.N = n ** dim
        order = sorted(offsets, key=lambda o: sum(c * n ** d for d, c in enumerate(o)))
        self.offsets = order
        self.lin = [sum(c * n ** d for d, c in enumerate(o)) for o in order]
        idx = torch.arange(self.N, device=DEV)
        coords = [(idx // n ** d) % n for d in range(dim)]
        self.valid = torch.ones(self.N, len(order), dtype=torch.bool, device=DEV)
        for k, o in enumerate(order):
            for d, c in enumerate(o):
                if c:
                    self.valid[:, k] &= (coords[d] + c >= 0) & (coords[d] + c < n)
        self.vals = torch.zeros(self.N, len(order), dtype=torch.float64, device=DEV)

    def product(self, u):
        y = torch.zeros(self.N, dtype=torch.float64, device=DEV)
        idx = torch.arange(self.N, device=DEV)
        for k, o in enumerate(self.lin):
            y += torch.where(self.valid[:, k], self.vals[:, k] * u[(idx + o).clamp(0, self.N - 1)], 0.0)
        return y

    def csr(self):
        idx = torch.arange(self.N, device=DEV, dtype=torch.int32)
        lin = torch.tensor(self.lin, device=DEV, dtype=torch.int32)
        rowptr = torch.zeros(self.N + 1, dtype=torch.int32, device=DEV)
        rowptr[1:] = self.valid.sum(1).cumsum(0).to(torch.int32)
        return rowptr, (idx[:, None] + lin)[self.valid], self.vals[self.valid]


def _conv_diff(dim, n, Pe, kdiff):
    """Centred differences of -div(K grad u) + Pe (w . grad u), wind (1, .., 1), scaled by h^2."""
    unit = [tuple(1 if e == d else 0 for e in range(dim)) for d in range(dim)]
    offs = [(0,) * dim] + unit + [tuple(-c for c in o) for o in unit]
    S = _Stencil(dim, n, offs)
    h = 1.0 / (n + 1)
    for k, o in enumerate(S.offsets):
        d = next((e for e, c in enumerate(o) if c), None)
        S.vals[:, k] = 2.0 * sum(kdiff) if d is None else -kdiff[d] + o[d] * Pe * h / 2.0
    return S


def _varcoef27(n, g, shift=0.05):
    """The nonsymmetric variable-coefficient 27-point M-matrix with row sums `shift`."""
    S = _Stencil(3, n, [(x, y, z) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1)])
    for t in range(14, 27):
        o = S.lin[t]
        xi, eta, s = (_uniform(g, S.N) for _ in range(3))
        S.vals[:, t] = -(1.0 + 0.3 * xi) + 0.5 * s
        S.vals[o:, 26 - t] = (-(1.0 + 0.3 * eta) - 0.5 * s)[: S.N - o]
    S.vals *= S.valid
    S.vals[:, 13] = shift - S.vals.sum(1)
    return S


def _stencil_of(case, g):
    family, n = case["family"], case["n"]
    if family == "convdiff2d":
        Pe = 60.0 + 40.0 * float(torch.rand(1, generator=g, device=DEV))
        return _conv_diff(2, n, Pe, (1.0, 1.0))
    if family == "aniso3d":
        return _conv_diff(3, n, 10.0, (1.0, 1.0, 1e-2))
    if family == "varcoef27":
        return _varcoef27(n, g)
    dim, pattern = P.STENCILS[family]
    S = _Stencil(dim, n, [o for o, _ in pattern])
    coef = dict(pattern)
    for k, o in enumerate(S.offsets):
        S.vals[:, k] = coef[o]
    return S


def _system(case, seed):
    """(stencil, u) of a case: the matrix first, then the vector, from one generator."""
    g = _generator(seed)
    S = _stencil_of(case, g)
    return S, _uniform(g, S.N)


def _train_inputs(case, seed):
    """A batch of chooser samples and the network in mid-training: features of their usual magnitudes, labels on
    the chooser's grid, weights of Glorot size, Adam moments of the gradients' size."""
    g = _generator(seed)
    nb = case["batch"]
    X = torch.randn(nb, 16, generator=g, device=DEV) * 2 + 1
    T = torch.stack([torch.rand(nb, generator=g, device=DEV) * 4.4 + 3.3, torch.rand(nb, generator=g, device=DEV) * 2,
                     torch.rand(nb, generator=g, device=DEV)], 1)
    parts = []
    for fi, fo in ((16, 64), (64, 64), (64, 3)):
        lim = math.sqrt(6.0 / (fi + fo))
        parts += [_uniform(g, fi * fo, torch.float32) * lim, _uniform(g, fo, torch.float32) * 0.1]
    params = torch.cat(parts)
    m = torch.randn(params.numel(), generator=g, device=DEV) * 0.02
    v = (torch.rand(params.numel(), generator=g, device=DEV) + 0.1) * 1e-3
    shift = torch.full((16,), 1.0, device=DEV)
    scale = torch.full((16,), 0.5, device=DEV)
    return {"params": params, "m": m, "v": v, "shift": shift, "scale": scale, "X": X, "T": T.contiguous()}


LR, STEP = 3e-3, 500


def prepare(case, seed):
    if case["kind"] == "train":
        return {"case": case, "loss": torch.zeros(1, device=DEV)} | _train_inputs(case, seed)
    S, u = _system(case, seed)
    state = {"case": case}
    if case["kind"] == "solve":
        state["b"] = S.product(u)
        state["x"] = torch.zeros_like(u)
        state["ws"] = B.Workspace()
        state["params"] = B.make_params(restart=case["m"], inner=case["inner"], basis=case["basis"], rtol=RTOL,
                                        max_iters=40000, check_mode=1, poly_degree=case["degree"],
                                        bj_block=case["bj"], ortho=case["ortho"])
        state["matrix"] = B.Matrix(*(t.cpu().numpy() for t in S.csr()))
        return state
    state["x64"], state["x32"] = u, u.float()
    state["y64"], state["y32"] = torch.empty_like(u), torch.empty_like(state["x32"])
    if case["kind"] == "spmv":
        state["matrix"] = B.Matrix(*(t.cpu().numpy() for t in S.csr()))
    else:
        state["csr"] = S.csr()
        nbytes = B.lib().gmresir_matrix_storage_bytes(S.N, state["csr"][1].numel())
        state["storage"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

class _Handle:
    """A matrix handle made from CSR arrays that are on the GPU already."""

    def __init__(self, rowptr, colidx, vals, storage):
        self.handle = ctypes.c_void_p()
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        st = B.lib().gmresir_matrix_create(rowptr.numel() - 1, colidx.numel(), rowptr.data_ptr(), colidx.data_ptr(),
                                           vals.data_ptr(), storage.data_ptr(), storage.numel(), stream,
                                           ctypes.byref(self.handle))
        if st != B.OK:
            raise B.GmresirError("gmresir_matrix_create", st)

    def close(self):
        B.lib().gmresir_matrix_destroy(self.handle)


def run(state):
    case = state["case"]
    if case["kind"] == "solve":
        M, ws = state["matrix"], state["ws"]
        state["x"].zero_()
        roots = B.gmresir_poly_setup(M, case["degree"], seed=12345, ws=ws) if case["degree"] else None
        st, _, _ = B.gmresir_solve(M, state["b"], state["x"], state["params"], poly_roots=roots, ws=ws)
        if st != B.OK:
            raise RuntimeError("not converged: status %d" % st)
        return state["x"]
    if case["kind"] == "train":
        B.gmresir_mlp_train_step(state["params"], state["m"], state["v"], state["shift"], state["scale"], state["X"],
                                 state["T"], LR, STEP, state["loss"])
        return {"params": state["params"], "m": state["m"], "v": state["v"], "loss": state["loss"]}
    M = state["matrix"] if case["kind"] == "spmv" else _Handle(*state["csr"], state["storage"])
    B.gmresir_spmv(M, state["x64"], state["y64"], "fp64")
    B.gmresir_spmv(M, state["x32"], state["y32"], "fp32")
    if case["kind"] == "setup":
        M.close()
    return {"y64": state["y64"], "y32": state["y32"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without, and its exact results
# ---------------------------------------------------------------------------

def _counts(case):
    """(rows, nonzeros) of a case's matrix."""
    family, n = case["family"], case["n"]
    if family == "convdiff2d":
        return n * n, P.stencil_nnz_2d5(n)
    if family == "aniso3d":
        return n ** 3, P.stencil_nnz_3d7(n)
    if family == "varcoef27":
        return n ** 3, P.stencil_nnz_27(n)
    return n ** P.STENCILS[family][0], P.stencil_nnz(family, n)


def work(case):
    """Bytes and flops of one pass.  A solve counts `iters` inner iterations (what the systems of its kind take):
    the matrix values once, the vectors in and out, and the basis (on average half of m columns) once for each
    data-dependent pass over it -- three for two-pass CGS2, two for the one-reduction form; a polynomial adds its
    products, block Jacobi its inverses.  The matrix's structure is not counted: a stencil needs no index per entry."""
    if case["kind"] == "train":
        nb, npar = case["batch"], 5443
        return {"bytes": 4.0 * (nb * 19 + 6 * npar), "flops": 6.0 * npar * nb}
    N, nnz = _counts(case)
    if case["kind"] == "spmv":
        return {"bytes": 12.0 * nnz + 24.0 * N, "flops": 4.0 * nnz}
    if case["kind"] == "setup":
        # CSR read, both sliced copies and the fp32 CSR copy written, then the two products
        return {"bytes": (12.0 + 16.0) * nnz + 4.0 * N + 12.0 * nnz + 24.0 * N, "flops": 4.0 * nnz}
    sT = 8 if case["inner"] == "fp64" else 4
    sS = {"fp64": 8, "fp32": 4, "bf16": 2}[case["basis"]]
    cols = min(case["m"], case["iters"]) / 2.0
    sweeps = 2 if case["ortho"] else 3
    products = 1 + case["degree"]
    per_iter = products * (sT * nnz + 2.0 * sT * N) + sweeps * sS * N * cols + case["bj"] * sT * N
    flops = 2.0 * nnz * products + 8.0 * N * cols + 2.0 * case["bj"] * N
    return {"bytes": per_iter * case["iters"], "flops": flops * case["iters"]}


def _exact_train(case, seed):
    s = {k: t.double() for k, t in _train_inputs(case, seed).items()}
    P0 = s["params"].clone().requires_grad_(True)
    at, W = 0, []
    for fi, fo in ((16, 64), (64, 64), (64, 3)):
        W.append((P0[at:at + fi * fo].view(fi, fo), P0[at + fi * fo:at + fi * fo + fo]))
        at += fi * fo + fo
    h = (s["X"] - s["shift"]) * s["scale"]
    h = torch.tanh(h @ W[0][0] + W[0][1])
    h = torch.tanh(h @ W[1][0] + W[1][1])
    y = h @ W[2][0] + W[2][1]
    loss = ((y - s["T"]) ** 2).mean()
    (g,) = torch.autograd.grad(loss, P0)
    m = 0.9 * s["m"] + 0.1 * g
    v = 0.999 * s["v"] + 0.001 * g * g
    step = LR * (m / (1 - 0.9 ** STEP)) / ((v / (1 - 0.999 ** STEP)).sqrt() + 1e-8)
    return {"params": (P0 - step).detach(), "m": m, "v": v, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    S, u = _system(case, seed)
    if case["kind"] == "solve":
        return u
    y = S.product(u)
    return {"y64": y, "y32": S.product(u.float().double())}
