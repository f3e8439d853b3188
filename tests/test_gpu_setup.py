"""Matrix set-up on the GPU against a plain restatement of its rules.

The tile table, the layout choice, the slice pointers, the offset lists and
the values of the sliced copy are read back from the matrix storage and
compared exactly (they are integers and copies of the input)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B
from paper_2109_01232_amd import problems as P

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def random_rows(n, lens, seed, span=None):
    """Rows of the given lengths, ascending columns (within `span` of the row if given)."""
    rng = np.random.default_rng(seed)
    cols = []
    for r in range(n):
        lo, hi = (0, n) if span is None else (max(0, r - span), min(n, r + span + 1))
        cols.append(lo + np.sort(rng.choice(hi - lo, min(int(lens[r]), hi - lo), replace=False)))
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])])
    return P.CSR(n, rowptr.astype(np.int32), np.concatenate(cols).astype(np.int32), rng.standard_normal(rowptr[-1]))


def greedy_tiles(rp):
    """At most 512 rows and 2560 nonzeros, ends on multiples of 8 rows; a longer row alone."""
    n, out = len(rp) - 1, [0]
    while out[-1] < n:
        r0 = out[-1]
        r = min(r0 + 512, int(np.searchsorted(rp, rp[r0] + 2560, side="right")) - 1)
        if r == r0:
            r += 1
        elif r < n and (r & ~7) > r0:
            r &= ~7
        out.append(r)
    return np.array(out)


def check(A):
    rp, ci, n, nnz = A.rowptr.astype(np.int64), A.colidx.astype(np.int64), A.n, A.nnz
    M = B.Matrix.from_csr(A)
    up = lambda v: (v + 255) // 256 * 256
    raw = M.storage.cpu().numpy()
    E = nnz + nnz // 4 + min(n, 4096) * 4
    ns = (n + 63) // 64
    at = [0]
    for size in (4 * nnz, 4 * (n + 1), 4 * (ns + 1), 4 * E, 4 * E, 8 * E):
        at.append(at[-1] + up(size))
    part = lambda k, dt, cnt: raw[at[k]:at[k] + cnt * np.dtype(dt).itemsize].view(dt)
    tiles = greedy_tiles(rp)
    assert M.tiles == len(tiles) - 1
    assert np.array_equal(part(1, np.int32, len(tiles)), tiles)
    assert np.array_equal(part(0, np.float32, nnz), A.vals.astype(np.float32))
    lens = np.diff(rp)
    offs = ci - np.repeat(np.arange(n), lens)
    rows = [np.arange(64 * s, min(n, 64 * s + 64)) for s in range(ns)]
    K = [int(lens[r].max()) for r in rows]
    unions = [np.unique(offs[rp[r[0]]:rp[r[-1] + 1]]) for r in rows]
    ordered = all(np.all(np.diff(offs[rp[i]:rp[i + 1]]) > 0) for i in range(n))
    sell = nnz > 0 and max(K) <= 512 and 64 * sum(K) <= E
    U = [len(u) for u in unions]
    shared = sell and ordered and max(U) <= 512 and 64 * sum(U) <= min(E, 1.25 * 64 * sum(K))
    layout = 0 if not sell else 3 if shared else 2 if np.abs(offs).max() <= 32767 else 1
    assert M.layout == layout
    if sell:
        width = U if shared else K
        sptr = 64 * np.concatenate([[0], np.cumsum(width)])
        assert np.array_equal(part(2, np.int32, ns + 1), sptr)
        v64 = np.zeros(sptr[-1])
        col = np.zeros(sptr[-1], dtype=np.int64)
        for s in range(ns):
            for lane in range(64):
                r = 64 * s + lane
                slots = sptr[s] + 64 * np.arange(width[s]) + lane
                col[slots] = r if r < n else 0
                if r < n:
                    k = np.searchsorted(unions[s], offs[rp[r]:rp[r + 1]]) if shared else np.arange(lens[r])
                    v64[slots[k]] = A.vals[rp[r]:rp[r + 1]]
                    col[slots[k]] = ci[rp[r]:rp[r + 1]]
        assert np.array_equal(part(5, np.float64, sptr[-1]), v64)
        assert np.array_equal(part(4, np.float32, sptr[-1]), v64.astype(np.float32))
        if shared:
            assert np.array_equal(part(3, np.int32, sptr[-1] // 64), np.concatenate(unions))
        elif layout == 2:
            row = np.concatenate([np.tile(np.where(64 * s + np.arange(64) < n, 64 * s + np.arange(64), 0), width[s])
                                  for s in range(ns)])
            assert np.array_equal(part(3, np.int16, sptr[-1]), col - row)
        else:
            assert np.array_equal(part(3, np.int32, sptr[-1]), col)
    M.close()
    return layout


def lengths(n, seed, lo, hi):
    return np.random.default_rng(seed).integers(lo, hi + 1, n)


CASES = {
    # rows around the slice, tile and unit sizes
    **{f"tiny{n}": (lambda n=n: random_rows(n, lengths(n, n, 0, 3), n)) for n in (1, 7, 8, 9, 63, 64, 65, 511, 513)},
    # whole and partial tile segments (8192 rows), one and several
    "stencil_8100": lambda: P.stencil_matrix("laplace2d_5", 90),
    "stencil_16384": lambda: P.stencil_matrix("biharmonic2d_13", 128),
    "stencil_17576": lambda: P.stencil_matrix("box3d_27", 26),
    # tiles cut by nonzeros, rows up to the longest that keeps starts on multiples of 8, and past it
    "row320": lambda: random_rows(9000, np.where(lengths(9000, 1, 0, 99) == 0, 320, 6), 1),
    "row321": lambda: random_rows(9000, np.where(lengths(9000, 2, 0, 99) == 0, 321, 6), 2),
    "row513": lambda: random_rows(3000, np.where(lengths(3000, 3, 0, 99) == 0, 513, 300), 3),
    "row2561": lambda: random_rows(3000, np.where(np.arange(3000) == 1700, 2561, 5), 4),
    # slices wider than a wave stages (mostly 4 entries a row, some slices 60)
    "uneven": lambda: random_rows(20000, np.where(np.arange(20000) // 64 % 40 == 3, 60, 4), 5, span=200),
    # equal rows, far and near columns; few entries in many rows; none at all
    "far": lambda: random_rows(70000, np.full(70000, 3), 6),
    "near": lambda: random_rows(20000, np.full(20000, 9), 7, span=300),
    "sparse": lambda: random_rows(70000, np.where(np.arange(70000) % 1000 == 7, 2, 0), 8),
    "empty": lambda: P.CSR(700, np.zeros(701, np.int32), np.zeros(0, np.int32), np.zeros(0)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_setup_tables(case):
    say("setup", case)
    layout = check(CASES[case]())
    assert layout == {"stencil_8100": 3, "stencil_16384": 3, "stencil_17576": 3, "far": 1, "near": 2, "row513": 0,
                      "row2561": 0, "empty": 0}.get(case, layout)


def test_setup_many_slices_per_block():
    """More than 256 slices per block of the slice-pointer scan: a diagonal
    matrix of 16.8 M rows (one offset per slice)."""
    n = 64 * 256 * 1024 + 64 * 700 + 5
    d = np.random.default_rng(0).uniform(1, 2, n)
    say("setup diagonal", n)
    M = B.Matrix(np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), d)
    assert M.layout == 3 and M.tiles == -(-n // 512)
    x = torch.rand(n, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)
    B.gmresir_spmv(M, x, y, "fp64")
    assert torch.equal(y, torch.from_numpy(d).cuda() * x)


@pytest.mark.parametrize("where,message", [("decrease", "decreases at row 5000"), ("first", "rowptr"),
                                           ("last", "rowptr")])
def test_setup_refuses_bad_row_pointers(where, message):
    """Row pointers that fall, or whose ends are not 0 and nnz: refused, and
    no entry outside the arrays is touched on the way (the set-up kernels
    skip slices whose pointers are out of order or range)."""
    A = P.stencil_matrix("laplace2d_5", 90)
    rp = A.rowptr.copy()
    if where == "decrease":
        rp[5001] = rp[5000] - 3
    elif where == "first":
        rp[0] = 1
    else:
        rp[-1] -= 1
    t = [torch.from_numpy(a).cuda() for a in (rp, A.colidx, A.vals)]
    need = B.lib().gmresir_matrix_storage_bytes(A.n, A.nnz)
    store = torch.empty(need, dtype=torch.uint8, device="cuda")
    import ctypes

    h = ctypes.c_void_p()
    say("setup bad rowptr", where)
    st = B.lib().gmresir_matrix_create(A.n, A.nnz, *(x.data_ptr() for x in t), store.data_ptr(), need, None,
                                       ctypes.byref(h))
    assert st == B.ERR_INVALID_ARG and message in B.last_error() and not h.value
