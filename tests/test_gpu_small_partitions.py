"""Cycle kernel of small systems at the edges of its partition.

A block has 64 RL rows.  RL = 2 and 3 up to 64 blocks, 4, 6, 8, 12 and 16 up to
256, as far as the columns of a wave (4, 8 or 16: restart up to 28, 56 or 112)
times RL fit its registers: 128 values of fp32, 64 of fp64.  The last size of
each and one row more, against the phases launched one by one: the same bits.
With a preconditioner, against the general kernels at the parity bars."""
import pytest

torch = pytest.importorskip("torch")

from paper_2109_01232_amd import binding as B

from gpu_common import say
from test_gpu_small_cycle import KINDS, banded, both
from test_gpu_small_precond import SIDES, compare, roots_of, system

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


def sizes(m, words):
    slots = 4 if m <= 28 else 8 if m <= 56 else 16
    rls = [rl for rl in (2, 3, 4, 6, 8, 12, 16) if slots * rl * words <= 128]
    last = [64 * rl * (64 if rl < 4 else 256) for rl in rls]
    return sorted(set(last + [n + 1 for n in last[:-1]]))


CASES = [(inner, basis, m, n) for inner, basis in KINDS for m in (28, 56, 112)
         for n in sizes(m, 2 if inner == "fp64" else 1)]


@pytest.mark.parametrize("inner,basis,m,n", CASES)
def test_partitions(inner, basis, m, n):
    say("small partitions", inner, basis, m, n)
    both(banded(n, (-300, -1, 0, 1, 300), m), m, inner, basis, m + 3, oracle=n <= 12289 and m == 28)


@pytest.mark.parametrize("inner,basis", KINDS)
@pytest.mark.parametrize("n", [8192, 8193, 12288, 12289])
def test_preconditioned(n, inner, basis):
    say("small partitions, preconditioned", n, inner, basis)
    M, b = system(n, SIDES)
    compare(M, b, 30, inner, basis, 30, bj_block=8)
    compare(M, b, 30, inner, basis, 12, poly_degree=4, poly_roots=roots_of(5, 2))
