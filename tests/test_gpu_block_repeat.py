"""Block Davidson solves repeat bit for bit: every reduction of the solver adds in a
fixed order, and every element of the projected matrix has one writer.  Two to eight
roots (four and eight columns a launch; the new columns within one group of eight
rows of the basis and across two), FP64 and mixed."""
import pytest

from paper_2601_16169_amd import inputs as I
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nroots,m_max", [(2, 24), (3, 24), (5, 32), (8, 32)])
@pytest.mark.parametrize("mixed", [False, True])
def test_block_solves_repeat(nroots, m_max, mixed):
    torch = need_gpu()
    from paper_2601_16169_amd import sqd
    banner(f"block solves repeat: {nroots} roots, mixed {mixed}")
    p = I.small_problem(12, 5, 4, 201, 163, 7)
    ctx = sqd.Context(0)
    try:
        ctx.set_hamiltonian(p.ints.h, p.ints.eri, p.ints.ecore)
        sp = ctx.build_space(p.nalpha, p.nbeta, p.astr, p.bstr)
        runs = [sp.davidson_block(nroots, tol=1e-9, max_iter=60, m_max=m_max,
                                  mode=sqd.DAV_MIXED if mixed else sqd.DAV_FP64) for _ in range(4)]
        e0, x0, r0 = runs[0][:3]
        for e, x, r in (q[:3] for q in runs[1:]):
            assert list(e) == list(e0)
            assert torch.equal(x, x0)
            assert [q["iterations"] for q in r] == [q["iterations"] for q in r0]
        sp.close()
    finally:
        ctx.close()
