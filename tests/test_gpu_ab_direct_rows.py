"""The row-staged alpha-beta kernel (sqd_sigma_noalloc; SQD_TUNE_AB_VARIANT 2) on rows
around the sixteen entries that a lane has at hand, with more slices than one group of
waves takes, and with one or two sources a pass, against the oracle: FP64 1e-12, FP32
2e-6, the bars of every sigma test."""
import pytest

from paper_2601_16169_amd import inputs as I
from oracle import core
from tests.gpu_util import banner, need_gpu, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norb,nea,neb,na,nb", [
    (6, 3, 1, 20, 6),        # five singles a row: four and one
    (9, 3, 1, 20, 9),        # eight: one pair of blocks, nothing left
    (10, 3, 1, 20, 10),      # nine
    (7, 3, 3, 30, 35),       # twelve: a pair of blocks and one
    (12, 4, 4, 9, 495),      # 32
    (16, 8, 8, 40, 1),       # no singles
    (16, 8, 8, 30, 4500),    # 71 slices: two groups of waves; four sources in FP32
    (16, 8, 8, 12, 9800),    # one source a pass (FP64), 154 slices
])
def test_row_staged_alpha_beta(norb, nea, neb, na, nb):
    torch = need_gpu()
    from paper_2601_16169_amd import sqd
    banner(f"row-staged alpha-beta: norb {norb}, {na} x {nb}")
    ints = I.make_integrals(norb, 2 * norb, 9)
    a, b = I.all_strings(norb, nea), I.all_strings(norb, neb)
    p = I.Problem("ab_direct", ints, nea, neb, I.random_subset(a, min(na, len(a)), 1), I.random_subset(b, min(nb, len(b)), 2))
    ctx = sqd.Context(0)
    try:
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        sp = ctx.build_space(nea, neb, p.astr, p.bstr)
        c = I.random_vector(sp.dim, 3)
        ct = torch.tensor(c, device="cuda:0")
        ref = core.Space.from_problem(p).sigma(c)
        for prec, bar in ((sqd.FP64, 1e-12), (sqd.FP32, 2e-6)):
            sp.sigma(ct, precision=prec)
            out = torch.full_like(ct, float("nan"))
            sp.sigma_noalloc(ct, out, precision=prec)
            assert max(rel_err(out.cpu().numpy(), ref)) <= bar, (prec, rel_err(out.cpu().numpy(), ref))
            ctx.set_tuning(sqd.TUNE_AB_VARIANT, 2)
            got = sp.sigma(ct, precision=prec)
            ctx.set_tuning(sqd.TUNE_AB_VARIANT, 0)
            assert max(rel_err(got.cpu().numpy(), ref)) <= bar, (prec, rel_err(got.cpu().numpy(), ref))
        sp.close()
    finally:
        ctx.close()
