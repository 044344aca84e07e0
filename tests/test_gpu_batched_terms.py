"""Batches whose rows put their spaces on either side of every choice of the
batched products: four rows in half of the LDS, four rows in all of it, two
rows, and rows too long for two (all spaces by the separate launches); rows of
one string; rows of Y read by one, two and four groups of threads.  Energies
<= 1e-9 Ha against the single-space FP64 solve (both within the square of the
residual tolerance), residuals of the returned vectors with the row-staged
single-space product <= 1e-8 (the tolerance, and rounding)."""
import numpy as np
import pytest

from paper_2601_16169_amd import inputs as I
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [(1, 1), (7, 60), (40, 100), (33, 128), (50, 129), (20, 256), (90, 257)],
    [(300, 300), (2600, 9), (9, 2600)],
    [(64, 65), (2100, 12), (5200, 10), (10, 5200)],
    [(50, 70), (10300, 6)],
], ids=["short", "half", "two_rows", "longest"])
@pytest.mark.parametrize("mode", [0, 1])
def test_batched_rows(sizes, mode):
    need_gpu()
    banner(f"batched rows {sizes} mode {mode}")
    from paper_2601_16169_amd import sqd
    norb, nel = 16, 8
    ints = I.make_integrals(norb, 32, seed=71)
    every = I.all_strings(norb, nel)
    ctx = sqd.Context(0)
    try:
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        spaces = [ctx.build_space(nel, nel, I.random_subset(every, a, 10 * b + a), I.random_subset(every, b, 7 * a + b))
                  for a, b in sizes]
        E, vecs, reps, rc = ctx.davidson_batched(spaces, tol=1e-9, mode=mode, max_iter=300)
        assert rc == 0
        for (a, b), sp, e, v, r in zip(sizes, spaces, E, vecs, reps):
            assert r["converged"], (a, b)
            e1, _, r1 = sp.davidson(tol=1e-9, max_iter=300)
            assert r1["converged"] and abs(e - e1) <= 1e-9, (a, b, e, e1)
            ctx.set_tuning(sqd.TUNE_AB_VARIANT, 2)
            res = float((sp.sigma(v) - e * v).norm())
            ctx.set_tuning(sqd.TUNE_AB_VARIANT, 0)
            assert res <= 1e-8 and abs(float(v.norm()) - 1) <= 1e-12, (a, b, res)
        for sp in spaces:
            sp.close()
    finally:
        ctx.close()
