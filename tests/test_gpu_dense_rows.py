"""Products over dense sets of long strings at the lines where the one launch gives way to
the separate kernels: two whole rows against windows (896 beta strings beside longer alpha
rows, 1844 alpha strings beside longer beta rows), one round of four-row workgroups (921 to
1024 beta strings), two rounds in FP32 (2048).  The automatic choice against the row-staged
kernels that a caller chooses (FP64 1e-12, FP32 2e-6, the bars of every sigma test); solves
in both modes against each other, and a captured product against its eager call."""
import pytest

from paper_2601_16169_amd import inputs as I
from tests.gpu_util import banner, need_gpu, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb", [
    (4900, 895), (4900, 896), (1843, 4900), (1844, 4900),
    (4000, 920), (4000, 921), (4000, 1024), (4000, 1025),
    (3800, 2048), (3800, 2049),
])
def test_products_at_the_lines(na, nb):
    torch = need_gpu()
    from paper_2601_16169_amd import sqd
    banner(f"dense rows: {na} x {nb}")
    every = I.all_strings(16, 8)
    ints = I.make_integrals(16, 8, 5, diag_range=(-10.0, 2.0))
    stream = torch.cuda.Stream()
    ctx = sqd.Context(0, stream)
    try:
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        sp = ctx.build_space(8, 8, I.random_subset(every, na, 1), I.random_subset(every, nb, 2))
        i = sp.info()
        long = int(nb > na)
        assert i["nnz_single"][long] + i["nnz_double"][long] > 235 * max(na, nb)
        with torch.cuda.stream(stream):
            c = torch.tensor(I.random_vector(sp.dim, 3), device="cuda:0")
            out = torch.empty_like(c)
            for prec, bar in ((sqd.FP64, 1e-12), (sqd.FP32, 2e-6)):
                got = sp.sigma(c, precision=prec)
                ctx.set_tuning(sqd.TUNE_SS_WINDOW, 1)
                ctx.set_tuning(sqd.TUNE_AB_VARIANT, 2)
                ref = sp.sigma(c, precision=prec)
                ctx.set_tuning(sqd.TUNE_SS_WINDOW, 0)
                ctx.set_tuning(sqd.TUNE_AB_VARIANT, 0)
                stream.synchronize()
                assert max(rel_err(got.cpu().numpy(), ref.cpu().numpy())) <= bar, prec
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=stream):
                    sp.sigma(c, out, precision=prec)
                for _ in range(3):
                    out.fill_(float("nan"))
                    graph.replay()
                    stream.synchronize()
                    assert torch.equal(out, got), prec
                del graph
            e = [sp.davidson(tol=1e-8, max_iter=100, mode=m)[0] for m in (sqd.DAV_FP64, sqd.DAV_MIXED)]
        stream.synchronize()
        assert abs(e[0] - e[1]) <= 1e-9 * abs(e[0])
        sp.close()
    finally:
        ctx.close()
