"""Products captured in a HIP graph on a space whose earlier calls were others:
the terms by themselves after whole products only, the whole product after single
terms only, and density matrices on a space that had none before (another space's
call has grown the scratch).  Rows that the one launch takes four and two at a
time, and rows that the separate launches walk by windows.  Every replay is
compared with the eager call made afterwards: FP64 1e-12 and FP32 2e-6 in the
norms of every sigma test (the routes may differ in the order of their sums)."""
import numpy as np
import pytest

from paper_2601_16169_amd import inputs as I
from tests.gpu_util import banner, need_gpu, rel_err

pytestmark = pytest.mark.gpu


def _replays(torch, stream, call, between, out):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call()
    got = []
    for _ in range(3):
        with torch.cuda.stream(stream):
            out.fill_(float("nan"))
            graph.replay()
        stream.synchronize()
        got.append(out.cpu().numpy())
        with torch.cuda.stream(stream):
            between()
        stream.synchronize()
    return got


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("na,nb", [(70, 97), (60, 5000), (5000, 40)])
@pytest.mark.parametrize("before", ["whole", "terms"])
def test_captured_after_others(na, nb, precision, before):
    torch = need_gpu()
    from paper_2601_16169_amd import sqd
    banner(f"captured after {before}: {na} x {nb} precision {precision}")
    every = I.all_strings(16, 8)
    ints = I.make_integrals(16, 8, 5)
    stream = torch.cuda.Stream()
    ctx = sqd.Context(0, stream)
    try:
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        sp = ctx.build_space(8, 8, I.random_subset(every, na, 1), I.random_subset(every, nb, 2))
        singles = [sqd.TERM_AA, sqd.TERM_BB, sqd.TERM_AB]
        whole = sqd.TERM_DIAG | sqd.TERM_AA | sqd.TERM_BB | sqd.TERM_AB
        with torch.cuda.stream(stream):
            c = torch.tensor(I.random_vector(sp.dim, 3), device="cuda:0")
            c2 = torch.tensor(I.random_vector(sp.dim, 4), device="cuda:0")
            out, other = torch.empty_like(c), torch.empty_like(c)
            for terms in [whole] if before == "whole" else singles:
                sp.sigma(c, out, precision=precision, terms=terms)
        stream.synchronize()
        masks = singles if before == "whole" else [whole]
        eager_mask = whole if before == "whole" else sqd.TERM_AB
        got = {}
        for terms in masks:
            got[terms] = _replays(torch, stream, lambda: sp.sigma(c, out, precision=precision, terms=terms),
                                  lambda: sp.sigma(c2, other, precision=precision, terms=eager_mask), out)
        for terms in masks:
            with torch.cuda.stream(stream):
                ref = sp.sigma(c, precision=precision, terms=terms)
            stream.synchronize()
            for k, y in enumerate(got[terms]):
                assert max(rel_err(y, ref.cpu().numpy())) <= (2e-6 if precision else 1e-12), (terms, k)
        sp.close()
    finally:
        ctx.close()


def test_captured_first_rdm():
    torch = need_gpu()
    from paper_2601_16169_amd import sqd
    banner("captured first rdm")
    stream = torch.cuda.Stream()
    ctx = sqd.Context(0, stream)
    try:
        every = I.all_strings(10, 5)
        ints = I.make_integrals(10, 20, 5)
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        first, sp = (ctx.build_space(5, 5, I.random_subset(every, n, 1), I.random_subset(every, n - 7, 2))
                     for n in (200, 150))
        with torch.cuda.stream(stream):
            first.rdm(torch.tensor(I.random_vector(first.dim, 2), device="cuda:0"))
            c = torch.tensor(I.random_vector(sp.dim, 3), device="cuda:0")
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out1, out2 = sp.rdm(c)
        got = []
        for _ in range(3):
            with torch.cuda.stream(stream):
                out1.fill_(float("nan"))
                out2.fill_(float("nan"))
                graph.replay()
            stream.synchronize()
            got.append((out1.cpu().numpy(), out2.cpu().numpy()))
            with torch.cuda.stream(stream):
                first.rdm(torch.tensor(I.random_vector(first.dim, 4), device="cuda:0"))
            stream.synchronize()
        with torch.cuda.stream(stream):
            r1, r2 = sp.rdm(c)
        stream.synchronize()
        for g1, g2 in got:
            assert max(rel_err(g1, r1.cpu().numpy())) <= 1e-12 and max(rel_err(g2, r2.cpu().numpy())) <= 1e-12
        first.close()
        sp.close()
    finally:
        ctx.close()
