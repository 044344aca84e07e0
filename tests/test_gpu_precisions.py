"""Products of both precisions on one space whose rows the one launch takes two at
a time in FP64 and four in FP32 (more than 4863 and up to about 10000 strings): the
two use different schedules of the alpha-beta term, and neither may take the other's
away.  A captured product is replayed after eager products of the other precision, a
mixed solve and a batched solve, and a product whose eager call came before those of
the other precision can still be captured.  Replays are compared with an eager call
bit for bit: the same kernels on the same tables."""
import numpy as np
import pytest

from paper_2601_16169_amd import inputs as I
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb", [(60, 5000), (5300, 40)])
@pytest.mark.parametrize("precision", [0, 1])
def test_capture_beside_the_other_precision(na, nb, precision):
    torch = need_gpu()
    from paper_2601_16169_amd import sqd
    banner(f"captured beside the other precision: {na} x {nb} precision {precision}")
    every = I.all_strings(16, 8)
    ints = I.make_integrals(16, 8, 5)
    stream = torch.cuda.Stream()
    ctx = sqd.Context(0, stream)
    try:
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        sp = ctx.build_space(8, 8, I.random_subset(every, na, 1), I.random_subset(every, nb, 2))
        with torch.cuda.stream(stream):
            c = torch.tensor(I.random_vector(sp.dim, 3), device="cuda:0")
            out, other, x = torch.empty_like(c), torch.empty_like(c), torch.empty_like(c)
            ref = sp.sigma(c, precision=precision)
            first_other = sp.sigma(c, precision=1 - precision)   # before the capture
            sp.davidson(tol=1e-3, max_iter=3, mode=sqd.DAV_MIXED, out=x)   # ... and the largest scratch
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sp.sigma(c, out, precision=precision)
        between = [lambda: None,
                   lambda: sp.sigma(c, other, precision=1 - precision),
                   lambda: sp.davidson(tol=1e-3, max_iter=3, mode=sqd.DAV_MIXED, out=x),
                   lambda: ctx.davidson_batched([sp], tol=1e-3, max_iter=3, mode=sqd.DAV_MIXED)]
        for k, f in enumerate(between):
            with torch.cuda.stream(stream):
                f()
                out.fill_(float("nan"))
                graph.replay()
            stream.synchronize()
            assert torch.equal(out, ref), k
        with torch.cuda.stream(stream):
            sp.sigma(c, other, precision=1 - precision)
        stream.synchronize()
        assert torch.equal(other, first_other)
        # the other precision's product, captured after this one's
        graph2 = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph2, stream=stream):
            sp.sigma(c, other, precision=1 - precision)
        with torch.cuda.stream(stream):
            other.fill_(float("nan"))
            graph2.replay()
            graph.replay()
        stream.synchronize()
        assert torch.equal(other, first_other) and torch.equal(out, ref)
        sp.close()
    finally:
        ctx.close()
