"""y = H x from the stored H where a block of rows stages its parts of x, at the
edges of its blocks and batches: blocks of 32 rows and more, one and two blocks of
an alpha string, rows without singles, rows of x that fit the LDS sixteen times,
twice and once, strings whose alpha neighbours fill one and several batches; and
beside them shapes that take the rows from the L2.  Against the stored elements
multiplied on the host in extended precision.  Bar: 4e-14 of sum |H| |x| of the row:
a lane adds at most 180 elements of a row (of up to 11000, every 64th), the exchange
six more, each with a rounding of 1.1e-16, and twice that is allowed."""
import numpy as np
import pytest

from paper_2601_16169_amd import inputs as I
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norb,nel,na,nb", [
    (10, 5, 252, 252), (12, 6, 540, 32), (12, 6, 540, 31), (12, 6, 300, 129), (12, 6, 256, 130), (12, 6, 400, 257),
    (16, 8, 600, 516), (16, 2, 120, 120), (16, 8, 20, 5000), (16, 8, 70, 3000), (14, 1, 14, 14), (16, 8, 2000, 33),
    (12, 6, 924, 64)])
def test_stored_rows(norb, nel, na, nb):
    torch = need_gpu()
    banner(f"stored rows norb {norb} {na} x {nb}")
    from paper_2601_16169_amd import sqd
    ints = I.make_integrals(norb, 2 * norb, seed=3)
    every = I.all_strings(norb, nel)
    ctx = sqd.Context(0)
    try:
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        sp = ctx.build_space(nel, nel, I.random_subset(every, na, 11), I.random_subset(every, nb, 12))
        nnz = sp.store_hamiltonian()
        rp, col, val = sp.stored_hamiltonian(nnz)
        x = np.random.default_rng(5).standard_normal(sp.dim)
        y = sp.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
        ref = np.add.reduceat((val * x[col]).astype(np.longdouble), rp[:-1]).astype(np.float64)
        size = np.add.reduceat(np.abs(val * x[col]), rp[:-1])
        assert (np.abs(y - ref) <= 4e-14 * size).all()
        # an infinity reaches the rows that hold its column, and no others
        j = sp.dim // 2
        x[j] = np.inf
        y = sp.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
        hit = np.add.reduceat((col == j).astype(np.int64), rp[:-1]) > 0
        assert np.isfinite(y[~hit]).all() and not np.isfinite(y[hit]).any()
        sp.close()
    finally:
        ctx.close()


def test_stored_rows_graph_replays():
    """The staged product captured in a HIP graph, without an eager call of it
    before: every replay equals the eager product, bit for bit, with eager products
    of another vector between the replays."""
    torch = need_gpu()
    banner("stored rows graph capture")
    from paper_2601_16169_amd import sqd
    stream = torch.cuda.Stream()
    ctx = sqd.Context(0, stream)
    try:
        ints = I.make_integrals(10, 20, seed=3)
        every = I.all_strings(10, 5)
        ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
        sp = ctx.build_space(5, 5, every, every[:130].copy())
        sp.store_hamiltonian()
        with torch.cuda.stream(stream):
            c, c2 = (torch.tensor(I.random_vector(sp.dim, k), device="cuda:0") for k in (23, 24))
            out, other = torch.empty_like(c), torch.empty_like(c)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sp.spmv(c, out)
        with torch.cuda.stream(stream):
            eager = sp.spmv(c).clone()
        for rep in range(4):
            with torch.cuda.stream(stream):
                out.fill_(float("nan"))
                graph.replay()
            stream.synchronize()
            assert torch.equal(out, eager), f"replay {rep} differs"
            with torch.cuda.stream(stream):
                sp.spmv(c2, other)
            stream.synchronize()
        sp.close()
    finally:
        ctx.close()
